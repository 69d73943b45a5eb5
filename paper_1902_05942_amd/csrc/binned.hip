// Insert-accumulate with the cell sums added in LDS by the workgroup that owns
// them, for gfx950.
//
// Device atomics run at ~24 G lines/s on MI355X whatever the footprint, and a
// random access of any kind moves a whole cache line, so the cost of the
// insert is the number of per-cell operations it sends to memory.  This path
// sends one per group of vertices that share a key within a window of up to
// 4096 consecutive vertices, and no device atomic for the sums (but where a bucket
// runs full, or a bin holds more cells than six passes sum):
//   aggregate  per window: the vertices are merged by key in an LDS hash table
//              (count and fixed-point sums added with LDS atomics; the LDS
//              serialises the lanes of a coherent run on one entry more cheaply
//              than a wavefront prefix sum over them costs in VALU work); each
//              group then probes / claims its cell once (compare-and-swap on
//              new cells only) and writes one record {slot, count, sums} into
//              the bucket of its bin (a contiguous slot range); every vertex
//              receives its group's slot.  A window takes its places in all
//              buckets with one device atomic per bin it reaches, so a bin's
//              records of a window are neighbours in memory
//   reduce     per bin: a bitmap of the slots its records name gives every
//              cell a dense index (by population counts), the records are
//              summed in LDS by that index, then count and sums are added to
//              the cells with plain loads and stores by the workgroup that owns
//              them, occupancy bits set; with a temporal blend (Section 3.4.1)
//              in the same launch, the owner also blends each cell's final
//              average with the previous table's value of its key and stores
//              the temporal value
// Integer sums make the result identical to the atomic insert.
//
// What it measured (MI355X; all launches of one call, the temporal blend in
// reduce): 1920x1080x3 vertices (1.1M groups) 163 us, 3840x2160x4 (11M groups)
// 815 us.  The counting sort it replaces (a record of 32 bytes staged per
// workgroup, histograms scanned over the workgroups, records scattered to their
// bins' ranges, LDS sums for every slot of a bin, windows of a fixed 4096
// vertices) took 234 and 1544 us: incoherent vertices hardly merge, so the
// records' way through memory is what the insert costs, and a window of mostly
// distinct keys overflowed its LDS table and sent its vertices to the table one
// by one.  Small calls go another way (small_insert_kernel: device atomics).
#include <mutex>
#include <type_traits>

#include "pf_kernels.h"
#include "pf_merge.h"
#include "pf_once.h"
#include "pf_ops.h"

namespace pfk {

namespace binned {

constexpr int kT = 1024;                     // threads of aggregate
constexpr uint32_t kMaxSteps = 4;            // vertices per thread and chunk, at most
constexpr uint32_t kMaxGroups = 512;         // two workgroups on each of 256 CUs
constexpr uint32_t kFlush = 2;               // LDS entries per thread
constexpr uint32_t kCap = 1920;              // LDS entries of a window
constexpr uint32_t kLimit = kCap / 8 * 7;    // seven eighths full, a free entry is still a few probes away
constexpr uint32_t kMaxLog2Slots = 25;
constexpr uint32_t kSmall = 5u << 16;        // vertices up to which a call has one launch (and the blend's)
constexpr uint32_t kSmallGroups = 192;       // workgroups of such a call before they get twice the threads
constexpr uint32_t kMinWindowed = 1u << 19;  // vertices from which pf_insert_accumulate merges by windows
constexpr uint32_t kMaxBins = 512, kMaxParts = 8;
constexpr uint32_t kMaxLog2BinSlots = 17;    // the bin's bitmap and its prefix counts take 32 KB of LDS
constexpr int kR = 512;                      // threads of reduce: two workgroups on a CU, all bins at once
constexpr uint32_t kCells = 2048;            // cells of a bin summed in LDS at a time
constexpr uint32_t kHold = 4;                // records a thread of reduce keeps in registers
constexpr uint32_t kMark = 16;               // records whose slots are read together after those
constexpr int kPair = 2;                     // cells a thread of reduce updates together

// A record is 16 bytes: one word of slot, count and kind, three of sums.  A
// group whose sums all fit 32 bits and whose count fits 6 is one record; others
// are followed by records of kind 1 that add to the high parts:
//   kind 0: count 1 + c, sums sign-extended;  kind 1: count 64 c, sums << 32.
// (Contributions below 128 / vertices at 24 fraction bits fit one record; with
// 32-byte records of full sums a 3840x2160x4 frame moved twice the bytes.)
constexpr uint32_t kSlotBits = 25, kCountMask = 63u;
static_assert(kMaxLog2Slots == kSlotBits && kSlotBits + 7 == 32, "slot, 6 bits of count and the kind in one word");

// Inputs of key construction when the insert builds the keys itself.
struct FusedKeys {
    const float *px, *py, *pz, *nx, *ny, *nz;
    const uint8_t *valid;
    KeyArgs a;
    uint64_t *key_out;  // nullable
};

// A record buffer's view as aggregate writes it: bucket (bin, part) holds up
// to part_cap records; cnt counts the places taken (possibly beyond part_cap:
// those groups went to their cells by device atomics, and spill[bin] is set).
struct Buckets {
    uint4 *rec;
    uint32_t *cnt, *spill;
    uint32_t bin_shift, nbins, parts, part_cap;
};

struct Plan {
    uint32_t nbins, bin_shift, groups, chunk, parts, part_cap;
    size_t lds_aggregate, lds_reduce;
    size_t off_cnt, off_rec, bytes;
    uint32_t nzero;  // words from off_cnt on that start at zero: ticket, spill flags, bucket counts
};

// Steps of kT vertices spread over as many workgroups as there are, in chunks
// of equal size; returns the steps.
static uint32_t deal_chunks(uint32_t n, uint32_t &chunk, uint32_t &groups) {
    const uint32_t nsteps = n ? (n + kT - 1) / kT : 1;
    const uint32_t rounds = (nsteps + kMaxGroups * kMaxSteps - 1) / (kMaxGroups * kMaxSteps);
    const uint32_t steps = (nsteps + kMaxGroups * rounds - 1) / (kMaxGroups * rounds);
    chunk = steps * kT;
    const uint32_t nchunks = (nsteps + steps - 1) / steps;
    groups = nchunks < kMaxGroups ? nchunks : kMaxGroups;
    return nsteps;
}

// LDS of aggregate for chunks of `chunk` vertices and nbins bins.
static constexpr size_t aggregate_lds(uint32_t chunk, uint32_t nbins) {
    return (size_t)kCap * 36 + (size_t)nbins * 8 + (4 + kMaxSteps) * 4 + (size_t)chunk * 2;
}

static size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// (Calls of up to kSmall vertices launch nothing of it; their workspace's size is
// still this plan's, so that a call is refused or accepted as before.)
Plan make_plan(uint32_t n, uint32_t log2_slots) {
    Plan p;
    // a bin per 1024 vertices up to 256 (a window of ~1500 groups then takes
    // a handful of neighbouring places in each), 512 for more than 2^22
    // vertices: reduce gains more than aggregate's places cost (8M incoherent
    // keys: 206 -> 161 us against 450 -> 460; 3840x2160x4: 190 -> 149 against
    // 657 -> 677; at 1920x1080x3 the two are even)
    uint32_t log2_bins = 0;
    while (log2_bins < 8 && (1024u << log2_bins) < n) ++log2_bins;
    if (n > 1u << 22) log2_bins = 9;
    if (log2_slots > kMaxLog2BinSlots && log2_bins < log2_slots - kMaxLog2BinSlots)
        log2_bins = log2_slots - kMaxLog2BinSlots;
    const uint32_t most = log2_slots > 5 ? log2_slots - 5 : 0;  // a bin owns whole bitmap words
    if (log2_bins > most) log2_bins = most;
    p.nbins = 1u << log2_bins;
    p.bin_shift = log2_slots - log2_bins;
    const uint32_t nsteps = deal_chunks(n, p.chunk, p.groups);
    // a bucket is split into one part per XCD (workgroups are dealt to the 8
    // XCDs in turn), so that a line of records is completed through one L2
    p.parts = nsteps >= 64 ? kMaxParts : 1;
    // room for four records a vertex in all (twice what a call can write
    // when every group needs two), and some for uneven parts of small calls
    const uint64_t nparts = (uint64_t)p.nbins * p.parts;
    p.part_cap = (uint32_t)((4ull * n + nparts - 1) / nparts) + 32;
    p.nzero = 1 + p.nbins + p.nbins * p.parts;
    p.lds_aggregate = aggregate_lds(p.chunk, p.nbins);
    const uint32_t words = p.bin_shift > 5 ? 1u << (p.bin_shift - 5) : 1u;
    p.lds_reduce = (size_t)kCells * 32 + (size_t)words * 8;
    p.off_cnt = 0;
    p.off_rec = align256((size_t)p.nzero * 4);
    p.bytes = p.off_rec + align256((size_t)nparts * p.part_cap * sizeof(uint4)) + 256;
    return p;
}

template <bool kOcc>
__device__ __forceinline__ uint32_t claim(const Tab &t, uint64_t key) {
    return claim_from<kOcc>(t, key, fingerprint_of(key), home_of(key, t.mask), 0);
}

// Whether a group needs records of kind 1, and how many.
__device__ __forceinline__ uint32_t extra_records(uint32_t count, uint64_t s0, uint64_t s1, uint64_t s2) {
    const bool fits = (int64_t)s0 == (int32_t)s0 && (int64_t)s1 == (int32_t)s1 && (int64_t)s2 == (int32_t)s2;
    const uint32_t high = (count - 1) >> 6;
    return (high + kCountMask - 1) / kCountMask + (!fits && high == 0 ? 1u : 0u);
}

// One group's records from place `pos` of its bucket part on; a group whose
// records do not all fit goes to its cell by device atomics instead.
__device__ __forceinline__ void put_records(const Buckets &bk, const Tab &t, uint32_t part, uint32_t pos,
                                            uint32_t extra, uint32_t s, uint32_t count, uint64_t s0, uint64_t s1,
                                            uint64_t s2) {
    const uint32_t bin = s >> bk.bin_shift;
    if (pos < bk.part_cap && pos + extra < bk.part_cap) {
        uint4 *w = bk.rec + ((size_t)bin * bk.parts + part) * bk.part_cap + pos;
        w[0] = make_uint4(s | ((count - 1) & kCountMask) << kSlotBits, (uint32_t)s0, (uint32_t)s1, (uint32_t)s2);
        uint32_t high = (count - 1) >> 6;
        // what the sign-extended low parts leave, in units of 2^32
        uint32_t h0 = (uint32_t)((s0 - (uint64_t)(int64_t)(int32_t)s0) >> 32);
        uint32_t h1 = (uint32_t)((s1 - (uint64_t)(int64_t)(int32_t)s1) >> 32);
        uint32_t h2 = (uint32_t)((s2 - (uint64_t)(int64_t)(int32_t)s2) >> 32);
        for (uint32_t e = 1; e <= extra; ++e) {
            const uint32_t c = min(high, kCountMask);
            w[e] = make_uint4(s | c << kSlotBits | 0x80000000u, h0, h1, h2);
            high -= c;
            h0 = h1 = h2 = 0;
        }
    } else {
        // places below part_cap that no group fills are read by reduce:
        // records that add nothing
        for (uint32_t e = pos; e <= pos + extra && e < bk.part_cap; ++e)
            bk.rec[((size_t)bin * bk.parts + part) * bk.part_cap + e] = make_uint4(s | 0x80000000u, 0, 0, 0);
        accumulate(t, s, count, (int64_t)s0, (int64_t)s1, (int64_t)s2);
        __hip_atomic_fetch_or(&t.occ[s >> 5], 1u << (s & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bk.spill[bin] = 1;
    }
}

// The count words of a call start at zero (a kernel of its own: a memset is
// not safe to capture in a graph).
__global__ __launch_bounds__(kT) void zero_kernel(uint32_t *p, uint32_t n) {
    for (uint32_t k = threadIdx.x; k < n; k += kT) p[k] = 0;
}

// A vertex's inputs: its contribution and its key, or (kKeys) the position
// and normal its key is built from (Algorithm 1, as pf_build_keys).
template <bool kKeys>
struct VertexIn {
    float c[3];
    float x[kKeys ? 3 : 1], nr[kKeys ? 3 : 1];
    uint64_t key;
};

template <bool kKeys>
__device__ __forceinline__ VertexIn<kKeys> load_vertex(const FusedKeys &fk, const uint64_t *key, const float *r,
                                                       const float *g, const float *b, uint32_t i) {
    VertexIn<kKeys> in{};
    in.c[0] = r[i];
    in.c[1] = g[i];
    in.c[2] = b[i];
    if constexpr (kKeys) {
        in.x[0] = fk.px[i];
        in.x[1] = fk.py[i];
        in.x[2] = fk.pz[i];
        in.nr[0] = fk.nx[i];
        in.nr[1] = fk.ny[i];
        in.nr[2] = fk.nz[i];
    } else {
        in.key = key[i];
    }
    return in;
}

// Where a window's groups go: kBuckets, records for reduce; kAtomics, straight
// to their cells by device atomics (no workspace), kFloatAtomics the same with
// binary32 sums.
enum Sink { kBuckets, kAtomics, kFloatAtomics };

// Key, contribution (fixed point; kFloatAtomics: as it is) and flags of a
// vertex; rnd: its PCG32 outputs.
template <bool kKeys, typename V>
__device__ __forceinline__ uint32_t vertex_value(const FusedKeys &fk, const VertexIn<kKeys> &in, const uint32_t rnd[3],
                                                 int frac_bits, uint64_t &k, V &q0, V &q1, V &q2) {
    uint32_t f = 0;
    k = in.key;
    if constexpr (kKeys) {
        uint32_t fp, home;
        f = vertex_key(in.x, in.nr, true, fk.a.cam, fk.a.s, fk.a.inv_s, rnd, fk.a.mask, k, fp, home);
    }
    if (f == 0) {
        if constexpr (std::is_same<V, float>::value)
            f = float_contribution(in.c[0], in.c[1], in.c[2], q0, q1, q2);
        else
            f = fixed_point(in.c[0], in.c[1], in.c[2], frac_bits, q0, q1, q2);
    }
    return f;
}

// What a thread keeps of a vertex until its window is flushed (16 bits): its
// LDS entry, kAlone (no room in LDS), or kFlagged and its flags.
constexpr uint32_t kAlone = 0xffffu, kFlagged = 0x8000u;

// kKeys: keys are built here from positions and normals (fk) and the flags
// are outputs only; otherwise key[] and flags[] come from pf_build_keys.
//
// Bound by memory requests: the claims fetch a 128-byte line for each group's
// 4-byte probe (without them 1920x1080x3 took 84 us of 118, 3840x2160x4 476 of
// 655), the record writes cost 24 and 105 us, the key arithmetic nothing.  A
// workgroup takes chunks of `chunk` consecutive vertices, lists a chunk's valid
// ones in LDS (bounce segments keep one vertex in four; 138 -> 124 us and 711
// -> 659 us at the two sizes above) and goes through the list in steps of one
// vertex per thread.  The steps are gathered into windows: a window ends when
// the next step's vertices might not find room in the LDS table any more (more
// than kLimit entries in use), so coherent streams merge over 4096 vertices,
// while streams of mostly distinct keys (small images, bounces, shuffled keys)
// flush as often as the table needs.
template <bool kKeys, Sink kSink>
__global__ __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(8, 8))) void aggregate_kernel(
    Tab t, const uint64_t *__restrict__ key, const float *__restrict__ r, const float *__restrict__ g,
    const float *__restrict__ b, uint8_t *__restrict__ flags, uint32_t *__restrict__ slot_out, uint32_t n,
    uint32_t chunk, Buckets bk, uint32_t *__restrict__ ticket, FusedKeys fk) {
    extern __shared__ __align__(16) unsigned char lds[];
    unsigned long long *lkey = reinterpret_cast<unsigned long long *>(lds);
    unsigned long long *ls0 = lkey + kCap, *ls1 = ls0 + kCap, *ls2 = ls1 + kCap;
    uint32_t *lcnt = reinterpret_cast<uint32_t *>(ls2 + kCap);  // count, then the group's slot
    uint32_t *taken = lcnt + kCap;      // [nbins] places the window takes in each bin
    uint32_t *place = taken + bk.nbins;  // [nbins] the first of them
    uint32_t *misc = place + bk.nbins;  // [0] overflowed vertices, [1] the next chunk, [2] valid vertices
    uint32_t *created = misc + 4;       // [kMaxSteps] LDS entries created by each step of the chunk
    uint16_t *list = reinterpret_cast<uint16_t *>(created + kMaxSteps);  // the chunk's valid vertices
    using V = std::conditional_t<kSink == kFloatAtomics, float, int64_t>;
    const uint32_t tid = threadIdx.x;
    const uint32_t part = kSink == kBuckets ? blockIdx.x % bk.parts : 0u;
    for (uint32_t k = tid; k < bk.nbins; k += kT) taken[k] = 0;
    if (tid < 4 + kMaxSteps) misc[tid] = 0;
    for (uint32_t j = tid; j < kCap; j += kT) {
        lkey[j] = kEmpty;
        ls0[j] = 0;
        ls1[j] = 0;
        ls2[j] = 0;
        lcnt[j] = 0;
    }
    __syncthreads();
    const PcgJump jp(fk.a.seed, fk.a.idx_base);
    const uint32_t nchunks = (n + chunk - 1) / chunk;
    // the valid bytes (or input flags) of a chunk's vertices, loaded ...
    auto load_live = [&](uint32_t ci, uint32_t raw[kMaxSteps]) {
        const uint32_t c0 = ci * chunk, i1 = ci < nchunks ? min(n, c0 + chunk) : 0u;
#pragma unroll
        for (uint32_t u = 0; u < kMaxSteps; ++u) {
            const uint32_t i = c0 + u * kT + tid;
            raw[u] = kKeys ? 0u : 1u;
            if (i < i1) raw[u] = kKeys ? (fk.valid ? fk.valid[i] : 1u) : flags[i];
        }
    };
    // ... and taken as one bit per step
    auto live_bits = [&](const uint32_t raw[kMaxSteps]) -> uint32_t {
        uint32_t m = 0;
#pragma unroll
        for (uint32_t u = 0; u < kMaxSteps; ++u) m |= ((raw[u] != 0) == kKeys ? 1u : 0u) << u;
        return m;
    };
    // chunks differ in cost (coherent, incoherent or empty parts of the
    // stream): after its first two a workgroup takes the next one there is.
    // It draws a chunk's number while it works on the chunk before the last
    // (drawn by every workgroup at the launch's start, the tickets' atomics on
    // one address held all of them up for 6 us), and reads its valid bytes
    // before the chunk before it ends.
    uint32_t ci = blockIdx.x, next = blockIdx.x + gridDim.x, drawn = 0;
    uint32_t raw[kMaxSteps];
    load_live(ci, raw);
    uint32_t live = live_bits(raw);
    while (ci < nchunks) {
        const uint32_t c0 = ci * chunk, i1 = min(n, c0 + chunk);
        // masked vertices (sky, escaped paths) read nothing more and get
        // their outputs here
#pragma unroll
        for (uint32_t u = 0; u < kMaxSteps; ++u) {
            const uint32_t i = c0 + u * kT + tid;
            const bool v = (live >> u) & 1u;
            const uint32_t at = wave_reserve(&misc[2], v);
            if (v) {
                list[at] = (uint16_t)(u * kT + tid);
            } else if (i < i1) {
                if (kKeys) flags[i] = PF_V_INVALID;
                if (kKeys && fk.key_out) fk.key_out[i] = 0;
                if (kSink == kBuckets || slot_out) slot_out[i] = kNoSlot;
            }
        }
        __syncthreads();
        const uint32_t nlive = misc[2], nsteps = (nlive + kT - 1) / kT;
        uint32_t w0 = 0;  // the window's first step
        do {
            uint64_t code = 0;  // 16 bits per step
            uint32_t u = w0;
            while (u < nsteps) {
                const uint32_t l = u * kT + tid;
                uint32_t c = kFlagged;
                bool fresh = false;
                if (l < nlive) {
                    const uint32_t i = c0 + list[l];
                    const VertexIn<kKeys> in = load_vertex<kKeys>(fk, key, r, g, b, i);
                    uint32_t rnd[3] = {0, 0, 0};
                    if constexpr (kKeys)
                        for (int d = 0; d < 3; ++d) rnd[d] = jp.output(d, i);
                    uint64_t k;
                    V q0, q1, q2;
                    c = vertex_value<kKeys>(fk, in, rnd, t.frac_bits, k, q0, q1, q2);
                    if (kKeys && fk.key_out) fk.key_out[i] = k;
                    if (c == 0) {
                        // (a caller's key may be the empty entry's)
                        const int e = !kKeys && k == kEmpty ? -1 : lds_insert(lkey, kCap, k, fresh);
                        if (e >= 0) {
                            atomicAdd(&lcnt[e], 1u);
                            lds_add(&ls0[e], q0);
                            lds_add(&ls1[e], q1);
                            lds_add(&ls2[e], q2);
                            c = (uint32_t)e;
                        } else {
                            c = kAlone;
                        }
                    } else {
                        c |= kFlagged;
                    }
                }
                const uint64_t m = __ballot(fresh);
                if ((tid & 63) == 0 && m) atomicAdd(&created[u], (uint32_t)__popcll(m));
                code |= (uint64_t)c << (16 * u);
                ++u;
                if (u == nsteps) break;
                // go on while the next step's vertices are sure to find room
                const uint32_t next = min(nlive - u * kT, (uint32_t)kT);
                if ((u - w0) * kT + next <= kLimit) continue;
                __syncthreads();
                uint32_t used = 0;
                for (uint32_t v = w0; v < u; ++v) used += created[v];
                if (used + next > kLimit) break;
            }
            __syncthreads();
            // one probe / claim per group; a thread's
            // entries issue their home-slot loads, then their compare-and-swaps
            // on empty home slots, before either result is needed
            uint64_t gk[kFlush];
            uint32_t fs[kFlush], ff[kFlush], fcur[kFlush];
#pragma unroll
            for (uint32_t v = 0; v < kFlush; ++v) {
                const uint32_t j = v * kT + tid;
                gk[v] = j < kCap ? lkey[j] : kEmpty;
                fs[v] = 0;
                ff[v] = 0;
                fcur[v] = 0;
                if (gk[v] != kEmpty) {
                    fs[v] = home_of(gk[v], t.mask);
                    ff[v] = fingerprint_of(gk[v]);
                    fcur[v] = load_fp_probe(&t.cell_at(fs[v]).fp);
                }
            }
            bool won[kFlush];
#pragma unroll
            for (uint32_t v = 0; v < kFlush; ++v) {
                won[v] = false;
                if (gk[v] != kEmpty && fcur[v] == 0) {
                    uint32_t expected = 0;
                    won[v] =
                        __hip_atomic_compare_exchange_strong(&t.cell_at(fs[v]).fp, &expected, ff[v], __ATOMIC_RELAXED,
                                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    fcur[v] = won[v] ? ff[v] : expected;
                }
            }
            // the group's rank among the window's records of its bin
            uint32_t slot[kFlush], cnt[kFlush] = {}, rank[kFlush];
#pragma unroll
            for (uint32_t v = 0; v < kFlush; ++v) {
                const uint32_t j = v * kT + tid;
                slot[v] = kNoSlot;
                if (gk[v] == kEmpty) continue;
                if (won[v]) claimed<kSink != kBuckets>(t, fs[v], gk[v]);
                // the home slot holds another key: probe on from the next
                slot[v] = fcur[v] == ff[v] ? fs[v]
                                           : claim_from<kSink != kBuckets>(t, gk[v], ff[v], (fs[v] + 1) & t.mask, 1);
                cnt[v] = lcnt[j];
                lcnt[j] = slot[v];
                if (slot[v] == kNoSlot) {
                    atomicAdd(&misc[0], cnt[v]);
                } else if constexpr (kSink == kBuckets) {
                    rank[v] = atomicAdd(&taken[slot[v] >> bk.bin_shift],
                                        1u + extra_records(cnt[v], ls0[j], ls1[j], ls2[j]));
                }
            }
            if constexpr (kSink != kBuckets) {
#pragma unroll
                for (uint32_t v = 0; v < kFlush; ++v) {
                    const uint32_t j = min(v * kT + tid, kCap - 1);
                    accumulate_wave(t, slot[v], cnt[v], lds_value(&ls0[j], V()), lds_value(&ls1[j], V()),
                                    lds_value(&ls2[j], V()));
                }
            }
            __syncthreads();
            // the window's places, one device atomic per bin; the vertices get
            // their slots while they are on their way
            uint32_t first_place = 0;
            const uint32_t want = tid < bk.nbins ? taken[tid] : 0u;
            if (want)
                first_place = __hip_atomic_fetch_add(&bk.cnt[tid * bk.parts + part], want, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll 1
            for (uint32_t v = w0; v < u; ++v) {
                const uint32_t l = v * kT + tid;
                if (l >= nlive) break;
                const uint32_t i = c0 + list[l];
                const uint32_t c = (uint32_t)(code >> (16 * v)) & 0xffffu;
                uint32_t s = kNoSlot, f = 0;
                if (c < kFlagged) {
                    s = lcnt[c];
                    f = s == kNoSlot ? (uint32_t)PF_V_OVERFLOW : 0u;
                } else if (c == kAlone) {  // no room in the LDS table: a group of its own
                    const VertexIn<kKeys> in = load_vertex<kKeys>(fk, key, r, g, b, i);
                    uint32_t rnd[3] = {0, 0, 0};
                    if constexpr (kKeys)
                        for (int d = 0; d < 3; ++d) rnd[d] = jp.output(d, i);
                    uint64_t k;
                    V q0, q1, q2;
                    vertex_value<kKeys>(fk, in, rnd, t.frac_bits, k, q0, q1, q2);
                    s = claim<kSink != kBuckets>(t, k);
                    if (s == kNoSlot) {
                        f = PF_V_OVERFLOW;
                        atomicAdd(&misc[0], 1u);
                    } else if constexpr (kSink == kBuckets) {
                        const uint32_t extra = extra_records(1, (uint64_t)q0, (uint64_t)q1, (uint64_t)q2);
                        const uint32_t pos =
                            __hip_atomic_fetch_add(&bk.cnt[(s >> bk.bin_shift) * bk.parts + part], 1u + extra,
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        put_records(bk, t, part, pos, extra, s, 1u, (uint64_t)q0, (uint64_t)q1, (uint64_t)q2);
                    } else {
                        accumulate(t, s, 1u, q0, q1, q2);
                    }
                } else {
                    f = c & 0xffu;
                }
                if (kKeys || f) flags[i] = (uint8_t)f;
                if (kSink == kBuckets || slot_out) slot_out[i] = s;
            }
            if (want) {
                place[tid] = first_place;
                taken[tid] = 0;
            }
            if (u == nsteps) {  // for the next chunk
                if (tid < kMaxSteps) created[tid] = 0;
                if (tid == 0) {
                    if (kSink != kBuckets)
                        misc[1] = ci + gridDim.x;  // no workspace, no ticket: chunks in turn
                    else if (ci >= gridDim.x)
                        misc[1] = 2 * gridDim.x + drawn;
                    misc[2] = 0;
                }
            }
            __syncthreads();
            if (u == nsteps) {
                const uint32_t after = ci < gridDim.x ? next : misc[1];
                load_live(after, raw);
                if (kSink == kBuckets && tid == 0) drawn = atomicAdd(ticket, 1u);
                ci = after;
            }
#pragma unroll
            for (uint32_t v = 0; v < kFlush; ++v) {
                const uint32_t j = v * kT + tid;
                if (gk[v] == kEmpty) continue;
                if (kSink == kBuckets && slot[v] != kNoSlot) {
                    const uint64_t s0 = ls0[j], s1 = ls1[j], s2 = ls2[j];
                    put_records(bk, t, part, place[slot[v] >> bk.bin_shift] + rank[v],
                                extra_records(cnt[v], s0, s1, s2), slot[v], cnt[v], s0, s1, s2);
                }
                lkey[j] = kEmpty;  // emptied for the next window
                ls0[j] = 0;
                ls1[j] = 0;
                ls2[j] = 0;
                lcnt[j] = 0;
            }
            w0 = u;
            if (u == nsteps) live = live_bits(raw);
            __syncthreads();
        } while (w0 < nsteps);
    }
    if (tid == 0 && misc[0]) add_u64(&t.stats[PF_STAT_PART_OVF + (blockIdx.x & 15)], misc[0]);
}

// The insert of a small call: a vertex per thread; a workgroup's vertices merge
// by key in an LDS table (keys included, kKeys), the thread that made a key's
// entry claims its cell and adds the sums by device atomics.  Bound by its one
// chain of latencies where cells are many, and by the visits of the workgroups
// to the same few cells where voxels are coarse: a compare-and-swap and a line
// of atomics each, and every workgroup meets the empty cell.  (With a claim per
// vertex 300k vertices of one cell took 1100 us, this 16; whole frames of
// 401x229x3 at cell size 0.01 / 1 / 10: 42.8 / 281 / 356 -> 42.7 / 38.7 / 39.9 us.)
// So the threads a workgroup double at kSmallGroups workgroups, from 128 on (512
// threads at 401x229x3: 41.6 / 57 / 77 us; 64x64 by 128 / 256 / 512 / 1024 threads
// 20.2 / 20.5 / 22.3 / 27.6, as by a claim per vertex), and beyond
// kSmallGroups of 1024 the slots after the home slot are read one at a time:
// kAhead 4 saves a small call latency (200x150x3 43.4 -> 37.9 us) but reads the
// lines that others are claiming (401x229x3 at cell size 10: 40 -> 56).
// Whole frames by buckets -> this: 290x170x3 48 -> 38 us, 401x229x3 46 -> 43,
// 430x250x3 49 -> 46, 570x570x1 39 -> 34, 400x400x2 44.5 -> 45, so kSmall is
// 5 * 2^16.
template <bool kKeys, uint32_t kSmallT, uint32_t kAhead>
__global__ __launch_bounds__(kSmallT) void small_insert_kernel(Tab t, const uint64_t *__restrict__ key,
                                                               const float *__restrict__ r,
                                                               const float *__restrict__ g,
                                                               const float *__restrict__ b,
                                                               uint8_t *__restrict__ flags,
                                                               uint32_t *__restrict__ slot_out, uint32_t n,
                                                               FusedKeys fk) {
    // LDS entries: never full; two workgroups of 1024 fit a CU
    constexpr uint32_t kSmallCap = kSmallT < 1024 ? 2 * kSmallT : kSmallT / 2 * 3;
    __shared__ unsigned long long lkey[kSmallCap], lsum[3][kSmallCap];
    __shared__ uint32_t lcnt[kSmallCap], lslot[kSmallCap];
    for (uint32_t j = threadIdx.x; j < kSmallCap; j += kSmallT) {
        lkey[j] = kEmpty;
        lsum[0][j] = 0;
        lsum[1][j] = 0;
        lsum[2][j] = 0;
        lcnt[j] = 0;
    }
    const uint32_t i = blockIdx.x * kSmallT + threadIdx.x;
    const bool in = i < n;
    uint32_t f = PF_V_INVALID;
    if constexpr (kKeys) {
        if (in && (fk.valid == nullptr || fk.valid[i] != 0)) f = 0;
    } else {
        if (in) f = flags[i];
    }
    const uint32_t f0 = f;
    uint64_t k = 0;
    int64_t q0 = 0, q1 = 0, q2 = 0;
    if (f == 0) {
        const VertexIn<kKeys> vin = load_vertex<kKeys>(fk, key, r, g, b, i);
        uint32_t rnd[3] = {0, 0, 0};
        if constexpr (kKeys) {
            const PcgJump jp(fk.a.seed, fk.a.idx_base);
            for (int d = 0; d < 3; ++d) rnd[d] = jp.output(d, i);
        }
        f = vertex_value<kKeys>(fk, vin, rnd, t.frac_bits, k, q0, q1, q2);
    }
    __syncthreads();
    int e = -1;
    bool claims = false;  // this thread claims a cell: for its entry, or alone
    uint32_t slot = kNoSlot;
    if (f == 0) {
        // (a caller's key may be the empty entry's)
        if (kKeys || k != kEmpty) e = lds_insert(lkey, kSmallCap, k, claims);
        if (e >= 0) {
            atomicAdd(&lcnt[e], 1u);
            lds_add(&lsum[0][e], q0);
            lds_add(&lsum[1][e], q1);
            lds_add(&lsum[2][e], q2);
        } else {
            claims = true;
        }
        if (claims) slot = find_or_claim<kAhead>(t, k);
        if (claims && e >= 0) lslot[e] = slot;
    }
    __syncthreads();
    uint32_t cnt = 1;
    if (e >= 0) {
        cnt = lcnt[e];
        q0 = (int64_t)lsum[0][e];
        q1 = (int64_t)lsum[1][e];
        q2 = (int64_t)lsum[2][e];
        if (!claims) slot = lslot[e];
    }
    if (f == 0 && slot == kNoSlot) {
        f = PF_V_OVERFLOW;
        if (claims) add_u64(&t.stats[PF_STAT_PART_OVF + (blockIdx.x & 15)], (unsigned long long)cnt);
    }
    if (in) {
        if (kKeys && fk.key_out) fk.key_out[i] = k;
        if (kKeys || f != f0) flags[i] = (uint8_t)f;
        slot_out[i] = slot;
    }
    accumulate_wave(t, claims ? slot : kNoSlot, cnt, q0, q1, q2);
}

// The temporal blend done by reduce: the previous table (has_prev) and the
// blend's parameters as pf_temporal_update / pf_temporal_integrate take them.
struct Blend {
    Tab prev;
    float alpha, beta;
    uint32_t cap;
};

// One workgroup per bin: the slots its records name, as a bitmap; a cell's
// index is the number of set bits before its own, so the LDS holds sums for the
// cells there are and not for the bin's slots (a frame fills a few percent of
// its table).  More than kCells cells take several passes over the records.
// The exclusive owner then adds the sums to the cells and sets the occupancy
// bits of its words.
// Bound by its chain of latencies (counts, records, cells, the previous table's
// slots) where bins are small and by LDS atomics and record reads where they are
// large, so two workgroups of 512 threads share a CU, a thread's first cells are
// requested before the records are summed, and records are read a batch ahead
// (256 bins and one workgroup of 1024 threads a CU: 3840x2160x4 190 -> 134 us, 8M
// incoherent keys 206 -> 145 us, 1920x1080x3 40 -> 38 us).
// A bin of more than kMaxPasses passes' cells (bins of 2^14 slots and more, well
// filled: tables from 2^22 slots on, 2^23 above 2^22 vertices) sends its records to
// the cells by device atomics instead, once.  33M keys drawn from load x 2^25 cells
// (at load 0.5 86% of them occur; with every cell present 0.5 / 0.7 take 3994 / 5050
// us), 2^25 slots, all launches, passes / atomics at loads 0.15 (4.8 passes) 2526 /
// 2905 us, 0.2 (6.4) 3025 / 3053, 0.3 3813 / 3316, 0.5 4947 / 3773, 0.7 5922 / 4111.
// kBlend: it also computes the temporal values of the cells (which are final:
// every record of a slot is in the slot's bin), as pf_temporal_update does.
constexpr uint32_t kMaxPasses = 6;
template <bool kBlend = false, bool kHasPrev = false, bool kIntegrate = false>
__global__ __launch_bounds__(kR) __attribute__((amdgpu_waves_per_eu(4, 4))) void reduce_kernel(Tab t, Buckets bk, Blend bl) {
    extern __shared__ unsigned long long lred[];
    unsigned long long *sum0 = lred, *sum1 = lred + kCells, *sum2 = lred + 2 * kCells;
    uint32_t *cnt = reinterpret_cast<uint32_t *>(lred + 3 * kCells);
    uint32_t *list = cnt + kCells;  // the cells' slots within the bin
    const uint32_t words = bk.bin_shift > 5 ? 1u << (bk.bin_shift - 5) : 1u;
    uint32_t *bits = list + kCells, *before = bits + words;  // bitmap, set bits before each word
    __shared__ uint32_t seg[kMaxParts + 1], wave_sum[kR / 64], s_hits;
    const uint32_t tid = threadIdx.x, bin = blockIdx.x, base = bin << bk.bin_shift;
    const uint32_t in_bin = (1u << bk.bin_shift) - 1;
    if (tid <= kMaxParts) seg[tid] = tid < bk.parts ? min(bk.cnt[bin * bk.parts + tid], bk.part_cap) : 0u;
    if (tid == 0) s_hits = 0;
    // cells that got sums by device atomics (a full bucket) are in the
    // occupancy bitmap already; they are blended too
    const bool spilled = kBlend && bk.spill[bin] != 0;
    for (uint32_t w = tid; w < words; w += kR) bits[w] = spilled ? t.occ[(base >> 5) + w] : 0u;
    for (uint32_t k = tid; k < kCells; k += kR) {
        sum0[k] = 0;
        sum1[k] = 0;
        sum2[k] = 0;
        cnt[k] = 0;
    }
    __syncthreads();
    uint32_t end[kMaxParts], m = 0;  // where each part's records end in the bin's sequence
#pragma unroll
    for (uint32_t x = 0; x < kMaxParts; ++x) {
        m += seg[x];
        end[x] = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
    }
    auto record = [&](uint32_t j) -> const uint4 * {
        uint32_t x = 0, from = 0;
#pragma unroll
        for (uint32_t y = 0; y + 1 < kMaxParts; ++y)
            if (j >= end[y]) {
                x = y + 1;
                from = end[y];
            }
        return bk.rec + ((size_t)bin * bk.parts + x) * bk.part_cap + (j - from);
    };
    auto load_records = [&](uint32_t j0, uint4 (&q)[kHold]) {
#pragma unroll
        for (uint32_t u = 0; u < kHold; ++u)
            if (j0 + u * kR + tid < m) q[u] = *record(j0 + u * kR + tid);
    };
    auto mark = [&](uint32_t word) {
        const uint32_t loc = word & in_bin;
        atomicOr(&bits[loc >> 5], 1u << (loc & 31));
    };
    uint4 held[kHold];
    load_records(0, held);
#pragma unroll
    for (uint32_t u = 0; u < kHold; ++u)
        if (u * kR + tid < m) mark(held[u].x);
    for (uint32_t j0 = kHold * kR; j0 < m; j0 += kMark * kR) {
        uint32_t word[kMark];
#pragma unroll
        for (uint32_t u = 0; u < kMark; ++u)
            if (j0 + u * kR + tid < m) word[u] = record(j0 + u * kR + tid)->x;
#pragma unroll
        for (uint32_t u = 0; u < kMark; ++u)
            if (j0 + u * kR + tid < m) mark(word[u]);
    }
    __syncthreads();
    // set bits before each word: a thread takes `per` consecutive words
    const uint32_t per = (words + kR - 1) / kR, b0 = tid * per;
    uint32_t own = 0;
    for (uint32_t w = b0; w < min(words, b0 + per); ++w) own += (uint32_t)__popc(bits[w]);
    uint32_t incl = own;
#pragma unroll
    for (uint32_t off = 1; off < 64; off <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)incl, off);
        if ((tid & 63) >= off) incl += v;
    }
    if ((tid & 63) == 63) wave_sum[tid >> 6] = incl;
    __syncthreads();
    uint32_t run = incl - own, ncells = 0;
#pragma unroll
    for (uint32_t w = 0; w < kR / 64; ++w) {
        if (w < (tid >> 6)) run += wave_sum[w];
        ncells += wave_sum[w];
    }
    const uint32_t run0 = run;
    for (uint32_t w = b0; w < min(words, b0 + per); ++w) {
        before[w] = run;
        const uint32_t v = bits[w];
        run += (uint32_t)__popc(v);
        // occupancy: the words of this bin belong to this workgroup
        if (v) t.occ[(base >> 5) + w] |= v;
    }
    const bool direct = ncells > kMaxPasses * kCells;
    if (direct) {
        for (uint32_t j0 = 0; j0 < m; j0 += kR) {  // uniform: accumulate_wave is the wavefront's
            uint32_t slot = kNoSlot, c = 0;
            int64_t v[3] = {0, 0, 0};
            if (j0 + tid < m) {
                const uint4 q = *record(j0 + tid);
                const bool high = q.x >> 31;
                slot = base + (q.x & in_bin);
                c = (q.x >> kSlotBits) & kCountMask;
                c = high ? 64u * c : 1u + c;
                const uint32_t w[3] = {q.y, q.z, q.w};
                for (int k = 0; k < 3; ++k) v[k] = high ? (int64_t)((uint64_t)w[k] << 32) : (int64_t)(int32_t)w[k];
            }
            accumulate_wave(t, slot, c, v[0], v[1], v[2]);
        }
        if (!kBlend) return;
        __threadfence();  // the cells are read below by other threads of the workgroup
        __syncthreads();
        __threadfence();
    }
    uint32_t hits = 0;
    for (uint32_t c0 = 0; c0 < ncells; c0 += kCells) {
        const uint32_t nc = min(ncells - c0, kCells);
        if (c0) {
            __syncthreads();  // the last pass's cells are written
            for (uint32_t k = tid; k < nc; k += kR) {
                sum0[k] = 0;
                sum1[k] = 0;
                sum2[k] = 0;
                cnt[k] = 0;
            }
        }
        uint32_t at = run0;
        for (uint32_t w = b0; w < min(words, b0 + per); ++w)
            for (uint32_t v = bits[w]; v; v &= v - 1, ++at)
                if (at - c0 < nc) list[at - c0] = w * 32 + (uint32_t)__builtin_ctz(v);
        __syncthreads();
        // a thread's first cells are requested before the records are summed
        struct CellIn {
            uint4 lo, hi;
            uint64_t key;
        };
        auto load_cells = [&](uint32_t k0, CellIn (&in)[kPair]) {
#pragma unroll
            for (int v = 0; v < kPair; ++v) {
                const uint32_t k = k0 + v * kR + tid;
                if (k >= nc) continue;
                const uint4 *w4 = t.words_at(base + list[k]);  // 4 sixteen-byte words per slot record
                in[v].lo = w4[0];
                in[v].hi = w4[1];
                if constexpr (kBlend && kHasPrev) in[v].key = (uint64_t)w4[2].x | (uint64_t)w4[2].y << 32;
            }
        };
        CellIn in[kPair];
        load_cells(0, in);
        auto add = [&](const uint4 &q) {
            const uint32_t loc = q.x & in_bin;
            const uint32_t k = before[loc >> 5] + (uint32_t)__popc(bits[loc >> 5] & ((1u << (loc & 31)) - 1u)) - c0;
            if (k >= nc) return;  // another pass's cell
            const uint32_t c = (q.x >> kSlotBits) & kCountMask;
            unsigned long long v0, v1, v2;
            if (__builtin_expect(q.x >> 31, 0)) {
                v0 = (unsigned long long)q.y << 32;
                v1 = (unsigned long long)q.z << 32;
                v2 = (unsigned long long)q.w << 32;
                atomicAdd(&cnt[k], 64u * c);
            } else {
                v0 = (unsigned long long)(int64_t)(int32_t)q.y;
                v1 = (unsigned long long)(int64_t)(int32_t)q.z;
                v2 = (unsigned long long)(int64_t)(int32_t)q.w;
                atomicAdd(&cnt[k], 1u + c);
            }
            atomicAdd(&sum0[k], v0);
            atomicAdd(&sum1[k], v1);
            atomicAdd(&sum2[k], v2);
        };
        // the records after those held are one batch ahead of the sums
        uint4 q[kHold];
#pragma unroll
        for (uint32_t u = 0; u < kHold; ++u) q[u] = held[u];
        for (uint32_t j0 = 0; j0 < (direct ? 0u : m); j0 += kHold * kR) {
            uint4 ahead[kHold];
            load_records(j0 + kHold * kR, ahead);
#pragma unroll
            for (uint32_t u = 0; u < kHold; ++u)
                if (j0 + u * kR + tid < m) add(q[u]);
#pragma unroll
            for (uint32_t u = 0; u < kHold; ++u) q[u] = ahead[u];
        }
        __syncthreads();
        for (uint32_t k0 = 0; k0 < nc; k0 += kPair * kR) {
            if (k0) load_cells(k0, in);
            uint32_t sl[kPair], fp[kPair], n[kPair], keep[kPair];
            uint64_t key[kPair];
            bool has[kPair];
            float v[kPair][3];
#pragma unroll
            for (int w = 0; w < kPair; ++w) {
                const uint32_t k = k0 + w * kR + tid;
                has[w] = k < nc;
                if (!has[w]) continue;
                sl[w] = base + list[k];
                pf_cell cl;
                cl.fp = in[w].lo.x;
                cl.count = in[w].lo.y + cnt[k];
                const uint64_t s0 = ((uint64_t)in[w].lo.z | (uint64_t)in[w].lo.w << 32) + sum0[k];
                const uint64_t s1 = ((uint64_t)in[w].hi.x | (uint64_t)in[w].hi.y << 32) + sum1[k];
                const uint64_t s2 = ((uint64_t)in[w].hi.z | (uint64_t)in[w].hi.w << 32) + sum2[k];
                uint4 *w4 = t.words_at(sl[w]);
                w4[0] = make_uint4(cl.fp, cl.count, (uint32_t)s0, (uint32_t)(s0 >> 32));
                w4[1] = make_uint4((uint32_t)s1, (uint32_t)(s1 >> 32), (uint32_t)s2, (uint32_t)(s2 >> 32));
                if constexpr (kBlend) {
                    cl.sum[0] = (int64_t)s0;
                    cl.sum[1] = (int64_t)s1;
                    cl.sum[2] = (int64_t)s2;
                    if constexpr (kHasPrev) key[w] = in[w].key;
                    fp[w] = cl.fp;
                    n[w] = cl.count;
                    keep[w] = kIntegrate ? min(cl.count, bl.cap) : cl.count;
#pragma unroll
                    for (int c = 0; c < 3; ++c) v[w][c] = t.average(cl, c);
                }
            }
            if constexpr (kBlend)
                hits += blend_cells<kHasPrev, kIntegrate, kPair, false>(t, bl.prev, sl, has, key, fp, v, n, keep,
                                                                        bl.alpha, bl.beta, bl.cap);
        }
    }
    if constexpr (kBlend && kHasPrev) {
        // one device atomic per workgroup, spread over 32 partial counters
        if (hits) atomicAdd(&s_hits, hits);
        __syncthreads();
        if (tid == 0 && s_hits) add_u64(&t.stats[PF_STAT_PART_HIT + (blockIdx.x & 31)], s_hits);
    }
}

}  // namespace binned

size_t binned_workspace_bytes(uint32_t n, uint32_t log2_slots) {
    if (log2_slots > binned::kMaxLog2Slots) return 0;
    return binned::make_plan(n, log2_slots).bytes;
}

namespace binned {

// blend: NULL for the insert alone; else the temporal blend in reduce
// (has_prev: blend->prev is a table; integrate: temporal integration).
template <bool kKeys>
static hipError_t run(const Tab &t, const uint64_t *key, const float *r, const float *g, const float *b,
                      uint8_t *flags, uint32_t *slot_out, uint32_t n, void *ws, const FusedKeys &fk,
                      const Blend *blend, bool has_prev, bool integrate, hipStream_t st) {
    if (n <= kSmall) {
        const auto launch = [&](auto kernel, uint32_t threads) {
            kernel<<<(n + threads - 1) / threads, threads, 0, st>>>(t, key, r, g, b, flags, slot_out, n, fk);
        };
        if (n <= kSmallGroups * 128)
            launch(small_insert_kernel<kKeys, 128, 4>, 128);
        else if (n <= kSmallGroups * 256)
            launch(small_insert_kernel<kKeys, 256, 4>, 256);
        else if (n <= kSmallGroups * 512)
            launch(small_insert_kernel<kKeys, 512, 4>, 512);
        else if (n <= kSmallGroups * 1024)
            launch(small_insert_kernel<kKeys, 1024, 4>, 1024);
        else
            launch(small_insert_kernel<kKeys, 1024, 1>, 1024);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || !blend) return e;
        return launch_temporal(t, has_prev ? &blend->prev : nullptr, blend->alpha, integrate ? 1 : 0, blend->cap, st);
    }
    const uint32_t log2_slots = 32 - __builtin_clz(t.mask + 1) - 1;
    const Plan p = make_plan(n, log2_slots);
    char *base = reinterpret_cast<char *>((reinterpret_cast<uintptr_t>(ws) + 255) / 256 * 256);
    uint32_t *ticket = reinterpret_cast<uint32_t *>(base + p.off_cnt);
    Buckets bk;
    bk.spill = ticket + 1;
    bk.cnt = bk.spill + p.nbins;
    bk.rec = reinterpret_cast<uint4 *>(base + p.off_rec);
    bk.bin_shift = p.bin_shift;
    bk.nbins = p.nbins;
    bk.parts = p.parts;
    bk.part_cap = p.part_cap;
    constexpr size_t kAggregateLds = aggregate_lds(kMaxSteps * kT, kMaxBins);
    constexpr size_t kReduceLds = kCells * 32 + (8 << (kMaxLog2BinSlots - 5));
    static_assert(kAggregateLds <= 80 * 1024, "two workgroups of aggregate share a CU");
    static LargeLds aggregate, reduce;
    hipError_t e = aggregate.allow(kAggregateLds, aggregate_kernel<kKeys, kBuckets>);
    if (e == hipSuccess)
        e = reduce.allow(kReduceLds, reduce_kernel<false, false, false>, reduce_kernel<true, false, false>,
                         reduce_kernel<true, true, false>, reduce_kernel<true, false, true>,
                         reduce_kernel<true, true, true>);
    if (e != hipSuccess) return e;
    zero_kernel<<<1, kT, 0, st>>>(ticket, p.nzero);
    aggregate_kernel<kKeys, kBuckets><<<p.groups, kT, p.lds_aggregate, st>>>(t, key, r, g, b, flags, slot_out, n,
                                                                             p.chunk, bk, ticket, fk);
    const Blend none{};
    const Blend &bl = blend ? *blend : none;
    if (!blend)
        reduce_kernel<<<p.nbins, kR, p.lds_reduce, st>>>(t, bk, bl);
    else if (!has_prev && !integrate)
        reduce_kernel<true, false, false><<<p.nbins, kR, p.lds_reduce, st>>>(t, bk, bl);
    else if (has_prev && !integrate)
        reduce_kernel<true, true, false><<<p.nbins, kR, p.lds_reduce, st>>>(t, bk, bl);
    else if (!has_prev)
        reduce_kernel<true, false, true><<<p.nbins, kR, p.lds_reduce, st>>>(t, bk, bl);
    else
        reduce_kernel<true, true, true><<<p.nbins, kR, p.lds_reduce, st>>>(t, bk, bl);
    return hipGetLastError();
}

}  // namespace binned

bool insert_by_windows(uint32_t n) { return n >= binned::kMinWindowed; }

hipError_t launch_insert_windows(const Tab &t, const uint64_t *key, const float *r, const float *g, const float *b,
                                 uint8_t *flags, uint32_t *slot_out, uint32_t n, hipStream_t st) {
    using namespace binned;
    static LargeLds large;
    const hipError_t e = large.allow(aggregate_lds(kMaxSteps * kT, 0), aggregate_kernel<false, kAtomics>,
                                     aggregate_kernel<false, kFloatAtomics>);
    if (e != hipSuccess) return e;
    uint32_t chunk, groups;
    deal_chunks(n, chunk, groups);
    const size_t lds = aggregate_lds(chunk, 0);
    const FusedKeys none{};
    const Buckets no_buckets{};
    if (t.fsum)
        aggregate_kernel<false, kFloatAtomics><<<groups, kT, lds, st>>>(t, key, r, g, b, flags, slot_out, n, chunk,
                                                                       no_buckets, nullptr, none);
    else
        aggregate_kernel<false, kAtomics><<<groups, kT, lds, st>>>(t, key, r, g, b, flags, slot_out, n, chunk,
                                                                  no_buckets, nullptr, none);
    return hipGetLastError();
}

hipError_t launch_insert_binned(const Tab &t, const uint64_t *key, const float *r, const float *g, const float *b,
                                uint8_t *flags, uint32_t *slot_out, uint32_t n, void *ws, hipStream_t st) {
    binned::FusedKeys none{};
    return binned::run<false>(t, key, r, g, b, flags, slot_out, n, ws, none, nullptr, false, false, st);
}

hipError_t launch_keys_insert_binned(const Tab &t, const float *px, const float *py, const float *pz,
                                     const float *nx, const float *ny, const float *nz, const uint8_t *valid,
                                     const KeyArgs &a, uint64_t *key_out, const float *r, const float *g,
                                     const float *b, uint8_t *flags, uint32_t *slot_out, uint32_t n, void *ws,
                                     hipStream_t st) {
    const binned::FusedKeys fk{px, py, pz, nx, ny, nz, valid, a, key_out};
    return binned::run<true>(t, nullptr, r, g, b, flags, slot_out, n, ws, fk, nullptr, false, false, st);
}

hipError_t launch_keys_insert_binned_temporal(const Tab &t, const float *px, const float *py, const float *pz,
                                              const float *nx, const float *ny, const float *nz,
                                              const uint8_t *valid, const KeyArgs &a, uint64_t *key_out,
                                              const float *r, const float *g, const float *b, uint8_t *flags,
                                              uint32_t *slot_out, uint32_t n, void *ws, const Tab *prev,
                                              float alpha_old, int mode, uint32_t cap, hipStream_t st) {
    const binned::FusedKeys fk{px, py, pz, nx, ny, nz, valid, a, key_out};
    binned::Blend bl{};
    if (prev) bl.prev = *prev;
    bl.alpha = alpha_old;
    bl.beta = 1.0f - alpha_old;
    bl.cap = cap;
    return binned::run<true>(t, nullptr, r, g, b, flags, slot_out, n, ws, fk, &bl, prev != nullptr, mode == 1, st);
}

// ---- the insert without a workspace argument, for callers that cannot
// allocate.  Its workspace is a file-scope device array; on the host the
// array's name is not a device address, so every use goes through the
// address hipGetSymbolAddress returns for the current device (kept per
// device).  All calls on one device share the array: calls that overlap in
// time on one device (different streams, or host threads) race.

namespace binned {

constexpr uint32_t kNoAllocBatch = PF_NOALLOC_BATCH;  // vertices per pass over the scratch
constexpr size_t kScratchBytes = PF_NOALLOC_SCRATCH_BYTES;
constexpr int kMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

static std::mutex scratch_mutex;
static void *scratch_ptr[kMaxDevices];

// The current device's address of `scratch`, looked up once per device.
static hipError_t scratch_address(void **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        scratch_ptr[dev] = p;
    }
    *out = scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace binned

bool noalloc_fits(uint32_t log2_slots) {
    return log2_slots <= binned::kMaxLog2Slots &&
           binned::make_plan(binned::kNoAllocBatch, log2_slots).bytes + 256 <= binned::kScratchBytes;
}

hipError_t launch_keys_insert_binned_noalloc(const Tab &t, const float *px, const float *py, const float *pz,
                                             const float *nx, const float *ny, const float *nz,
                                             const uint8_t *valid, const KeyArgs &a, uint64_t *key_out,
                                             const float *r, const float *g, const float *b, uint8_t *flags,
                                             uint32_t *slot_out, uint32_t n, hipStream_t st) {
    void *ws = nullptr;
    hipError_t e = binned::scratch_address(&ws);
    if (e != hipSuccess) return e;
    // the insert accumulates, so consecutive batches give the table one
    // call would; each batch's workspace is written before it is read
    for (uint32_t i0 = 0; i0 < n; i0 += binned::kNoAllocBatch) {
        const uint32_t m = n - i0 < binned::kNoAllocBatch ? n - i0 : binned::kNoAllocBatch;
        KeyArgs ab = a;
        ab.idx_base = a.idx_base + i0;
        const binned::FusedKeys fk{px + i0, py + i0, pz + i0, nx + i0, ny + i0, nz + i0,
                                   valid ? valid + i0 : nullptr, ab, key_out ? key_out + i0 : nullptr};
        e = binned::run<true>(t, nullptr, r + i0, g + i0, b + i0, flags + i0, slot_out + i0, m, ws, fk, nullptr,
                              false, false, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace pfk
