// Fallbacks for voxels with few vertices (Section 3.3) for gfx950.
//
// The work is per sparse voxel, not per vertex.  A workgroup takes a range
// of occupancy words and lists in LDS the occupied slots of the range whose
// count is below the threshold; the listed voxels are then searched, each
// writing its pooled average into its temporal value, which the lookup with
// use_blend returns.
//   kMode 0, neighbourhood search, over the 27 voxels (dx, dy, dz) =
//     (c % 3 - 1, c / 3 % 3 - 1, c / 9 - 1) away at the same level and normal
//     class.  A workgroup takes up to 256 of its listed voxels at a time
//     through steps whose loads do not depend on each other: own cells and
//     keys; the home slots' occupancy bits of all 26 neighbours of all voxels;
//     the slots whose bit is set, listed in LDS, so that every lane probes one;
//     the quotients, one component a lane.  Bound by the latency of these
//     steps: with 8 lanes a voxel going through key, bits, fingerprint, key and
//     cell one voxel after the other, the waves waited 80% of their time
//     (1280x720x3, 134k sparse voxels with 4.7 present neighbours: 64 us, now
//     44 us);
//   kMode 1, similar normals along the probe run: one lane per voxel.  The
//     key's home slot does not depend on its normal class, so the voxels at
//     its position and level with other normals lie in its probe run, from
//     the home slot to the first empty one (at most max_probe slots), which
//     the occupancy bitmap shows; the lane reads the keys of that run and
//     counts the voxels with the same position bits whose normal class
//     vector has a positive dot product with its own.
// A key whose home slot is empty is not in the table (linear probing with
// no deletions), and the occupancy bitmap (1 bit per slot, L2-resident) says
// so without a random read of the slot: most candidate neighbours are
// absent.  Sums and counts are pooled as integers (exact, order-free) and
// divided once as the lookup divides: (float)((double)S * 2^-F / (double)N).
#include "pf_kernels.h"
#include "pf_merge.h"
#include "pf_ops.h"

namespace pfk {

constexpr int kLdThreads = 256;
constexpr uint32_t kLdWords = kLdThreads / 4;  // four lanes per occupancy word, 8 slots each
constexpr uint32_t kLdSlots = kLdWords * 32;
constexpr uint32_t kBatch = kLdThreads;  // voxels whose neighbours are searched together
constexpr uint32_t kWork = 2048;         // slots to probe listed at a time
constexpr uint64_t kCoordMask = (1ull << 51) - 1;

__device__ __forceinline__ int class_sign(uint64_t key, int axis) {
    const uint32_t v = (uint32_t)(key >> (56 + 2 * axis)) & 3u;
    return v == 1 ? 1 : (v == 2 ? -1 : 0);
}

__device__ __forceinline__ bool occupied(const Tab &t, uint32_t s) { return (t.occ[s >> 5] >> (s & 31)) & 1u; }

__device__ __forceinline__ void add_cell(const Tab &t, uint32_t s, uint32_t &n, uint64_t &a0, uint64_t &a1,
                                         uint64_t &a2) {
    const uint4 *c = t.words_at(s);
    const uint4 lo = c[0], hi = c[1];
    n += lo.y;
    a0 += (uint64_t)lo.z | (uint64_t)lo.w << 32;
    a1 += (uint64_t)hi.x | (uint64_t)hi.y << 32;
    a2 += (uint64_t)hi.z | (uint64_t)hi.w << 32;
}

__device__ __forceinline__ void store_pooled(const Tab &t, uint32_t s, uint32_t n, uint64_t a0, uint64_t a1,
                                             uint64_t a2) {
    float *v = reinterpret_cast<float *>(&t.blend_at(s));
    v[0] = cell_average((int64_t)a0, n, t.frac_bits);
    v[1] = cell_average((int64_t)a1, n, t.frac_bits);
    v[2] = cell_average((int64_t)a2, n, t.frac_bits);
}

// Candidate c's key for the voxel with key K; false outside the key range.
__device__ __forceinline__ bool neighbour_key(uint64_t K, uint32_t c, uint64_t &key) {
    const int d[3] = {(int)(c % 3) - 1, (int)(c / 3 % 3) - 1, (int)(c / 9) - 1};
    key = K & ~kCoordMask;
    bool in = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int x = (int)((K >> (17 * a)) & 0x1ffffu) - 65536 + d[a];
        in = in && x > -65536 && x < 65536;
        key |= (uint64_t)(uint32_t)(x + 65536) << (17 * a);
    }
    return in;
}

// Sums of a batch of voxels, in LDS.
struct Pool {
    unsigned long long key[kBatch], sum[3][kBatch];
    uint32_t count[kBatch];
    uint32_t nwork, slot[kWork];
    uint16_t pair[kWork];  // voxel, candidate
};

// Probes for `key` from its (occupied) home slot p on and adds its cell to
// voxel v's sums.  A slot's cell and key are one line, requested together; the
// key decides (equal keys have equal fingerprints), an empty cell ends the run.
__device__ __forceinline__ void pool_key(const Tab &t, Pool &P, uint32_t v, uint64_t key, uint32_t p) {
    for (uint32_t d = 0; d < t.max_probe; ++d) {
        const uint4 *w = t.words_at(p);
        const uint4 lo = w[0], hi = w[1];
        const uint64_t kk = t.key_at(p);
        if (lo.x == 0) return;
        if (kk == key) {
            atomicAdd(&P.count[v], lo.y);
            atomicAdd(&P.sum[0][v], (unsigned long long)lo.z | (unsigned long long)lo.w << 32);
            atomicAdd(&P.sum[1][v], (unsigned long long)hi.x | (unsigned long long)hi.y << 32);
            atomicAdd(&P.sum[2][v], (unsigned long long)hi.z | (unsigned long long)hi.w << 32);
            return;
        }
        p = (p + 1) & t.mask;
    }
}

// Neighbourhood search for the nb listed voxels.
__device__ __forceinline__ void search_cubes(const Tab &t, Pool &P, const uint32_t *list, uint32_t nb) {
    const uint32_t tid = threadIdx.x;
    if (tid == 0) P.nwork = 0;
    if (tid < nb) {
        const uint4 *w = t.words_at(list[tid]);
        const uint4 lo = w[0], hi = w[1];
        P.key[tid] = t.key_at(list[tid]);
        P.count[tid] = lo.y;
        P.sum[0][tid] = (unsigned long long)lo.z | (unsigned long long)lo.w << 32;
        P.sum[1][tid] = (unsigned long long)hi.x | (unsigned long long)hi.y << 32;
        P.sum[2][tid] = (unsigned long long)hi.z | (unsigned long long)hi.w << 32;
    }
    __syncthreads();
    // 32 lanes a voxel, one candidate each (27 of them; the voxel itself is in
    // the sums); eight voxels a lane have their bits loaded together
    const uint32_t c = tid & 31;
    constexpr uint32_t kGroups = kLdThreads / 32, kTogether = 8;
    for (uint32_t v0 = 0; v0 < nb; v0 += kGroups * kTogether) {
        uint32_t home[kTogether], word[kTogether];
#pragma unroll
        for (uint32_t u = 0; u < kTogether; ++u) {
            const uint32_t v = v0 + u * kGroups + (tid >> 5);
            uint64_t key;
            home[u] = kNoSlot;
            word[u] = 0;
            if (v < nb && c < 27 && c != 13 && neighbour_key(P.key[v], c, key)) {
                home[u] = home_of(key, t.mask);
                word[u] = t.occ[home[u] >> 5];
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < kTogether; ++u) {
            const uint32_t v = v0 + u * kGroups + (tid >> 5);
            const bool want = (word[u] >> (home[u] & 31)) & 1u;
            const uint32_t at = wave_reserve(&P.nwork, want);
            if (!want) continue;
            if (at < kWork) {
                P.slot[at] = home[u];
                P.pair[at] = (uint16_t)(v << 5 | c);
            } else {  // the list is full: probed here
                uint64_t key;
                neighbour_key(P.key[v], c, key);
                pool_key(t, P, v, key, home[u]);
            }
        }
    }
    __syncthreads();
    for (uint32_t w = tid; w < min(P.nwork, kWork); w += kLdThreads) {
        uint64_t key;
        neighbour_key(P.key[P.pair[w] >> 5], P.pair[w] & 31u, key);
        pool_key(t, P, P.pair[w] >> 5, key, P.slot[w]);
    }
    __syncthreads();
    for (uint32_t x = tid; x < 3 * nb; x += kLdThreads) {
        const uint32_t v = x / 3, k = x % 3;
        reinterpret_cast<float *>(&t.blend_at(list[v]))[k] =
            cell_average((int64_t)P.sum[k][v], P.count[v], t.frac_bits);
    }
}

// Similar normals along the probe run of voxel s (key K), one lane.
__device__ __forceinline__ void search_normals(const Tab &t, uint64_t K, uint32_t &n, uint64_t &a0, uint64_t &a1,
                                               uint64_t &a2) {
    uint32_t p = home_of(K, t.mask);
    for (uint32_t d = 0; d < t.max_probe;) {
        // the occupied slots from p on, up to the next word boundary, in
        // order: the run ends at the first clear bit
        const uint32_t sh = p & 31;
        const uint32_t w = t.occ[p >> 5] >> sh;
        // (a table of fewer than 32 slots wraps inside its only word)
        const uint32_t span = min(min(32 - sh, t.max_probe - d), t.mask + 1 - p);
        const uint32_t run = min(w == 0xffffffffu ? 32u : (uint32_t)__builtin_ctz(~w), span);
        uint64_t kk[4];
        uint32_t done = 0;
        while (done < run) {
            const uint32_t m = min(run - done, 4u);
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) kk[u] = u < m ? t.key_at((p + done + u) & t.mask) : 0ull;
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                if (u >= m) continue;
                int dot = 0;
#pragma unroll
                for (int a = 0; a < 3; ++a) dot += class_sign(K, a) * class_sign(kk[u], a);
                if (((kk[u] ^ K) & kPosMask) == 0 && dot > 0) add_cell(t, (p + done + u) & t.mask, n, a0, a1, a2);
            }
            done += m;
        }
        if (run < span) break;  // an empty slot ends the run
        d += span;
        p = (p + span) & t.mask;
    }
}

template <int kMode>
__global__ __launch_bounds__(kLdThreads) void low_density_kernel(Tab t, uint32_t below) {
    __shared__ uint32_t list[kLdSlots];
    __shared__ uint32_t nlist;
    const uint32_t nwords = t.nwords();
    const uint32_t nranges = (nwords + kLdWords - 1) / kLdWords;
    for (uint32_t rg = blockIdx.x; rg < nranges; rg += gridDim.x) {
        if (threadIdx.x == 0) nlist = 0;
        __syncthreads();
        const uint32_t j = rg * kLdWords + (threadIdx.x >> 2);
        if (j < nwords) {
            // the counts of the lane's (up to 8) occupied slots are loaded together
            const uint32_t b0 = 8 * (threadIdx.x & 3);
            const uint32_t w = (t.occ[j] >> b0) & 0xffu;
            uint32_t cnt[8];
#pragma unroll
            for (uint32_t b = 0; b < 8; ++b) cnt[b] = ((w >> b) & 1u) ? t.cell_at(j * 32 + b0 + b).count : 0u;
#pragma unroll
            for (uint32_t b = 0; b < 8; ++b)
                if (((w >> b) & 1u) && cnt[b] < below) list[atomicAdd(&nlist, 1u)] = j * 32 + b0 + b;
        }
        __syncthreads();
        const uint32_t m = nlist;
        if constexpr (kMode == 0) {
            __shared__ Pool P;
            for (uint32_t q = 0; q < m; q += kBatch) {
                search_cubes(t, P, list + q, min(m - q, kBatch));
                __syncthreads();  // the sums are rebuilt for the next voxels
            }
        } else {
            for (uint32_t q = threadIdx.x; q < m; q += kLdThreads) {
                const uint32_t s = list[q];
                uint32_t n = 0;
                uint64_t a0 = 0, a1 = 0, a2 = 0;
                search_normals(t, t.key_at(s), n, a0, a1, a2);
                store_pooled(t, s, n, a0, a1, a2);
            }
        }
        __syncthreads();  // the list is rebuilt for the next range
    }
}

hipError_t launch_low_density(const Tab &t, uint32_t below, int mode, hipStream_t st) {
    const uint32_t ranges = (t.nwords() + kLdWords - 1) / kLdWords;
    const uint32_t blocks = ranges < 8192 ? ranges : 8192;
    if (mode == 0)
        low_density_kernel<0><<<blocks, kLdThreads, 0, st>>>(t, below);
    else
        low_density_kernel<1><<<blocks, kLdThreads, 0, st>>>(t, below);
    return hipGetLastError();
}

}  // namespace pfk
