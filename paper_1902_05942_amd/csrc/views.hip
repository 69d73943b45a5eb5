// Many views in one persistent launch on gfx950.  A cooperative grid of
// resident workgroups walks three phases -- clear, keys + insert, temporal blend
// -- separated by grid-wide barriers; the lookup follows as a launch of its own.
// Within a phase the work items of all views (chunks of bitmap words, windows of
// vertices) are dealt to the workgroups round-robin, so small and large views
// share the whole chip.  Each group of vertices that share a key in a window
// claims its cell once and adds to it by device atomics, a cell a line
// (accumulate_wave); the blend lists the occupied cells.  (Records in buckets, a
// place each by a device atomic, summed per bin of slots in a phase of their own,
// took more: insert + third phase of 640x360, 800x600, 401x229 and 256x256 x3 277
// us against 213, of 1920x1080 and 1280x720 x3 483 against 425, of 200x90 and
// 150x150 x2 83 against 54.)  The per-vertex and per-cell arithmetic is that of the
// single-view kernels (pf_ops.h).
#include <algorithm>

#include "pf_grid.h"
#include "pf_kernels.h"
#include "pf_merge.h"
#include "pf_once.h"
#include "pf_ops.h"

namespace pfk {

namespace views {

using grid::Barrier;
using grid::grid_barrier;
using grid::kCounterStride;
using grid::kSubCounters;
using grid::poll;

constexpr int kIters = 8;            // block-sized steps per work item

__device__ __forceinline__ Tab to_tab(const pf_table &t) {
    Tab k;
    k.rec = reinterpret_cast<unsigned char *>(t.cell);
    k.occ = t.occ;
    k.stats = reinterpret_cast<unsigned long long *>(t.stats);
    k.mask = (uint32_t)((1ull << t.log2_slots) - 1);
    k.max_probe = t.max_probe;
    k.frac_bits = t.frac_bits;
    k.fsum = 0;  // float tables are rejected on the host
    return k;
}

// LDS merge table of the insert phase: the valid ones of agg_width consecutive
// vertices (block .. kIters * block) merge into at most min(3.375 * block, 1536)
// entries (with the list of valid vertices, kGroups<block> workgroups of them fill
// a compute unit's LDS; at 4 * block entries and without slots one less did, 12
// waves instead of 16 at 256 lanes).  An entry claims its cell when its window
// ends and keeps its sums while the workgroup's next items are of the same view,
// until another step might not find room (more than seven eighths in use): where
// voxels are coarse a workgroup goes to a cell once, not once an item (views of
// 1920x1080 and 1280x720 x3 at cell size 10, 256/256 and 1024/4096: 2500 and 536 ->
// 564 and 347 us; at 0.01 667 and 553 -> 686 and 553).  (With one window per
// agg_width vertices, small images overflowed the table and sent their vertices to
// the cells one by one, and a workgroup's 8 x block vertices left most workgroups
// without any: insert phase of 640x360, 800x600, 401x229 and 256x256 x3 267 -> 197
// us, of 200x90 and 150x150 x2 180 -> 56 us.)
template <int B>
constexpr uint32_t kMergeCap = 27 * B / 8 < 1536 ? 27 * B / 8 : 1536;
template <int B>
constexpr uint32_t kGroups = B == 64 ? 13 : B == 128 ? 8 : B == 256 ? 4 : 2;  // workgroups a compute unit's LDS holds
template <int B>
constexpr uint32_t kEntries = (kMergeCap<B> + B - 1) / B;  // merge-table entries per lane
template <int B>
struct Lds {
    union {
        struct {
            unsigned long long key[kMergeCap<B>];
            unsigned long long s0[kMergeCap<B>], s1[kMergeCap<B>], s2[kMergeCap<B>];
            uint32_t cnt[kMergeCap<B>], slot[kMergeCap<B>];
            uint16_t list[kIters * B];   // the item's valid vertices
            uint32_t nlive, created[kIters];  // valid vertices; entries created by each step
        } m;
        uint32_t cells[8 * B];  // blend: the occupied slots of a range
    };
    uint32_t first[3][PF_MAX_VIEWS + 1];  // per item kind: first global item of each view
    uint32_t hits, nlist, per_item, per_range;
};

// LDS is allotted in pieces of 1280 bytes; the launch rounds up to 2 KB as well
template <int B>
constexpr bool kFits = (sizeof(Lds<B>) + 16 + 2047) / 2048 * 2048 * kGroups<B> <= 160 << 10 &&
                       (sizeof(Lds<B>) + 16 + 1279) / 1280 * 1280 * kGroups<B> <= 160 << 10;
static_assert(kFits<64> && kFits<128> && kFits<256> && kFits<512> && kFits<1024>, "workgroups lost to LDS");

template <int B>
__device__ __forceinline__ void item_of(const Lds<B> &L, int phase, uint32_t nviews, uint32_t it, uint32_t &v,
                                        uint32_t &local) {
    v = 0;
    while (v + 1 < nviews && it >= L.first[phase][v + 1]) ++v;
    local = it - L.first[phase][v];
}

// What a lane keeps of a vertex until its window ends (16 bits): its LDS entry,
// kAlone, or kFlagged and its flags.
constexpr uint32_t kAlone = 0xffffu, kFlagged = 0x8000u;
constexpr uint32_t kUnclaimed = 0xfffffffeu;  // slot of an entry whose cell has not been claimed

// Key, flags and fixed-point contribution of vertex i of a view (masked
// vertices read nothing more than their valid byte).
__device__ __forceinline__ uint8_t view_vertex(const pf_view &d, const Tab &t, float inv_s, uint32_t i, uint64_t &key,
                                               int64_t &q0, int64_t &q1, int64_t &q2) {
    key = 0;
    q0 = q1 = q2 = 0;
    if (d.valid != nullptr && d.valid[i] == 0) return PF_V_INVALID;
    const float x[3] = {d.px[i], d.py[i], d.pz[i]};
    const float nr[3] = {d.nx[i], d.ny[i], d.nz[i]};
    uint32_t fp, home;
    const PcgJump jp(d.kp.seed, d.kp.idx_base);
    const uint32_t rnd[3] = {jp.output(0, i), jp.output(1, i), jp.output(2, i)};
    uint8_t fl = vertex_key(x, nr, true, d.kp.cam, d.kp.s, inv_s, rnd, t.mask, key, fp, home);
    if (fl == 0) fl = fixed_point(d.r[i], d.g[i], d.b[i], t.frac_bits, q0, q1, q2);
    return fl;
}

// Empties the cells of bitmap word j of t and the word.
__device__ __forceinline__ void clear_word(const Tab &t, uint32_t j) {
    uint32_t w = t.occ[j];
    if (w) t.occ[j] = 0;
    while (w) {
        const uint32_t b = __builtin_ctz(w);
        w &= w - 1;
        uint4 *c = t.words_at(j * 32 + b);
        c[0] = make_uint4(0, 0, 0, 0);
        c[1] = make_uint4(0, 0, 0, 0);
    }
}

// At least kWaves waves of this kernel fit a SIMD (the compiler keeps the
// registers within that), which bounds the resident workgroups from below
// independently of the occupancy query.  8, so that two workgroups of 1024 lanes
// share a compute unit and one's barriers hide behind the other, costs 17 spilled
// registers; it pays once the views give every workgroup many items (kMany
// vertices in all): 1024 lanes, widths 1024 / 4096, 4 -> 8 waves: eight views of
// 59.5M vertices 3326 / 2681 -> 3218 / 2482 us, 24.9M 1288 / 1066 -> 1285 / 1006, 18.7M
// 1095 / 917 -> 1106 / 880, 11.1M 671 / 567 -> 689 / 562, 9M 608 / 555 -> 633 / 565, 2.6M
// 325 / 308 -> 343 / 344.  (Smaller workgroups are bound by their LDS.)
constexpr uint64_t kMany = 1ull << 24;

template <int B, int kWaves>
__global__ __launch_bounds__(B) __attribute__((amdgpu_waves_per_eu(kWaves))) void views_kernel(
    const pf_view *__restrict__ views, uint32_t nviews, uint32_t agg, Barrier bar) {
    __shared__ Lds<B> L;
    constexpr uint32_t kItem = (uint32_t)B * kIters;
    // work items per view and kind: 0 clear cur (B bitmap words), 1 keys + insert
    // (agg vertices, or 8 x B), 2 temporal (a range of bitmap words)
    if (threadIdx.x == 0) {
        // items of the insert: agg vertices, fewer where the views would not
        // give every workgroup three
        // (and ranges of the blend: four lanes a bitmap word, fewer words likewise)
        uint64_t total = 0, words_total = 0;
        for (uint32_t v = 0; v < nviews; ++v) {
            total += views[v].n;
            words_total += ((1u << views[v].cur.log2_slots) + 31) / 32;
        }
        uint32_t per_range = B / 4;
        while (per_range > 8 && (uint64_t)per_range * gridDim.x > words_total) per_range /= 2;
        L.per_range = per_range;
        uint32_t per_item = agg ? agg : kItem;
        while (agg && per_item > (uint32_t)B && (uint64_t)per_item * 3 * gridDim.x > total) per_item /= 2;
        L.per_item = per_item;
        uint32_t acc[3] = {0, 0, 0};
        for (uint32_t v = 0; v < nviews; ++v) {
            const pf_view &d = views[v];
            const uint32_t words = ((1u << d.cur.log2_slots) + 31) / 32;
            const uint32_t items[3] = {(words + B - 1) / B, (d.n + per_item - 1) / per_item,
                                       d.temporal ? (words + per_range - 1) / per_range : 0u};
            for (int p = 0; p < 3; ++p) {
                L.first[p][v] = acc[p];
                acc[p] += items[p];
            }
        }
        for (int p = 0; p < 3; ++p) L.first[p][nviews] = acc[p];
    }
    // block 0 stamps the start and the end of every phase (wall clock, as
    // 64-bit values in status words 4..13) for the caller's diagnostics
    auto stamp = [&](int k) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            const uint64_t w = wall_clock64();
            bar.status[4 + 2 * k] = (uint32_t)w;
            bar.status[5 + 2 * k] = (uint32_t)(w >> 32);
        }
    };
    if (blockIdx.x == 0 && threadIdx.x == 0) bar.status[1] = gridDim.x;
    stamp(0);
    __syncthreads();
    const uint32_t G = gridDim.x;

    // ---- phase 0: clear the current tables (nothing to do where the last
    // launch emptied them)
    for (uint32_t it = blockIdx.x; it < L.first[0][nviews]; it += G) {
        uint32_t v, local;
        item_of(L, 0, nviews, it, v, local);
        const Tab t = to_tab(views[v].cur);
        const uint32_t j = local * B + threadIdx.x;  // one bitmap word per lane
        if (j < t.nwords()) clear_word(t, j);
        if (local == 0)
            for (uint32_t k = threadIdx.x; k < PF_STATS_LEN; k += B) t.stats[k] = 0;
    }
    if (!grid_barrier(bar, 1)) return;
    stamp(1);

    // ---- phase 1: keys and insertion.  agg == 0: one claim and one set of
    // device atomics per vertex.  Otherwise an item is agg consecutive vertices
    // (a power of two, block <= agg <= kIters * block; fewer for small views,
    // down to block): its valid ones are listed and merged by key in LDS in
    // windows that end before the table is full; a window's new entries claim
    // their cells, a full table's go to them.
    constexpr uint32_t kCap = kMergeCap<B>, limit = kCap / 8 * 7;
    const uint32_t per_item = L.per_item, per = per_item / B;  // vertices per lane and item (1, 2, 4 or 8)
    const uint32_t tid = threadIdx.x;
    uint32_t used = 0, table_of = 0;  // entries in use, and the view they are of
    auto empty_entry = [&](uint32_t j) {
        L.m.key[j] = kEmpty;
        L.m.s0[j] = 0;
        L.m.s1[j] = 0;
        L.m.s2[j] = 0;
        L.m.cnt[j] = 0;
    };
    if (agg)
        for (uint32_t j = tid; j < kCap; j += B) empty_entry(j);
    // an entry's sums to its cell; every lane of a wavefront calls
    auto add_entry = [&](const Tab &t, uint32_t j, uint32_t jl, bool has, uint32_t slot) {
        const uint32_t c = L.m.cnt[jl];
        accumulate_wave(t, slot, c, (int64_t)L.m.s0[jl], (int64_t)L.m.s1[jl], (int64_t)L.m.s2[jl]);
        if (!has) return;
        if (slot == kNoSlot) add_u64(&t.stats[PF_STAT_PART_OVF + (blockIdx.x & 15)], (unsigned long long)c);
        empty_entry(j);
    };
    // all entries (their cells are claimed)
    auto flush = [&](const Tab &t) {
#pragma unroll
        for (uint32_t e = 0; e < kEntries<B>; ++e) {
            const uint32_t j = e * B + tid, jl = min(j, kCap - 1);
            const bool has = j < kCap && L.m.key[jl] != kEmpty;
            add_entry(t, j, jl, has, has ? L.m.slot[jl] : kNoSlot);
        }
        used = 0;
    };
    for (uint32_t it = blockIdx.x; it < L.first[1][nviews]; it += G) {
        uint32_t v, local;
        item_of(L, 1, nviews, it, v, local);
        const pf_view &d = views[v];
        const Tab t = to_tab(d.cur);
        const float inv_s = 1.0f / d.kp.s;
        if (agg == 0) {
            for (int k = 0; k < kIters; ++k) {
                const uint32_t i = local * kItem + k * B + threadIdx.x;
                if (local * kItem + k * B >= d.n) break;
                uint64_t key = 0;
                int64_t q0 = 0, q1 = 0, q2 = 0;
                uint32_t slot = kNoSlot;
                if (i < d.n) {
                    uint8_t fl = view_vertex(d, t, inv_s, i, key, q0, q1, q2);
                    if (fl == 0) {
                        slot = find_or_claim(t, key);
                        if (slot == kNoSlot) {
                            fl = PF_V_OVERFLOW;
                            add_u64(&t.stats[PF_STAT_PART_OVF + (blockIdx.x & 15)], 1ull);
                        }
                    }
                    if (d.key) d.key[i] = key;
                    d.vflags[i] = fl;
                    d.slot[i] = slot;
                }
                accumulate_wave(t, slot, 1, q0, q1, q2);
            }
            continue;
        }
        const uint32_t c0 = local * per_item, i1 = min(d.n, c0 + per_item);
        if (tid < kIters) L.m.created[tid] = 0;
        if (tid == 0) L.m.nlive = 0;
        // the valid bytes first; masked vertices read nothing more
        uint32_t live = 0;
        for (uint32_t u = 0; u < per; ++u) {
            const uint32_t i = c0 + u * B + tid;
            live |= (i < i1 && (d.valid == nullptr || d.valid[i] != 0) ? 1u : 0u) << u;
        }
        __syncthreads();
        for (uint32_t u = 0; u < per; ++u) {
            const uint32_t i = c0 + u * B + tid;
            const bool v = (live >> u) & 1u;
            const uint32_t at = wave_reserve(&L.m.nlive, v);
            if (v) {
                L.m.list[at] = (uint16_t)(u * B + tid);
            } else if (i < i1) {
                d.vflags[i] = PF_V_INVALID;
                if (d.key) d.key[i] = 0;
                d.slot[i] = kNoSlot;
            }
        }
        __syncthreads();
        const uint32_t nlive = L.m.nlive, nsteps = (nlive + B - 1) / B;
        if (used && nsteps && v != table_of) {
            flush(to_tab(views[table_of].cur));
            __syncthreads();
        }
        if (nsteps) table_of = v;
        for (uint32_t w0 = 0, w1; w0 < nsteps; w0 = w1) {
            // a lane keeps 16 bits of a vertex until its window ends: its LDS
            // entry, kAlone (no room), or kFlagged and its flags
            uint64_t code[2] = {0, 0};
            uint32_t u = w0;
            while (true) {
                const uint32_t l = u * B + tid;
                uint32_t c = kFlagged;
                bool fresh = false;
                if (l < nlive) {
                    const uint32_t i = c0 + L.m.list[l];
                    uint64_t k;
                    int64_t q0, q1, q2;
                    c = view_vertex(d, t, inv_s, i, k, q0, q1, q2);
                    if (d.key) d.key[i] = k;
                    if (c == 0) {
                        const int e = lds_insert(L.m.key, kCap, k, fresh);
                        if (e >= 0) {
                            if (fresh) L.m.slot[e] = kUnclaimed;
                            atomicAdd(&L.m.cnt[e], 1u);
                            lds_add(&L.m.s0[e], q0);
                            lds_add(&L.m.s1[e], q1);
                            lds_add(&L.m.s2[e], q2);
                            c = (uint32_t)e;
                        } else {
                            c = kAlone;
                        }
                    } else {
                        c |= kFlagged;
                    }
                }
                const uint64_t m = __ballot(fresh);
                if ((tid & 63) == 0 && m) atomicAdd(&L.m.created[u], (uint32_t)__popcll(m));
                const uint64_t cb = (uint64_t)c << (16 * ((u - w0) & 3));
                if (u - w0 < 4)
                    code[0] |= cb;
                else
                    code[1] |= cb;
                ++u;
                if (u == nsteps) break;
                const uint32_t next = min(nlive - u * B, (uint32_t)B);
                if (used + (u - w0) * B + next <= limit) continue;
                __syncthreads();
                uint32_t now = used;
                for (uint32_t x = w0; x < u; ++x) now += L.m.created[x];
                if (now + next > limit) break;
            }
            w1 = u;
            __syncthreads();
            for (uint32_t x = w0; x < w1; ++x) used += L.m.created[x];
            const bool full = w1 < nsteps || used + B > limit;  // no room for another step
            // one claim per new entry; a lane's entries issue their home-slot
            // loads, then their compare-and-swaps on empty home slots, before
            // any result is used
            uint64_t gk[kEntries<B>];
            uint32_t sl[kEntries<B>], fs[kEntries<B>], ff[kEntries<B>], fc[kEntries<B>];
            bool won[kEntries<B>];
#pragma unroll
            for (uint32_t e = 0; e < kEntries<B>; ++e) {
                const uint32_t j = e * B + tid, jl = min(j, kCap - 1);
                gk[e] = j < kCap ? L.m.key[jl] : kEmpty;
                sl[e] = gk[e] != kEmpty ? L.m.slot[jl] : kNoSlot;
                fs[e] = ff[e] = fc[e] = 0;
                if (sl[e] == kUnclaimed) {
                    fs[e] = home_of(gk[e], t.mask);
                    ff[e] = fingerprint_of(gk[e]);
                    fc[e] = load_fp_probe(&t.cell_at(fs[e]).fp);
                }
            }
#pragma unroll
            for (uint32_t e = 0; e < kEntries<B>; ++e) {
                won[e] = false;
                if (sl[e] == kUnclaimed && fc[e] == 0) {
                    uint32_t expected = 0;
                    won[e] = __hip_atomic_compare_exchange_strong(&t.cell_at(fs[e]).fp, &expected, ff[e],
                                                                  __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                                  __HIP_MEMORY_SCOPE_AGENT);
                    fc[e] = won[e] ? ff[e] : expected;
                }
            }
#pragma unroll
            for (uint32_t e = 0; e < kEntries<B>; ++e) {
                const uint32_t j = e * B + tid, jl = min(j, kCap - 1);
                if (sl[e] == kUnclaimed) {
                    if (won[e]) claimed<true>(t, fs[e], gk[e]);
                    // the home slot holds another key: probe on from the next
                    sl[e] = fc[e] == ff[e] ? fs[e] : claim_from<true>(t, gk[e], ff[e], (fs[e] + 1) & t.mask, 1);
                    L.m.slot[j] = sl[e];
                }
                if (full) add_entry(t, j, jl, gk[e] != kEmpty, sl[e]);  // uniform
            }
            if (full) used = 0;
            __syncthreads();
#pragma unroll 1
            for (uint32_t x = w0; x < w1; ++x) {
                const uint32_t l = x * B + tid;
                if (l >= nlive) break;
                const uint32_t i = c0 + L.m.list[l], at = x - w0;
                const uint32_t c = (uint32_t)((at < 4 ? code[0] : code[1]) >> (16 * (at & 3))) & 0xffffu;
                uint32_t slot = kNoSlot;
                uint8_t fl = 0;
                if (c < kFlagged) {
                    slot = L.m.slot[c];
                    if (slot == kNoSlot) fl = PF_V_OVERFLOW;
                } else if (c == kAlone) {  // no room in the LDS table: on its own
                    uint64_t k;
                    int64_t q0, q1, q2;
                    view_vertex(d, t, inv_s, i, k, q0, q1, q2);
                    slot = find_or_claim(t, k);
                    if (slot != kNoSlot) {
                        accumulate(t, slot, 1, q0, q1, q2);
                    } else {
                        add_u64(&t.stats[PF_STAT_PART_OVF + (blockIdx.x & 15)], 1ull);
                        fl = PF_V_OVERFLOW;
                    }
                } else {
                    fl = (uint8_t)(c & 0xffu);
                }
                d.vflags[i] = fl;
                d.slot[i] = slot;
            }
            __syncthreads();  // the slots are read: the next window's follow
        }
    }
    if (used) flush(to_tab(views[table_of].cur));
    if (!grid_barrier(bar, 2)) return;
    stamp(2);

    // ---- phase 2: the temporal values of the occupied cells, listed range by
    // range so that every lane has one
    for (uint32_t it = blockIdx.x; it < L.first[2][nviews]; it += G) {
        uint32_t v, local;
        item_of(L, 2, nviews, it, v, local);
        const pf_view &d = views[v];
        const Tab cur = to_tab(d.cur);
        const bool has_prev = d.prev.cell != nullptr;
        const Tab prev = has_prev ? to_tab(d.prev) : cur;
        const float alpha = d.alpha_old, beta = 1.0f - d.alpha_old;
        const uint32_t wl = threadIdx.x >> 2, j = local * L.per_range + wl, sh = 8 * (threadIdx.x & 3);
        uint32_t w = wl < L.per_range && j < cur.nwords() ? (cur.occ[j] >> sh) & 0xffu : 0u;
        if (threadIdx.x == 0) {
            L.nlist = 0;
            L.hits = 0;
        }
        __syncthreads();
        if (w) {
            uint32_t at = atomicAdd(&L.nlist, (uint32_t)__popc(w));
            for (; w; w &= w - 1) L.cells[at++] = j * 32 + sh + (uint32_t)__builtin_ctz(w);
        }
        __syncthreads();
        uint32_t hits = 0;
        for (uint32_t q = threadIdx.x; q < L.nlist; q += B) {
            const uint32_t sl[1] = {L.cells[q]};
            const CellWords c = load_cell(cur, sl[0]);
            const bool has[1] = {true};
            const uint64_t key[1] = {c.key};
            const uint32_t fp[1] = {c.cell.fp}, n[1] = {c.cell.count};
            uint32_t keep[1] = {c.cell.count};
            float val[1][3] = {{cur.average(c.cell, 0), cur.average(c.cell, 1), cur.average(c.cell, 2)}};
            if (has_prev)
                hits += blend_cells<true, false, 1, false>(cur, prev, sl, has, key, fp, val, n, keep, alpha, beta, 0u);
            else
                blend_cells<false, false, 1, false>(cur, prev, sl, has, key, fp, val, n, keep, alpha, beta, 0u);
        }
        if (hits) atomicAdd(&L.hits, hits);
        __syncthreads();  // the list is read; the next range's follows
        if (threadIdx.x == 0 && L.hits) add_u64(&cur.stats[PF_STAT_PART_HIT + (blockIdx.x & 31)], L.hits);
    }
    // no barrier after it: the lookup is a launch of its own, workgroup 0 stamps
    // its own end
    stamp(3);
}

// The last phase, a launch of its own: the previous tables emptied (read for the
// last time by the blend), then every vertex looked up; the clear's items come
// first, so its scattered stores overlap the lookup's gathers.  A plain gather,
// bound by the lines in flight, that wants all the waves a compute unit holds: as
// the last phase of views_kernel, whose registers are the insert's, it had half
// of them (eight views of 59.5M vertices 750 -> 488 us; 540 when all phases shared
// 64 registers).  The launch's start takes the place of a grid barrier: whole
// calls of 640x360, 800x600, 401x229 and 256x256 x3 at 1024 lanes 327 -> 313 us, at
// 256 404 -> 365, of 200x90 and 150x150 x2 130 -> 113.  Two vertices a lane: 1 or 4
// are within 2%.
constexpr int kLookT = 256, kLook = 2;  // threads; vertices a lane has in flight
constexpr uint32_t kLookGroups = 8;     // workgroups a compute unit
__global__ __launch_bounds__(kLookT) __attribute__((amdgpu_waves_per_eu(8))) void views_lookup_kernel(
    const pf_view *__restrict__ views, uint32_t nviews, Barrier bar) {
    if (bar.status[0]) return;  // a phase before gave up waiting
    // lane v of every wavefront: where view v's items end among those of its kind
    static_assert(PF_MAX_VIEWS <= 64, "a lane a view");
    constexpr uint32_t kItem = kLookT * kLook;
    const uint32_t lane = threadIdx.x & 63;
    uint32_t end_clear = 0, end_look = 0;
    if (lane < nviews) {
        const pf_view &d = views[lane];
        end_clear = d.prev.cell ? (((1u << d.cur.log2_slots) + 31) / 32 + kLookT - 1) / kLookT : 0u;
        end_look = (d.n + kItem - 1) / kItem;
    }
    const uint32_t own_clear = end_clear, own_look = end_look;
#pragma unroll
    for (uint32_t off = 1; off < 64; off <<= 1) {
        const uint32_t c = (uint32_t)__shfl_up((int)end_clear, off), l = (uint32_t)__shfl_up((int)end_look, off);
        if (lane >= off) {
            end_clear += c;
            end_look += l;
        }
    }
    const uint32_t n_clear = (uint32_t)__shfl((int)end_clear, 63), n_look = (uint32_t)__shfl((int)end_look, 63);
    for (uint32_t it = blockIdx.x; it < n_clear + n_look; it += gridDim.x) {
        const bool clears = it < n_clear;
        const uint32_t k = clears ? it : it - n_clear;
        const int v = __builtin_ctzll(__ballot((clears ? end_clear : end_look) > k));
        const uint32_t local =
            k - (uint32_t)(clears ? __shfl((int)(end_clear - own_clear), v) : __shfl((int)(end_look - own_look), v));
        const pf_view &d = views[__builtin_amdgcn_readfirstlane(v)];
        if (clears) {
            const Tab t = to_tab(d.prev);
            const uint32_t j = local * kLookT + threadIdx.x;
            if (j < t.nwords()) clear_word(t, j);
            continue;
        }
        const Tab t = to_tab(d.cur);
        // the slots of a lane's vertices (kNoSlot for flagged ones), then every
        // value they read, then the stores
        uint32_t slot[kLook];
        float4 val[kLook];
        const uint32_t i0 = local * kItem + threadIdx.x;
#pragma unroll
        for (int u = 0; u < kLook; ++u) slot[u] = i0 + u * kLookT < d.n ? d.slot[i0 + u * kLookT] : kNoSlot;
#pragma unroll
        for (int u = 0; u < kLook; ++u)
            if (i0 + u * kLookT < d.n)
                val[u] = lookup_value(t, slot[u], i0 + u * kLookT, d.r, d.g, d.b, d.temporal != 0);
#pragma unroll
        for (int u = 0; u < kLook; ++u) {
            const uint32_t i = i0 + u * kLookT;
            if (i >= d.n) continue;
            d.r_out[i] = val[u].x;
            d.g_out[i] = val[u].y;
            d.b_out[i] = val[u].z;
            if (d.count_out) d.count_out[i] = slot[u] == kNoSlot ? 0u : (uint32_t)val[u].w;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {  // its own end
        const uint64_t w = wall_clock64();
        bar.status[12] = (uint32_t)w;
        bar.status[13] = (uint32_t)(w >> 32);
    }
}

__global__ void views_reset_kernel(uint32_t *ws, uint32_t words) {
    for (uint32_t j = threadIdx.x; j < words; j += blockDim.x) ws[j] = 0;
}

// Workspace: barrier counters, then the device copy of the descriptors.
static size_t align256(size_t x) { return (x + 255) / 256 * 256; }
static size_t descriptors_at() { return align256(sizeof(uint32_t) * kCounterStride * (2 * kSubCounters + 2)); }

// A device's compute units, the workgroups of a kernel that are resident on each
// at once, and its wall clock's rate: asked for once per device.
struct Shape {
    uint32_t cus, resident;
    uint64_t ticks_per_s;
};

template <int B, int kWaves = 4>
hipError_t launch_b(const pf_view *views, uint32_t nviews, uint32_t agg, uint32_t per_cu, uint32_t *ws,
                    hipStream_t st) {
    static PerDevice<Shape> shapes;
    Shape sh;
    const hipError_t q = shapes.get(sh, [](int dev, Shape &out) {
        int resident = 0, cus = 0, lds_cu = 0, khz = 0;
        hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&resident,
                                                         reinterpret_cast<const void *>(views_kernel<B, kWaves>), B, 0);
        if (e != hipSuccess) return e;
        // every workgroup of a cooperative grid must be resident at once: the
        // LDS-bound count is taken as well, with the static LDS rounded up to
        // 2 KB and to the hardware's 1280 bytes (a 128th of 160 KB), so that an
        // allocation granularity the occupancy query may not model cannot
        // leave a workgroup waiting for a slot
        e = hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev);
        if (e != hipSuccess) return e;
        hipFuncAttributes fa;
        e = hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(views_kernel<B, kWaves>));
        if (e != hipSuccess) return e;
        const size_t per_wg = std::max((fa.sharedSizeBytes + 2047) / 2048 * 2048,
                                       (fa.sharedSizeBytes + 1279) / 1280 * 1280);
        if (per_wg > 0 && lds_cu > 0 && (size_t)resident * per_wg > (size_t)lds_cu)
            resident = (int)((size_t)lds_cu / per_wg);
        // and the register-bound count the compiler guarantees (4 SIMDs)
        constexpr int by_waves = 4 * kWaves * 64 / B;
        if (resident > by_waves) resident = by_waves;
        if (resident < 1) return hipErrorInvalidConfiguration;
        e = hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev);
        if (e != hipSuccess) return e;
        out.resident = (uint32_t)resident;
        out.cus = (uint32_t)cus;
        out.ticks_per_s = (uint64_t)(khz > 0 ? khz : 100000) * 1000ull;
        return hipSuccess;
    });
    if (q != hipSuccess) return q;
    const Barrier bar = grid::barrier_at(ws, 2 * sh.ticks_per_s);  // a phase never takes seconds
    views_reset_kernel<<<1, 256, 0, st>>>(ws, grid::kWords);
    const uint32_t per = (per_cu == 0 || per_cu > sh.resident) ? sh.resident : per_cu;
    const uint32_t grid = per * sh.cus;
    void *args[] = {(void *)&views, (void *)&nviews, (void *)&agg, (void *)&bar};
    const hipError_t e = hipLaunchCooperativeKernel(reinterpret_cast<const void *>(views_kernel<B, kWaves>), dim3(grid),
                                                    dim3(B), args, 0, st);
    if (e != hipSuccess) return e;
    views_lookup_kernel<<<sh.cus * kLookGroups, kLookT, 0, st>>>(views, nviews, bar);
    return hipGetLastError();
}

}  // namespace views

size_t views_workspace_bytes(uint32_t nviews) {
    return views::descriptors_at() + views::align256(nviews * sizeof(pf_view));
}

hipError_t launch_views(const pf_view *host_views, uint32_t nviews, uint32_t block, uint32_t agg, uint32_t per_cu,
                        void *workspace, hipStream_t st) {
    pf_view *dev = reinterpret_cast<pf_view *>(reinterpret_cast<char *>(workspace) + views::descriptors_at());
    hipError_t e = hipMemcpyAsync(dev, host_views, nviews * sizeof(pf_view), hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return e;
    uint32_t *ws = reinterpret_cast<uint32_t *>(workspace);
    uint64_t total = 0;
    for (uint32_t v = 0; v < nviews; ++v) total += host_views[v].n;
    switch (block) {
        case 64: return views::launch_b<64>(dev, nviews, agg, per_cu, ws, st);
        case 128: return views::launch_b<128>(dev, nviews, agg, per_cu, ws, st);
        case 256: return views::launch_b<256>(dev, nviews, agg, per_cu, ws, st);
        case 512: return views::launch_b<512>(dev, nviews, agg, per_cu, ws, st);
        case 1024:
            return total >= views::kMany ? views::launch_b<1024, 8>(dev, nviews, agg, per_cu, ws, st)
                                         : views::launch_b<1024>(dev, nviews, agg, per_cu, ws, st);
        default: return hipErrorInvalidConfiguration;
    }
}

}  // namespace pfk
