// Temporal blend over two sets of averages (Section 3.4.1) for gfx950: the
// current table's cells listed range by range (list_cells), then one a lane, so
// the work beyond the bitmap read is proportional to the cells of the current
// frame.  Bound by the latency of a cell's chain (cell, previous table's slot,
// its key and value): four lanes a bitmap word, each walking its cells, took 22
// us for the 211k cells of a 1280x720x3 frame, this 18 us; 4k cells of a 2^14-slot
// table take 6 us, 46k of 2^16 slots 10 us.
#include "pf_kernels.h"
#include "pf_ops.h"

namespace pfk {

template <bool kHasPrev, bool kIntegrate, bool kLevels = false>
__global__ __launch_bounds__(kBlock) void temporal_kernel(Tab cur, Tab prev, float alpha, float beta, uint32_t cap) {
    __shared__ CellList L;
    uint32_t hits = 0;
    for (uint32_t rg = blockIdx.x; rg < list_ranges(cur); rg += gridDim.x) {
        const uint32_t m = list_cells(cur, rg, L);
        for (uint32_t q = threadIdx.x; q < m; q += kBlock) {
            const uint32_t s[1] = {L.slot[q]};
            const CellWords c = load_cell(cur, s[0]);
            const bool has[1] = {true};
            const uint64_t key[1] = {c.key};
            const uint32_t fp[1] = {c.cell.fp}, n[1] = {c.cell.count};
            uint32_t keep[1] = {kIntegrate ? min(c.cell.count, cap) : c.cell.count};
            float v[1][3] = {{cur.average(c.cell, 0), cur.average(c.cell, 1), cur.average(c.cell, 2)}};
            hits += blend_cells<kHasPrev, kIntegrate, 1, kLevels>(cur, prev, s, has, key, fp, v, n, keep, alpha, beta,
                                                                  cap);
        }
        __syncthreads();
    }
    if constexpr (kHasPrev) {
        // one device atomic per block, spread over 32 partial counters
        __shared__ uint32_t s_hits;
        if (threadIdx.x == 0) s_hits = 0;
        __syncthreads();
        if (hits) atomicAdd(&s_hits, hits);
        __syncthreads();
        if (threadIdx.x == 0 && s_hits) add_u64(&cur.stats[PF_STAT_PART_HIT + (blockIdx.x & 31)], s_hits);
    }
}

hipError_t launch_temporal(const Tab &cur, const Tab *prev, float alpha_old, int mode, uint32_t cap,
                           hipStream_t st) {
    const float beta = 1.0f - alpha_old;
    uint32_t blocks = list_ranges(cur);
    if (blocks > 16384) blocks = 16384;
    const bool levels = (mode & PF_TEMPORAL_ACROSS_LEVELS) != 0;
    mode &= ~PF_TEMPORAL_ACROSS_LEVELS;
    if (levels && prev) {  // without a previous table there is nothing to search
        if (mode == 1)
            temporal_kernel<true, true, true><<<blocks, kBlock, 0, st>>>(cur, *prev, 0.0f, 0.0f, cap);
        else
            temporal_kernel<true, false, true><<<blocks, kBlock, 0, st>>>(cur, *prev, alpha_old, beta, cap);
    } else if (mode == 1) {
        if (prev)
            temporal_kernel<true, true><<<blocks, kBlock, 0, st>>>(cur, *prev, 0.0f, 0.0f, cap);
        else
            temporal_kernel<false, true><<<blocks, kBlock, 0, st>>>(cur, cur, 0.0f, 0.0f, cap);
    } else {
        if (prev)
            temporal_kernel<true, false><<<blocks, kBlock, 0, st>>>(cur, *prev, alpha_old, beta, cap);
        else
            temporal_kernel<false, false><<<blocks, kBlock, 0, st>>>(cur, cur, alpha_old, beta, cap);
    }
    return hipGetLastError();
}

}  // namespace pfk
