// Merging of vertices that share a key inside a workgroup before they touch
// the table, shared by the binned insert (binned.hip) and the batched
// multi-view launch (views.hip): vertices merge by key in an LDS hash table
// of (key, count, fixed-point sums) entries.
#pragma once

#include "pf_device.h"

namespace pfk {

constexpr uint64_t kEmpty = ~0ull;  // no key has bit 63 set
constexpr uint32_t kLdsProbe = 32;  // LDS probes before a vertex goes alone

// Index of this lane among the lanes of its wavefront that pass want=true,
// the lowest of them reserving the whole range on *ctr.  Every lane of the
// wavefront must call.
__device__ __forceinline__ uint32_t wave_reserve(uint32_t *ctr, bool want) {
    const uint64_t m = __ballot(want);
    const uint32_t rank =
        __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    uint32_t base = 0;
    if (m != 0) {
        const int leader = __builtin_ctzll(m);
        if ((int)(threadIdx.x & 63) == leader) base = atomicAdd(ctr, (uint32_t)__popcll(m));
        base = __shfl(base, leader);
    }
    return base + rank;
}

// LDS entry of `key` in the window's table (inserted if absent, then fresh is
// set), or -1 when the kLdsProbe entries of its probe sequence hold other
// keys.  The probes are 1, 2, 3, ... apart, so that a nearly full table has
// no runs to walk along.
__device__ __forceinline__ int lds_insert(unsigned long long *lkey, uint32_t cap, uint64_t key, bool &fresh) {
    uint32_t j = (uint32_t)(((uint64_t)(uint32_t)((key * 0x9E3779B97F4A7C15ull) >> 32) * cap) >> 32);
#pragma unroll 1
    for (uint32_t d = 1; d <= kLdsProbe; ++d) {
        const unsigned long long old = atomicCAS(&lkey[j], (unsigned long long)kEmpty, (unsigned long long)key);
        fresh = old == kEmpty;
        if (fresh || old == key) return (int)j;
        j = j + d >= cap ? j + d - cap : j + d;
    }
    return -1;
}


}  // namespace pfk
