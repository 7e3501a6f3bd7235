// Work queues of the persistent kernels.
#pragma once

#include "dev_util.h"
#include "fdx_internal.h"

namespace fdx {

__device__ __forceinline__ uint32_t take_slot(uint32_t *head) {
    uint32_t k = 0;
    if (lane_id() == 0) k = atomicAdd(head, 1u);
    return uniform_u32(k);
}

// Next queue slot for this consumer, or kNone when all work is taken; called by a whole wave.  A
// workgroup has PER consumers (its waves, or one); w is this one; first is set at its first
// call, which takes the slot of the consumer's own number without an atomic: the counters start
// behind those.  Without an explicit list the groups are split into eight contiguous runs in tree
// order (at equal cumulative cost when bounds are given, else of equal group counts), one queue per
// XCD (consecutive workgroups are dispatched round-robin over the 8 XCDs, so workgroup b runs
// on XCD b % 8); a workgroup pops from its own XCD's queue, keeping neighbouring groups --
// which share most of their lists -- in one L2, and once that queue is empty takes slots
// from the other XCDs' queues, which balances the load.  With an explicit list (listed) of G it
// pops one shared queue.
//
// The counters share a cache line, and atomic additions to it from all XCDs follow one another at
// 12.4 ns each: 5120 waves that each tried eight queues kept the chip for 0.5 ms.  So a consumer
// whose queue is empty reads all counters with one load and only adds to one that has slots left.
// (A read before every addition made the force kernel of 245657 groups 16.5 ms, from 8.9.)
template <uint32_t PER>
__device__ __forceinline__ uint32_t pop_group(DevStatus *st, uint32_t G, const uint32_t *bounds,
                                              bool listed, bool first, uint32_t w) {
    if (listed) {
        const uint32_t own = gridDim.x * PER;
        if (first) {
            const uint32_t k = blockIdx.x * PER + w;
            return k < G ? k : kNone;
        }
        if (G <= own) return kNone;
        const uint32_t k = take_slot(&st->queue_head);
        return k < G - own ? own + k : kNone;
    }
    // lane q < 8: queue q's first group, and how many of it the counter hands out
    const uint32_t x = blockIdx.x % 8u, q = (uint32_t)lane_id() & 7u, chunk = (G + 7u) / 8u;
    const uint32_t lo = bounds ? bounds[q] : q * chunk;
    const uint32_t hi = bounds ? bounds[q + 1] : min(G, lo + chunk);
    const uint32_t own = (gridDim.x - q + 7u) / 8u * PER;          // consumers of that XCD
    const uint32_t n = hi > lo ? hi - lo : 0u, dyn = n > own ? n - own : 0u, base = lo + n - dyn;
    auto of = [](uint32_t v, uint32_t lane) {
        return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane);
    };
    if (first) {
        const uint32_t k = blockIdx.x / 8u * PER + w;
        if (k < of(n, x)) return of(lo, x) + k;
    } else if (of(dyn, x) != 0) {
        const uint32_t k = take_slot(&st->xcd_head[x]);
        if (k < of(dyn, x)) return of(base, x) + k;
    }
    while (__ballot(dyn != 0) != 0) {
        const bool left = dyn != 0 && __hip_atomic_load(&st->xcd_head[q], __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT) < dyn;
        const uint32_t m = (uint32_t)__ballot(left) & 0xFFu;
        if (m == 0) break;
        // the next queue after the own one
        const uint32_t rot = (m | m << 8) >> x & 0xFFu;
        const uint32_t t = (x + (uint32_t)__builtin_ctz(rot)) & 7u;
        const uint32_t k = take_slot(&st->xcd_head[t]);
        if (k < of(dyn, t)) return of(base, t) + k;
    }
    return kNone;
}

}  // namespace fdx
