// Work queues of the persistent force kernels.
#pragma once

#include "dev_util.h"
#include "fdx_internal.h"

namespace fdx {

// Next queue slot for this workgroup (thread 0), or kNone when all work is taken.  Without an
// explicit list the groups are split into eight contiguous runs in tree order (at equal
// cumulative cost when bounds are given, else of equal group counts), one queue per XCD
// (consecutive workgroups are dispatched round-robin over the 8 XCDs, so workgroup b runs on
// XCD b % 8); a workgroup pops from its own XCD's queue, keeping neighbouring groups -- which
// share most of their lists -- in one L2, and once that queue is empty takes slots from the
// other XCDs' queues, which balances the load.  With an explicit list (listed) it pops one shared
// queue.
__device__ __forceinline__ uint32_t pop_group(DevStatus *st, uint32_t G, const uint32_t *bounds,
                                              bool listed) {
    if (listed) return atomicAdd(&st->queue_head, 1u);
    const uint32_t x = blockIdx.x % 8u, chunk = (G + 7u) / 8u;
    uint32_t slot = kNone;
    for (uint32_t t = 0; t < 8u && slot == kNone; t++) {
        const uint32_t q = (x + t) & 7u;
        const uint32_t lo = bounds ? bounds[q] : q * chunk;
        const uint32_t hi = bounds ? bounds[q + 1] : min(G, lo + chunk);
        if (lo >= hi) continue;
        const uint32_t k = atomicAdd(&st->xcd_head[q], 1u);
        if (k < hi - lo) slot = lo + k;
    }
    return slot;
}

}  // namespace fdx
