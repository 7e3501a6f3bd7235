// Schedule of the in-place partition of a superparticle list (k_far.hip): near entries from its front
// and far ones from its back, in blocks read ahead from either end.  Plain C++ so that a host program
// can check it.
//
// Entries read and not yet written back are as many as the slots read and not yet overwritten; after
// each block as many ids as have a free slot on their side are written, which leaves at most one kind
// waiting, and the next block to be read comes from that kind's end.  A block is chosen, and its ids
// are read, two blocks before it is sorted in, so at most three blocks of one kind wait.
#pragma once

#include <cstdint>

#if defined(__HIPCC__)
#define FDX_PARTITION_HD __host__ __device__ __forceinline__
#else
#define FDX_PARTITION_HD inline
#endif

namespace fdx {

constexpr uint32_t kFarBlock = 128;               // entries read together
constexpr uint32_t kFarHeld = 4 * kFarBlock;      // ids waiting for a free slot, per kind
static_assert(kFarHeld >= 3 * kFarBlock, "three blocks of one kind may wait");

struct FarPartition {
    struct Block { uint32_t start, len, back; };
    uint32_t ns, lo, hi;                          // entries; those not yet chosen: [lo, hi)
    uint32_t held[2], room[2], put[2];            // near, far: ids waiting, free slots, ids written

    FDX_PARTITION_HD explicit FarPartition(uint32_t n)
        : ns(n), lo(0), hi(n), held{0, 0}, room{0, 0}, put{0, 0} {}
    // the next block, from the front or the back of what is left
    FDX_PARTITION_HD Block choose(uint32_t back) {
        Block b;
        b.len = hi - lo < kFarBlock ? hi - lo : kFarBlock;
        b.back = back;
        if (back) { hi -= b.len; b.start = hi; } else { b.start = lo; lo += b.len; }
        return b;
    }
    // block b is sorted in (its ids are counted in held): its slots are free, and this is the end
    // the next block comes from
    FDX_PARTITION_HD uint32_t sorted(const Block &b) {
        room[0] += b.back ? 0u : b.len;           // constant indices: the counts stay in registers
        room[1] += b.back ? b.len : 0u;
        return held[1] > room[1] ? 1u : 0u;
    }
    // ids of kind c to be written now, from held id held[c] on, to slot(c, 0 ..); then counted
    FDX_PARTITION_HD uint32_t ready(int c) {
        const uint32_t n = held[c] < room[c] ? held[c] : room[c];
        held[c] -= n;
        return n;
    }
    FDX_PARTITION_HD void written(int c, uint32_t n) { put[c] += n; room[c] -= n; }
    FDX_PARTITION_HD uint32_t slot(int c, uint32_t i) const {
        return c ? ns - 1u - (put[1] + i) : put[0] + i;
    }
};

}  // namespace fdx
