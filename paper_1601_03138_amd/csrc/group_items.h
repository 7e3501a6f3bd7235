// Work items of the kernels that take groups in a fixed order (density, cutoff force, far field, direct
// force launches): how many items a group makes and which block takes which, plain C++ so that a
// host program can check them.
//
// A group's runs of members (its passes) are independent, so they may be shared out over several
// waves or workgroups without changing a result.  Items are numbered part by part, item = part x
// groups + group: a part that few groups have makes one stretch of empty items, not a pattern of them
// over the chip.
//
// Blocks go to the 8 XCDs in turn, and the blocks of one XCD take runs of `run` consecutive blocks of
// items, so groups near each other, whose lists overlap, are worked on behind one L2, while every
// XCD still gets dense and sparse regions.  Grids are multiples of 8 run, or the whole of it.
#pragma once

#include <cstddef>
#include <cstdint>

#if defined(__HIPCC__)
#define FDX_ITEMS_HD __host__ __device__
#else
#define FDX_ITEMS_HD
#endif

namespace fdx {

constexpr uint32_t kXcdRun = 64;
FDX_ITEMS_HD inline uint32_t xcd_run_blocks(size_t blocks, uint32_t run = kXcdRun) {
    return (uint32_t)((blocks + 8 * run - 1) / (8 * run) * (8 * run));
}
FDX_ITEMS_HD inline uint32_t xcd_run_block(uint32_t vb, uint32_t run = kXcdRun) {
    const uint32_t nb = vb / 8u;
    return (nb / run * 8u + vb % 8u) * run + nb % run;
}
// longest run, at most `most`, with which every XCD gets 16 runs or more
inline uint32_t xcd_direct_run(size_t blocks, uint32_t most) {
    uint32_t r = most;
    while (r > 1 && 8 * 16 * (size_t)r > blocks) r >>= 1;
    return r;
}

struct GroupItems {
    uint32_t parts, run, blocks;      // items per group; blocks per XCD run; blocks in all
};
// Groups of up to `most` parts, split so that there are `want` items or more, per_block items to a
// block.
inline GroupItems group_items(size_t groups, uint32_t most, size_t want, uint32_t per_block,
                              uint32_t run_most) {
    const size_t p = groups ? (want + groups - 1) / groups : 1;
    GroupItems o;
    o.parts = p < 1 ? 1u : p < most ? (uint32_t)p : most;
    const size_t blocks = (groups * o.parts + per_block - 1) / per_block;
    o.run = xcd_direct_run(blocks, run_most);
    o.blocks = xcd_run_blocks(blocks, o.run);
    return o;
}

// Density: a wave takes runs of up to kRunMax members.  It needs several waves on every SIMD, and the
// groups of a small set, or large groups, are too few.  Whole call of 2e5 uniform particles, 4.2
// spacings, n_group 512: a wave per group 2.30 ms, 16384 items 0.67; 20000 particles, 7 spacings, n_group
// 64: 0.86 and 0.46; n_group 512: 3.57 and 0.57.  140 calls of 500 to 10^6 particles with 4096 / 8192 /
// 16384 / 32768 items: 0.48 / 0.47 / 0.47 / 0.47 of the time that a workgroup per group took.
constexpr uint32_t kRunMax = 16;
constexpr size_t kDensityItems = 16384;
inline GroupItems density_items(size_t groups, int n_group) {
    return group_items(groups, ((uint32_t)n_group + kRunMax - 1) / kRunMax, kDensityItems, 4, kXcdRun);
}

// Cutoff force: a workgroup takes a pass of up to kSiftPass members, all passes of a group unless
// groups are few.  3e5 uniform particles, n_group 512 (770 groups), FP32, cutoff of 6 spacings: 1.21 ms
// with a workgroup per group, 1.04 / 0.93 / 0.89 with 4096 / 8192 / 16384 items.
constexpr uint32_t kSiftPass = 80;        // 20 members per wave, three entries at a time
constexpr size_t kCutItems = 16384;
FDX_ITEMS_HD inline uint32_t sift_passes(uint32_t ni) { return (ni + kSiftPass - 1) / kSiftPass; }
inline GroupItems cut_items(size_t groups, int n_group) {
    return group_items(groups, sift_passes((uint32_t)n_group), kCutItems, 1, kXcdRun);
}

}  // namespace fdx
