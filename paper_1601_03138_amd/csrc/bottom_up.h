// Sums over a tree from the leaves up in one to three launches (moments, largest support radii).
//
// Cells are numbered breadth first and, within a level, in the order of their particles.  The sorted
// particles are cut into blocks of `span`.  Cells inside one block have all of their children inside
// it, so a workgroup finishes its block level by level with a barrier between levels.  What is left
// crosses a block boundary: at most one cell per boundary and level.  Those are finished with a thread
// per boundary, again level by level (a cell that crosses several boundaries belongs to the first):
// first the cells inside each group of kUpFan blocks, a workgroup per group, then the rest.
//
// Bound by the chain of loads from level to level (1.5 to 4 us each), for large sets by the bytes.  A
// launch per level waited for 22 launches, most of them of levels with few cells or none.  Moments
// of all cells (with the leaves' launch), before / now: 4096 particles 70 / 27 us, 21k 81 / 46 us,
// 2^20 137 / 98 us, 3 10^6 244 / 198 us, 2^24 705 / 673 us.
//
// Where a block's cells of a level start is known from the build: the scanned counts per tile of
// kTileW positions and level (tree_build's scratch).
#pragma once

#include "dev_util.h"
#include "fdx_internal.h"

namespace fdx {

constexpr int kUpThreads = 512;
constexpr uint32_t kUpFan = 32;          // blocks per group of the second launch
constexpr uint32_t kUpBlocks = kUpFan * kUpThreads;    // most blocks

// Particles per block, at least: 3 10^6 particles 198 us (2048: 211, 1024: 237).  Up to kUpOne
// particles one block: 4096 particles 26 us (two blocks and their boundary: 50).
constexpr uint32_t kUpMinSpan = 4096;
constexpr uint32_t kUpOne = 8192;

struct UpBlocks {
    const uint32_t *woff;                // tile starts, level-major
    const int64_t *off;
    uint64_t n;
    uint32_t ntiles, tiles, nb;          // tiles in all, per block; blocks
    int nsys;
};

inline UpBlocks up_blocks(size_t n, int nsys, const int64_t *off, const uint32_t *tree_scratch) {
    UpBlocks u;
    u.ntiles = (uint32_t)((n + kTileW - 1) / kTileW);
    u.woff = tree_scratch + (size_t)kLevels * u.ntiles;
    u.off = off;
    u.n = n;
    u.nsys = nsys;
    u.tiles = (u.ntiles + kUpBlocks - 1) / kUpBlocks;
    if (u.tiles < kUpMinSpan / kTileW) u.tiles = kUpMinSpan / kTileW;
    if (n <= kUpOne) u.tiles = kUpOne / kTileW;
    u.nb = (u.ntiles + u.tiles - 1) / u.tiles;
    if (!u.nb) u.nb = 1;
    return u;
}

// first cell of level L that starts in block b or later
__device__ __forceinline__ uint32_t up_first(const Cells &c, const UpBlocks &u, int L, uint32_t b) {
    const uint32_t c0 = c.lvl[L], c1 = c.lvl[L + 1];
    if (b == 0 || c0 == c1) return c0;
    if (b >= u.nb) return c1;
    if (L > 0)
        return min(max((uint32_t)u.nsys + u.woff[(size_t)(L - 1) * u.ntiles + (size_t)b * u.tiles], c0),
                   c1);
    const int64_t r = (int64_t)b * u.tiles * kTileW;
    int lo = 0, hi = u.nsys;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (u.off[mid] < r) lo = mid + 1; else hi = mid;
    }
    return (uint32_t)lo;
}

// what a level's step needs to know of a cell, loaded a level ahead (the steps are a serial chain of
// load latencies)
struct UpCell {
    uint32_t id, begin, first, count, nch;      // first: first child or first particle
};
__device__ __forceinline__ UpCell up_cell(const Cells &c, uint32_t k) {
    const uint2 lk = c.link[k];
    return {k, c.begin[k], lk.x, lk.y, c.node[k].w >> 8};
}

// the cells inside block blockIdx.x
template <class F>
__device__ __forceinline__ void up_inside(const Cells &c, const UpBlocks &u, F cell) {
    __shared__ uint32_t first[kLevels + 1], last[kLevels + 1];
    const uint32_t b = blockIdx.x;
    if (threadIdx.x <= kLevels) {
        first[threadIdx.x] = up_first(c, u, (int)threadIdx.x, b);
        last[threadIdx.x] = up_first(c, u, (int)threadIdx.x, b + 1);
    }
    __syncthreads();
    const uint64_t end = (uint64_t)(b + 1) * u.tiles * kTileW;
    int L = kLevels;
    while (L >= 0 && first[L] >= last[L]) L--;
    UpCell nxt{kNone, 0, 0, 0, 0};
    if (L >= 0 && first[L] + threadIdx.x < last[L]) nxt = up_cell(c, first[L] + threadIdx.x);
    while (L >= 0) {
        UpCell q = nxt;
        const uint32_t k1 = last[L];
        int M = L - 1;
        while (M >= 0 && first[M] >= last[M]) M--;
        nxt.id = kNone;
        if (M >= 0 && first[M] + threadIdx.x < last[M]) nxt = up_cell(c, first[M] + threadIdx.x);
        while (q.id != kNone) {
            if ((uint64_t)q.begin + q.count <= end) cell(q);
            const uint32_t k = q.id + kUpThreads;
            q.id = kNone;
            if (k < k1) q = up_cell(c, k);
        }
        __syncthreads();
        L = M;
    }
}

// Cells across the boundaries inside group blockIdx.x of `fan` blocks, within the group (fan <=
// kUpThreads; one group that holds all blocks: no cell is left out).
template <class F>
__device__ __forceinline__ void up_across(const Cells &c, const UpBlocks &u, uint32_t fan, F cell) {
    __shared__ uint32_t id[kLevels + 1][kUpThreads];
    __shared__ uint32_t any[kLevels + 1];
    if (threadIdx.x <= kLevels) any[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t span = (uint64_t)u.tiles * kTileW;
    const uint32_t g0 = blockIdx.x * fan, g1 = min(g0 + fan, u.nb);
    const uint64_t lo = g0 * span, hi = g1 < u.nb ? g1 * span : ~0ull;
    const uint32_t m = g1 - g0 - 1;              // boundaries g0 + 1 .. g1 - 1
#pragma unroll 4
    for (uint32_t i = threadIdx.x; i < m * (kLevels + 1); i += blockDim.x) {
        const uint32_t L = i / m, t = i - L * m, f = up_first(c, u, (int)L, g0 + t + 1);
        uint32_t k = kNone;
        if (f > c.lvl[L]) {
            const uint64_t r = (uint64_t)(g0 + t + 1) * span, b0 = c.begin[f - 1];
            const uint64_t e0 = b0 + c.count[f - 1];
            if (e0 > r && b0 + span >= r && b0 >= lo && e0 <= hi) k = f - 1;
        }
        id[L][t] = k;
        if (k != kNone) any[L] = 1;
    }
    __syncthreads();
    const bool mine = threadIdx.x < m;
    int L = kLevels;
    while (L >= 0 && !any[L]) L--;
    UpCell nxt{kNone, 0, 0, 0, 0};
    if (L >= 0 && mine && id[L][threadIdx.x] != kNone) nxt = up_cell(c, id[L][threadIdx.x]);
    while (L >= 0) {
        const UpCell q = nxt;
        int M = L - 1;
        while (M >= 0 && !any[M]) M--;
        nxt.id = kNone;
        if (M >= 0 && mine && id[M][threadIdx.x] != kNone) nxt = up_cell(c, id[M][threadIdx.x]);
        if (q.id != kNone) cell(q);
        __syncthreads();
        L = M;
    }
}

// the launches: inside(grid, threads, u), then across(grid, threads, u, fan) as often as needed.  Up
// to 2 kUpFan blocks one workgroup takes all boundaries.
template <class A, class B>
inline void up_launch(UpBlocks u, A inside, B across) {
    inside(u.nb, kUpThreads, u);
    if (u.nb > 2 * kUpFan) {
        const uint32_t ng = (u.nb + kUpFan - 1) / kUpFan;
        across(ng, 256, u, kUpFan);
        u.tiles *= kUpFan;
        u.nb = ng;
    }
    if (u.nb > 1) across(1, kUpThreads, u, (uint32_t)kUpThreads);
}

}  // namespace fdx
