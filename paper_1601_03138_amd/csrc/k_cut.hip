// Tree part of TreePM: monopole forces with the S2 cutoff over the shared group lists.
//
// The Newtonian pair force times g(xi), xi = 2 r / r_cut, the complement of the force between two
// S2 clouds of diameter r_cut (Hockney & Eastwood); r unsoftened, softening in the Newtonian
// factor only, no potential.  Particles and superparticles (monopole at the centre of mass) have
// the same pair term, so both lists run through one loop.
//
// One workgroup evaluates one group, or some of its passes: entries are staged 256 at a time in LDS, every wave sifts
// the tile for its run of members (sift.h) and evaluates what it kept.  A dropped entry lies
// beyond r_cut of every member of the run, where g = 0.  VALU bound.  2^24 uniform particles,
// r_cut three mesh widths, groups of 64 (976 entries per member, 113 particles within the
// cutoff), FP32 persistent launch: 15.6 -> 8.5 ms; before, every entry met every member, |r| took a
// second reciprocal square root and g was two polynomials that cancel towards the cutoff (FP32: off
// by up to 6.6e-6; now 3e-7).
//
// FP32: positions relative to the centre of the group's cell; each tile's sum is added to a
// compensated accumulator.  FP64: the same in FP64.
#include "dev_util.h"
#include "fdx_internal.h"
#include "group_queue.h"
#include "interact.h"
#include "sift.h"

namespace fdx {

namespace {

constexpr int kTileC = kSiftThreads;

struct CutArgs {
    const uint32_t *gbegin, *gcount;
    const double *gcentre;
    const double4 *jp;
    const double *seps;
    const double *mom;
    const uint64_t *seg;
    const uint32_t *cap, *cnt_e, *cnt_s, *list, *order, *bounds, *ngroups;
    double4 *fs;
    DevStatus *st;
    uint32_t G;
    GroupItems items;         // direct launch
    double r_cut;
};

// g(xi), defined by one polynomial up to 1 and one from 1 to 2, without a branch.  The outer one is
// (2 - xi)^5 (4 + 10 xi + 22 xi^2 + 7 xi^3) / 140, the inner one that plus
// (1 - xi)^6 (12 + 72 xi + 28 xi^2) / 140: sums of positive terms, so every digit of g holds up
// to the cutoff, and 0 from there on.
template <class T>
__device__ __forceinline__ T s2_cutoff(T xi) {
    xi = min(xi, (T)2);
    const T u = (T)2 - xi, u2 = u * u, u5 = u2 * u2 * u;
    const T s = max((T)1 - xi, (T)0), s2 = s * s, s6 = s2 * s2 * s2;
    T p = fma(xi, (T)0.05, (T)(22.0 / 140.0));
    p = fma(xi, p, (T)(10.0 / 140.0));
    p = fma(xi, p, (T)(4.0 / 140.0));
    const T t = fma(xi, fma(xi, (T)0.2, (T)(72.0 / 140.0)), (T)(12.0 / 140.0));
    return fma(s6, t, u5 * p);
}
__device__ __forceinline__ float cut_dist(float r2) { return __builtin_amdgcn_sqrtf(r2); }
// (coincident points get 1e-145.)  10^6 uniform particles, n_group 256, FP64, cutoff of 3 spacings: 2.28 ms
// with the general sqrt, 2.05 with this one.
__device__ __forceinline__ double cut_dist(double r2) { return sqrt_pos(r2 + 1e-290); }

template <class T>
struct CutSmem {
    using V = typename V4<T>::t;
    V tile[kTileC];
    union {
        V kept[kSiftWaves][kTileC];
        double red[kSiftThreads][3];
    };
    uint32_t slot;
};

template <class T>
__device__ __forceinline__ void cut_group(const CutArgs &a, uint32_t gi, uint32_t part, uint32_t parts,
                                          CutSmem<T> &sm) {
    using V = typename V4<T>::t;
    const uint32_t tid = threadIdx.x, lane = (uint32_t)lane_id();
    const int w = (int)(tid / kWave);
    const uint64_t lt = lanemask_lt();
    gi = uniform_u32(gi);
    const uint32_t gb = uniform_u32(a.gbegin[gi]), ni = uniform_u32(a.gcount[gi]);
    const uint32_t ne = uniform_u32(a.cnt_e[gi]), ns = uniform_u32(a.cnt_s[gi]);
    const uint32_t *epj = a.list + uniform_u64(a.seg[gi]);
    const uint32_t *spj = epj + uniform_u32(a.cap[gi]) - ns;
    const bool fp32 = sizeof(T) == 4;
    const double cx = fp32 ? uniform_f64(a.gcentre[3 * gi]) : 0.0;
    const double cy = fp32 ? uniform_f64(a.gcentre[3 * gi + 1]) : 0.0;
    const double cz = fp32 ? uniform_f64(a.gcentre[3 * gi + 2]) : 0.0;
    const T cut_s = (T)(2.0 / a.r_cut);
    const T reach2 = (T)a.r_cut * (T)a.r_cut * kSiftMargin<T>;
    const uint32_t nl = ne + ns;
    // entry k of the two lists: particles, then superparticles
    auto entry = [&](uint32_t k) {
        if (k < ne) return a.jp[epj[k]];
        const double *o = a.mom + 10 * (size_t)spj[k - ne];
        return make_double4(o[1], o[2], o[3], o[0]);
    };
    for (uint32_t pass = part; pass < sift_passes(ni); pass += parts) {
        const SiftMap m(ni, pass);
        const uint32_t r = gb + m.first + (m.active ? m.member : 0u);
        const double4 p = a.jp[r];
        const T xi = (T)(p.x - cx), yi = (T)(p.y - cy), zi = (T)(p.z - cz);
        const double e = a.seps[r];
        const T e2 = (T)(e * e);
        T bc[3], bh[3];
        sift_box<T>(xi, m.active, bc[0], bh[0]);
        sift_box<T>(yi, m.active, bc[1], bh[1]);
        sift_box<T>(zi, m.active, bc[2], bh[2]);
        Acc<T> ax, ay, az;
        const uint32_t share = kTileC / m.parts;
        double4 nxt = make_double4(0, 0, 0, 0);
        if (tid < nl) nxt = entry(tid);
        for (uint32_t t0 = 0; t0 < nl; t0 += kTileC) {
            const uint32_t nt = min((uint32_t)kTileC, nl - t0);
            __syncthreads();
            V v;
            v.x = (T)(nxt.x - cx); v.y = (T)(nxt.y - cy); v.z = (T)(nxt.z - cz); v.w = (T)nxt.w;
            sm.tile[tid] = v;
            __syncthreads();
            if (t0 + kTileC + tid < nl) nxt = entry(t0 + kTileC + tid);
            uint32_t cnt = 0;
            const uint32_t lo = m.part * share, hi = min(nt, lo + share);
            for (uint32_t q = lo; q < hi; q += kWave) {
                const uint32_t k = q + lane;
                const V J = sm.tile[k & (kTileC - 1)];
                const bool keep = k < hi && sift_dist2<T>(J.x, J.y, J.z, bc, bh) <= reach2;
                const uint64_t b = __ballot(keep);
                if (keep) sm.kept[w][cnt + (uint32_t)__popcll(b & lt)] = J;
                cnt += (uint32_t)__popcll(b);
            }
            wave_barrier();
            if (m.active) {
                T tx = 0, ty = 0, tz = 0;
#pragma unroll 4
                for (uint32_t k = m.slot; k < cnt; k += m.js) {
                    const V J = sm.kept[w][k];
                    const T dx = J.x - xi, dy = J.y - yi, dz = J.z - zi;
                    const T r2u = fma(dz, dz, fma(dy, dy, dx * dx));
                    const T ri = rsqrt_t(r2u + e2);
                    const T f = J.w * ri * (ri * ri) * s2_cutoff<T>(cut_dist(r2u) * cut_s);
                    tx = fma(f, dx, tx);
                    ty = fma(f, dy, ty);
                    tz = fma(f, dz, tz);
                }
                ax.add(tx); ay.add(ty); az.add(tz);
            }
        }
        __syncthreads();
        sm.red[tid][0] = ax.val(); sm.red[tid][1] = ay.val(); sm.red[tid][2] = az.val();
        __syncthreads();
        // one thread per (member, component) sums parts, then slots, in order
        for (uint32_t t = tid; t < 4u * m.n; t += kSiftThreads) {
            const uint32_t c = t & 3u, i = t >> 2;
            double s = 0;
            if (c < 3u)
                for (uint32_t q = 0; q < m.parts; q++)
                    for (uint32_t k = 0; k < m.js; k++) s += sm.red[m.thread_of(i, q, k)][c];
            reinterpret_cast<double *>(a.fs + gb + m.first + i)[c] = s;
        }
        __syncthreads();
    }
}

template <class T>
__global__ void __launch_bounds__(kSiftThreads) k_cut_direct(CutArgs a) {
    __shared__ CutSmem<T> sm;
    // XCD-aware order, as the Newtonian kernels'
    const uint32_t item = xcd_run_block(blockIdx.x, a.items.run);
    const uint32_t part = item / a.G, q = item - part * a.G;
    if (part >= a.items.parts) return;
    cut_group<T>(a, a.order ? a.order[q] : q, part, a.items.parts, sm);
}

template <class T>
__global__ void __launch_bounds__(kSiftThreads) k_cut_persistent(CutArgs a) {
    __shared__ CutSmem<T> sm;
    const uint32_t G = *a.ngroups;
    for (bool first = true;; first = false) {
        if (threadIdx.x < kWave) {
            const uint32_t k = pop_group<1>(a.st, G, a.bounds, a.order != nullptr, first, 0);
            if (threadIdx.x == 0) sm.slot = k;
        }
        __syncthreads();
        const uint32_t slot = sm.slot;
        __syncthreads();
        if (slot >= G) break;
        cut_group<T>(a, a.order ? a.order[slot] : slot, 0, 1, sm);
    }
}

template <class T>
hipError_t launch(const CutArgs &a, bool persistent, hipStream_t s) {
    if (!persistent) {
        if (!a.G) return hipSuccess;
        hipLaunchKernelGGL(k_cut_direct<T>, dim3(a.items.blocks), dim3(kSiftThreads), 0, s, a);
        return hipGetLastError();
    }
    int dev = 0, ncu = 256, per_cu = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, reinterpret_cast<const void *>(k_cut_persistent<T>), kSiftThreads, 0);
    size_t grid = (size_t)ncu * (per_cu < 1 ? 1 : per_cu);
    if (a.G && grid > a.G) grid = a.G;
    hipLaunchKernelGGL(k_cut_persistent<T>, dim3((unsigned)grid), dim3(kSiftThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t cut_force(size_t G, const ForceArgs &fa, hipStream_t s) {
    CutArgs a;
    a.gbegin = fa.g->begin; a.gcount = fa.g->count; a.gcentre = fa.g->centre;
    a.jp = fa.jp; a.seps = fa.seps; a.mom = fa.mom;
    a.seg = fa.seg; a.cap = fa.cap; a.cnt_e = fa.cnt_e; a.cnt_s = fa.cnt_s; a.list = fa.list;
    a.order = fa.order; a.bounds = fa.bounds;
    a.ngroups = fa.count ? fa.count : &fa.st->n_groups_c;
    a.fs = fa.fs; a.st = fa.st; a.G = (uint32_t)G; a.r_cut = fa.r_cut;
    a.items = cut_items(G, fa.n_group);   // runs of 64 blocks per XCD, 2^23 uniform: 3.30 ms, of 16 3.41
    // Few groups of many passes are left to the direct launch, which splits them, unless they are a list
    // of unknown length: 3e5 particles, n_group 512, FP32: 1.46 ms persistent, 0.89 direct.  With two
    // parts the queues' balance is worth more (10^6, n_group 256, FP64: 6.16 and 6.53).
    const bool persistent = fa.persistent && (fa.order || a.items.parts <= 2);
    return fa.fp32 ? launch<float>(a, persistent, s) : launch<double>(a, persistent, s);
}

}  // namespace fdx
