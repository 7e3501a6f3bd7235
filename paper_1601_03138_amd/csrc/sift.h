// Short-range pair loops over a group's list (TreePM cutoff force, SPH density): sifting.
//
// A group's list holds whatever reaches any of its members, so for a single member most entries
// lie beyond the cutoff.  The members are sorted along the space-filling curve, so runs of
// 5..20 of them fill small boxes: a wave keeps the entries within reach of its run's box, and only
// those meet the run's members.  Uniform particles, 64 members, runs of 16: cutoff of three
// spacings 460 of 976 entries are kept, of 4.2 spacings 900 of 1540.
#pragma once

#include "dev_util.h"

namespace fdx {

constexpr int kSiftThreads = 256;
constexpr int kSiftWaves = kSiftThreads / kWave;

// Mapping of a workgroup of four waves (TreePM): every wave has one run, or, in small groups, a
// run and a part of the entries.  Members [first, first + n) of a group in this pass, cut into
// nsub runs of bs; wave w takes run sub and the part-th of `parts` shares of every tile.  Its lanes
// are js slots of bs members: slot s meets the kept entries s, s + js, ...
struct SiftMap {
    uint32_t first, n, nsub, parts, bs, js, sub, part, slot, member;
    bool active;                          // this lane holds a member
    __device__ __forceinline__ SiftMap(uint32_t ni, uint32_t pass) {
        const uint32_t np = (ni + kSiftPass - 1) / kSiftPass, per = (ni + np - 1) / np;
        first = pass * per;
        n = first < ni ? min(per, ni - first) : 0u;
        nsub = n <= 16 ? 1u : (n <= 32 ? 2u : 4u);
        parts = kSiftWaves / nsub;
        bs = max((n + nsub - 1) / nsub, 1u);
        js = kWave / bs;
        const uint32_t w = uniform_u32(threadIdx.x / kWave), lane = (uint32_t)lane_id();
        sub = w % nsub;
        part = w / nsub;
        slot = lane / bs;
        member = sub * bs + lane % bs;
        active = slot < js && member < n;
    }
    // thread holding the partial sum of member i of the pass from part p, slot s
    __device__ __forceinline__ uint32_t thread_of(uint32_t i, uint32_t p, uint32_t s) const {
        return (p * nsub + i / bs) * kWave + s * bs + i % bs;
    }
};

// sqrt for x >= 1e-290, correctly rounded (no exception in 1.7e7 arguments over 570 decades): the hardware reciprocal square
// root y refined once as the root g, then the residual x - g^2 of the root.  The general sqrt
// spends as many instructions again on ranges that cannot occur here.
__device__ __forceinline__ double sqrt_pos(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y;
    const double h = 0.5 * y;
    g = fma(g, fma(-h, g, 0.5), g);
    return fma(fma(-g, g, x), h, g);
}

// centre and half-width of the box of the active lanes' points along one axis
template <class T>
__device__ __forceinline__ void sift_box(T v, bool active, T &centre, T &half) {
    T lo = active ? v : (T)INFINITY, hi = active ? v : (T)-INFINITY;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        lo = min(lo, __shfl_xor(lo, d, kWave));
        hi = max(hi, __shfl_xor(hi, d, kWave));
    }
    centre = (T)0.5 * (lo + hi);
    // a little more than half, so that rounding cannot leave a member outside
    half = max(hi - centre, centre - lo) * (T)(1.0 + (sizeof(T) == 4 ? 1e-6 : 1e-14));
}

// squared distance of a point from the box (0 inside)
template <class T>
__device__ __forceinline__ T sift_dist2(T x, T y, T z, const T (&c)[3], const T (&h)[3]) {
    const T dx = max((T)fabs(x - c[0]) - h[0], (T)0);
    const T dy = max((T)fabs(y - c[1]) - h[1], (T)0);
    const T dz = max((T)fabs(z - c[2]) - h[2], (T)0);
    return fma(dz, dz, fma(dy, dy, dx * dx));
}

// factor on the squared reach that covers the rounding of the test
template <class T> constexpr T kSiftMargin = (T)(1.0 + (sizeof(T) == 4 ? 1e-5 : 1e-12));

}  // namespace fdx
