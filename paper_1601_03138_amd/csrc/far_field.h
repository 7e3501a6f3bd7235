// Far superparticles of a group, FP32 group-relative evaluation.
//
// A superparticle much farther from a group than the group is wide exerts a field that varies
// little over the group, so the fields of all of them are summed once per group as one
// polynomial about the centre e of the group's box and the polynomial is evaluated at every
// member, instead of evaluating every (member, superparticle) pair.  The expanded function is the
// pair term itself (interact.h), softening and quadrupole included: with X the superparticle's
// centre of mass and r the member's position, both relative to e, eps the group's one softening,
// R^2 = |X|^2 + eps^2, z = X / R^2, s = r^2 / R^2,
//   (|X - r|^2 + eps^2)^(-L) = R^(-2L) sum_{m,k} c^L_{m,k} (z.r)^m s^k,
//   c^L_{m,k} = (L)_{m+k} 2^m (-1)^k / (m! k!)        (L = 1/2 and 5/2; (L)_n rising factorial),
//   (X - r).Q.(X - r) = X.Q.X - 2 (Q X).r + r.Q.r,
// kept to total degree 4 in r for the potential (3 for the acceleration).  No harmonicity is
// assumed, so the softened kernel is expanded exactly.
//
// A superparticle is far when |X| > kFarRatio x the radius of the group's box.  Of the omitted
// terms the largest, relative to the superparticle's own force, is of order (radius / |X|)^4; the
// directions differ from cell to cell, so they add up slowly.  Error of the FP32 path against the
// FP64 kernels on the same lists, rms over the particles of |da| / |a| (every pair evaluated ->
// kFarRatio 20, 24, 28):
//   2^20 Plummer, n_group 256, theta 0.5     1.38e-7 -> 1.38e-7, 1.31e-7, 1.30e-7
//   3e6 clustered, n_group 128, theta 0.6    1.22e-7 -> 1.47e-7, 1.20e-7, 1.21e-7
//   2^23 clustered, n_group 256, theta 0.5   1.69e-7 -> 1.94e-7, 1.64e-7, 1.62e-7
// (potential 7.1e-8 -> 5.5e-8 on the last).  24 is the smallest that loses nothing: the far sums
// round less than the pair loop did, which makes up for the omitted terms.  At 24 about 0.4 of the
// 2^24 clustered workload's superparticle entries are far.
//
// Coordinates are scaled by the side of the group's cell (a power of two times the root side, so
// the scaling is exact): high powers of R neither overflow nor underflow where they matter.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace fdx {

constexpr float kFarRatio = 24.0f;
// No expansion unless the root cell is this many times wider than the far distance: in a shallower
// tree few superparticles are far, and sifting the lists costs more than they save.  Ensemble of
// 512 systems of 1024..65536 particles (force + expansion; 8.57 ms without): 12: 8.73 ms, 16: 8.65;
// 3e6 clustered (5.00 ms without): 12: 4.51, 16: 4.57, 24: 4.59.
constexpr float kFarSpan = 16.0f;

// Beyond kFar3Ratio the fourth degree is left out (it adds 1.4e-8 to the rms at 64); about 0.7 of
// the far entries of the 2^24 clustered workload, at less than half the instructions.  The table
// above with it: 1.33e-7, 1.22e-7, 1.66e-7.
constexpr float kFar3Ratio = 64.0f;
// Systems of up to this many particles are not expanded: their trees are too shallow to gain
// (512 systems of 1024..65536 particles: 13.0 -> 13.1 ms per step with it; one of 2^20: 4.05 -> 3.87).
constexpr int64_t kFarMaxDirect = 131072;

// Geometry of a group's expansion (written with the group's box).  thr2 < 0: no expansion (the
// members' softenings differ, or the group is evaluated in FP64).
struct FarGeom {
    double ex, ey, ez;      // centre of the box
    double inv_h;           // 1 / side of the group's cell
    float thr2;             // (kFarRatio x box radius)^2
    float e2;               // (eps / h)^2
};

// Summed polynomial of one group: Phi = c0 + c1.r + (2nd) + (3rd) + (4th degree), Phi = -phi h.
// The orders that carry most of the field are held in FP64.
struct FarCoef {
    double c0, c1[3];
    float c2[6];            // xx yy zz xy xz yz
    float c3[10];           // xxx xxy xxz xyy xyz xzz yyy yyz yzz zzz
    float c4[15];           // xxxx xxxy xxxz xxyy xxyz xxzz xyyy xyyz xyzz xzzz yyyy yyyz yyzz yzzz zzzz
};

// Whether a group's far superparticles are expanded: the expansion costs a fixed amount per
// group (wave reductions, a second pass over the list) and about as much per far superparticle
// as evaluating seven members, so it needs enough pairs to save.  Force + expansion at a bound of
// 40000 / 65536 / 90000 pairs: 3e6 clustered 4.58 / 4.74 / 4.85 ms (5.17 without), 2^24 clustered
// 33.9 / 33.9 / 34.1 ms (43.0 without); a monopole pair costs less than half as much, so twice the
// bound.
template <bool QUAD>
__device__ __forceinline__ bool far_worth(float thr2, uint32_t ni, uint32_t ns) {
    constexpr uint32_t min_ni = QUAD ? 16 : 32;
    constexpr uint32_t min_pairs = QUAD ? 40000 : 80000;
    return thr2 >= 0.0f && ni >= min_ni && (uint64_t)ni * ns >= min_pairs;
}

// field of the summed polynomial at a member (x, y, z scaled offset from the centre): adds to
// the acceleration and the potential
__device__ __forceinline__ void far_eval(const FarCoef &c, double inv_h, float x, float y,
                                         float z, double &ax, double &ay, double &az,
                                         double &ph) {
    const float xx = x * x, yy = y * y, zz = z * z, xy = x * y, xz = x * z, yz = y * z;
    // gradient by degree; a homogeneous part of degree m is (r . its gradient) / m
    const float g2x = 2.f * c.c2[0] * x + c.c2[3] * y + c.c2[4] * z;
    const float g2y = c.c2[3] * x + 2.f * c.c2[1] * y + c.c2[5] * z;
    const float g2z = c.c2[4] * x + c.c2[5] * y + 2.f * c.c2[2] * z;
    const float *t = c.c3;
    const float g3x = 3.f * t[0] * xx + 2.f * (t[1] * xy + t[2] * xz) + t[3] * yy + t[4] * yz + t[5] * zz;
    const float g3y = t[1] * xx + 2.f * (t[3] * xy + t[7] * yz) + t[4] * xz + 3.f * t[6] * yy + t[8] * zz;
    const float g3z = t[2] * xx + t[4] * xy + 2.f * (t[5] * xz + t[8] * yz) + t[7] * yy + 3.f * t[9] * zz;
    const float *q = c.c4;
    const float xxx = xx * x, yyy = yy * y, zzz = zz * z, xyz = xy * z;
    const float g4x = 4.f * q[0] * xxx + 3.f * (q[1] * xx * y + q[2] * xx * z) +
                      2.f * (q[3] * x * yy + q[4] * xyz + q[5] * x * zz) + q[6] * yyy +
                      q[7] * yy * z + q[8] * y * zz + q[9] * zzz;
    const float g4y = q[1] * xxx + 2.f * q[3] * xx * y + q[4] * xx * z + 3.f * q[6] * x * yy +
                      2.f * q[7] * xyz + q[8] * x * zz + 4.f * q[10] * yyy +
                      3.f * q[11] * yy * z + 2.f * q[12] * y * zz + q[13] * zzz;
    const float g4z = q[2] * xxx + q[4] * xx * y + 2.f * q[5] * xx * z + q[7] * x * yy +
                      2.f * q[8] * xyz + 3.f * q[9] * x * zz + q[11] * yyy +
                      2.f * q[12] * yy * z + 3.f * q[13] * y * zz + 4.f * q[14] * zzz;
    const double k = inv_h * inv_h;
    ax += k * (c.c1[0] + (double)(g2x + (g3x + g4x)));
    ay += k * (c.c1[1] + (double)(g2y + (g3y + g4y)));
    az += k * (c.c1[2] + (double)(g2z + (g3z + g4z)));
    const float hx = 0.5f * g2x + ((1.f / 3.f) * g3x + 0.25f * g4x);
    const float hy = 0.5f * g2y + ((1.f / 3.f) * g3y + 0.25f * g4y);
    const float hz = 0.5f * g2z + ((1.f / 3.f) * g3z + 0.25f * g4z);
    ph -= inv_h * (c.c0 + ((double)x * (c.c1[0] + hx) + (double)y * (c.c1[1] + hy) +
                           (double)z * (c.c1[2] + hz)));
}

}  // namespace fdx
