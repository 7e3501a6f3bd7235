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
// A superparticle is far when |X| > kFarRatio x the radius of the group's box, whatever its mass:
// of the omitted terms the largest is 5 (radius / |X|)^4 = 3e-7 of the superparticle's own monopole
// force at the corner of the box, where the pair loop errs by up to 7e-7 on a single pair
// (roundings of 2^-24 of coordinates and formula), and less than a third of the pair loop's rms over
// the box.  So no single mass and no number of masses in one direction can make the expansion
// the larger error.  (A ratio of 24 leaves 1.5e-5, which only averages out where many directions
// contribute.)  Error of the FP32 path against the FP64 kernels on the same lists, rms and
// 99.9 % quantile of |da| / |a| over the members of groups that a ratio of 24 expands, for every pair
// evaluated / ratio 24 / ratio 64 (n_group 256, theta 0.5 unless said):
//   2^20 Plummer                          1.33e-7 6.0e-7 / 1.24e-7 5.4e-7 / 1.27e-7 5.7e-7
//   2^23 clustered                        1.77e-7 1.3e-6 / 1.69e-7 1.2e-6 / 1.71e-7 1.2e-6
//   3e6 clustered, n_group 128, theta 0.6 1.23e-7 7.7e-7 / 1.22e-7 7.7e-7 / 1.16e-7 7.3e-7
//   disc of 1.2e7 around 1000 x its mass  1.85e-7 5.5e-7 / 1.53e-6 8.4e-6 / 1.85e-7 5.5e-7
//   8e6 beside 3e4 of 1000 x their mass   1.63e-7 8.8e-7 / 1.49e-7 1.1e-6 / 5.4e-8 3.9e-7
//   2e6 beside 3e4 of 100 x, monopole     2.73e-7 1.4e-6 / 2.85e-7 1.7e-6 / 2.55e-7 1.4e-6
// The second to fourth degree are plain FP32 sums: beyond 64 radii they carry about 1/30 of an
// entry's force, so their rounding stays below the pair loop's.  At 64 about 0.30 of the 2^24
// clustered workload's superparticle interactions are far.
//
// Coordinates are scaled by the side of the group's cell (a power of two times the root side, so
// the scaling is exact): high powers of R neither overflow nor underflow where they matter.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace fdx {

constexpr float kFarRatio = 64.0f;
// No expansion unless the root cell is this many times wider than the far distance: in a shallower
// tree few superparticles are far, and sifting the lists costs more than they save.  Force and
// expansion with 4 / 8 / 12 / 32: 2^20 Plummer 2.46 / 2.41 / 2.50 / 2.52 ms (2.53 without), 3e6
// clustered, n_group 128, 4.83 / 4.85 / 4.85 / 4.94 ms (4.98), 2^24 clustered 36.8 / 36.7 / 37.0 /
// 37.7 ms (43.0).
constexpr float kFarSpan = 8.0f;
// Smallest n_group whose groups are expanded: with few members a pass over the list costs as much as
// the pairs it saves.  n_group 32: 8e6 clustered 26.2 ms with it, 24.9 without; 64: 14.2 and 14.0, 2^20
// Plummer 2.30 and 2.09; 100: 8e6 clustered 18.9 and 19.8.  Monopole pairs cost less than half as
// much: 64: 2e6 Plummer 2.74 and 2.56; 128: 8e6 clustered 11.29 and 11.10; 512: 3e6 2.27 and 2.30.
constexpr int kFarMinGroup = 65, kFarMinGroupMono = 129;
// Systems of up to this many particles are not expanded (each by its own size, whatever else is in the
// batch): their trees are shallow, and the expansion is a launch of serial chains.  Force + expansion,
// n_group 256, without / with it, Plummer and clustered: 10^5 particles 0.43 / 0.46 and 0.41 / 0.40 ms,
// 131072 0.49 / 0.51 and 0.48 / 0.47, 2 10^5 0.59 / 0.61 and 0.62 / 0.58, 5 10^5 1.25 / 1.21 and
// 1.36 / 1.20; 40000, n_group 512, 0.41 / 0.47 and 0.56 / 0.55.
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

// Accumulators: c[m][k] as coefficients of the monomials of r; s^k kept apart
// (k = 1: t01, t11, t21; k = 2: t02) and multiplied out after the sum
struct FarAcc {
    double c0 = 0, c1[3] = {0, 0, 0};
    float c2[6] = {}, c3[10] = {}, c4[15] = {};
    float t01 = 0, t11[3] = {}, t21[6] = {}, t02 = 0;

    template <bool QUAD>
    // a superparticle at (x, y, z), i = 1 / R
    __host__ __device__ inline void add(float x, float y, float z, float i, float M,
                                        const float (&q)[6]) {
        const float i2 = i * i;
        const float zx = x * i2, zy = y * i2, zz = z * i2;
        const float b = M * i;
        // quadrupole: A = X.Q.X / (2 R^5), v = Q X / R^5, h = coefficients of r.Q.r / (2 R^5)
        float A = 0, vx = 0, vy = 0, vz = 0, h[6] = {0, 0, 0, 0, 0, 0};
        if (QUAD) {
            const float i5 = i * i2 * i2;
            vx = i5 * fmaf(q[0], x, fmaf(q[3], y, q[4] * z));
            vy = i5 * fmaf(q[3], x, fmaf(q[1], y, q[5] * z));
            vz = i5 * fmaf(q[4], x, fmaf(q[5], y, q[2] * z));
            A = 0.5f * fmaf(x, vx, fmaf(y, vy, z * vz));
            const float i5h = 0.5f * i5;
            h[0] = i5h * q[0]; h[1] = i5h * q[1]; h[2] = i5h * q[2];
            h[3] = i5 * q[3]; h[4] = i5 * q[4]; h[5] = i5 * q[5];
        }
        c0 += (double)(b + A);
        const float w1 = fmaf(5.f, A, b);
        c1[0] += (double)fmaf(w1, zx, -vx);
        c1[1] += (double)fmaf(w1, zy, -vy);
        c1[2] += (double)fmaf(w1, zz, -vz);
        // (z.r) (p.r) + d h(r): a quadratic form, added to o or returned in it
        auto form = [&](float w, float u, float d, float (&o)[6], bool acc) {
            const float px = fmaf(w, zx, u * vx), py = fmaf(w, zy, u * vy), pz = fmaf(w, zz, u * vz);
            if (!QUAD) {
                o[0] = fmaf(zx, px, acc ? o[0] : 0.f);
                o[1] = fmaf(zy, py, acc ? o[1] : 0.f);
                o[2] = fmaf(zz, pz, acc ? o[2] : 0.f);
                o[3] = fmaf(zx, 2.f * py, acc ? o[3] : 0.f);
                o[4] = fmaf(zx, 2.f * pz, acc ? o[4] : 0.f);
                o[5] = fmaf(zy, 2.f * pz, acc ? o[5] : 0.f);
                return;
            }
            o[0] = fmaf(zx, px, acc ? fmaf(d, h[0], o[0]) : d * h[0]);
            o[1] = fmaf(zy, py, acc ? fmaf(d, h[1], o[1]) : d * h[1]);
            o[2] = fmaf(zz, pz, acc ? fmaf(d, h[2], o[2]) : d * h[2]);
            o[3] = fmaf(zx, py, fmaf(zy, px, acc ? fmaf(d, h[3], o[3]) : d * h[3]));
            o[4] = fmaf(zx, pz, fmaf(zz, px, acc ? fmaf(d, h[4], o[4]) : d * h[4]));
            o[5] = fmaf(zy, pz, fmaf(zz, py, acc ? fmaf(d, h[5], o[5]) : d * h[5]));
        };
        form(fmaf(17.5f, A, 1.5f * b), -5.f, 1.f, c2, true);
        t01 = fmaf(fmaf(-2.5f, A, -0.5f * b), i2, t01);
        // third degree: (z.r) x a quadratic form
        float n[6];
        form(fmaf(52.5f, A, 2.5f * b), -17.5f, 5.f, n, false);
        c3[0] = fmaf(zx, n[0], c3[0]);
        c3[1] = fmaf(zx, n[3], fmaf(zy, n[0], c3[1]));
        c3[2] = fmaf(zx, n[4], fmaf(zz, n[0], c3[2]));
        c3[3] = fmaf(zx, n[1], fmaf(zy, n[3], c3[3]));
        c3[4] = fmaf(zx, n[5], fmaf(zy, n[4], fmaf(zz, n[3], c3[4])));
        c3[5] = fmaf(zx, n[2], fmaf(zz, n[4], c3[5]));
        c3[6] = fmaf(zy, n[1], c3[6]);
        c3[7] = fmaf(zy, n[5], fmaf(zz, n[1], c3[7]));
        c3[8] = fmaf(zy, n[2], fmaf(zz, n[5], c3[8]));
        c3[9] = fmaf(zz, n[2], c3[9]);
        const float w11 = fmaf(-17.5f, A, -1.5f * b);
        t11[0] = fmaf(i2, fmaf(w11, zx, 2.5f * vx), t11[0]);
        t11[1] = fmaf(i2, fmaf(w11, zy, 2.5f * vy), t11[1]);
        t11[2] = fmaf(i2, fmaf(w11, zz, 2.5f * vz), t11[2]);
        // fourth degree: (z.r)^2 x a quadratic form, by way of the cubic (z.r) x the form
        form(fmaf(144.375f, A, 4.375f * b), -52.5f, 17.5f, n, false);
        float k[10];
        k[0] = zx * n[0];
        k[1] = fmaf(zx, n[3], zy * n[0]);
        k[2] = fmaf(zx, n[4], zz * n[0]);
        k[3] = fmaf(zx, n[1], zy * n[3]);
        k[4] = fmaf(zx, n[5], fmaf(zy, n[4], zz * n[3]));
        k[5] = fmaf(zx, n[2], zz * n[4]);
        k[6] = zy * n[1];
        k[7] = fmaf(zy, n[5], zz * n[1]);
        k[8] = fmaf(zy, n[2], zz * n[5]);
        k[9] = zz * n[2];
        c4[0] = fmaf(zx, k[0], c4[0]);
        c4[1] = fmaf(zx, k[1], fmaf(zy, k[0], c4[1]));
        c4[2] = fmaf(zx, k[2], fmaf(zz, k[0], c4[2]));
        c4[3] = fmaf(zx, k[3], fmaf(zy, k[1], c4[3]));
        c4[4] = fmaf(zx, k[4], fmaf(zy, k[2], fmaf(zz, k[1], c4[4])));
        c4[5] = fmaf(zx, k[5], fmaf(zz, k[2], c4[5]));
        c4[6] = fmaf(zx, k[6], fmaf(zy, k[3], c4[6]));
        c4[7] = fmaf(zx, k[7], fmaf(zy, k[4], fmaf(zz, k[3], c4[7])));
        c4[8] = fmaf(zx, k[8], fmaf(zy, k[5], fmaf(zz, k[4], c4[8])));
        c4[9] = fmaf(zx, k[9], fmaf(zz, k[5], c4[9]));
        c4[10] = fmaf(zy, k[6], c4[10]);
        c4[11] = fmaf(zy, k[7], fmaf(zz, k[6], c4[11]));
        c4[12] = fmaf(zy, k[8], fmaf(zz, k[7], c4[12]));
        c4[13] = fmaf(zy, k[9], fmaf(zz, k[8], c4[13]));
        c4[14] = fmaf(zz, k[9], c4[14]);
        form(fmaf(-78.75f, A, -3.75f * b), 17.5f, -2.5f, n, false);
        for (int u = 0; u < 6; u++) t21[u] = fmaf(i2, n[u], t21[u]);
        t02 = fmaf(fmaf(4.375f, A, 0.375f * b), i2 * i2, t02);
    }

    // multiply the powers of r^2 out into the monomials
    __host__ __device__ inline void fold() {
        for (int u = 0; u < 3; u++) c2[u] += t01;
        c3[0] += t11[0]; c3[3] += t11[0]; c3[5] += t11[0];
        c3[1] += t11[1]; c3[6] += t11[1]; c3[8] += t11[1];
        c3[2] += t11[2]; c3[7] += t11[2]; c3[9] += t11[2];
        c4[0] += t21[0] + t02; c4[10] += t21[1] + t02; c4[14] += t21[2] + t02;
        c4[3] += t21[0] + t21[1] + 2.f * t02;
        c4[5] += t21[0] + t21[2] + 2.f * t02;
        c4[12] += t21[1] + t21[2] + 2.f * t02;
        c4[1] += t21[3]; c4[6] += t21[3]; c4[8] += t21[3];
        c4[2] += t21[4]; c4[7] += t21[4]; c4[9] += t21[4];
        c4[4] += t21[5]; c4[11] += t21[5]; c4[13] += t21[5];
    }
};

// Whether a group's far superparticles are expanded: the expansion costs a fixed amount per
// group (wave reductions, a second pass over the list) and about as much per far superparticle
// as evaluating seven members, so it needs enough listed pairs, of which 0.1 to 0.3 are far, to
// save.  Force + expansion at a bound of 20000 / 40000 / 80000 / 160000 pairs: 3e6 clustered,
// n_group 128, 4.79 / 4.85 / 4.90 / 4.96 ms (4.98 without), 10^6 clustered 2.90 / 2.93 / 3.01 / 3.06
// (3.42), 2^24 clustered 36.7 / 36.7 / 36.8 / 37.7 ms (43.0).  Members, at least: 16 / 32 / 48 / 64 / 96:
// 2^24 clustered 35.9 / 36.1 / 36.8 / 37.5 / 38.7 ms.  A monopole pair costs less than half as much.
template <bool QUAD>
__device__ __forceinline__ bool far_worth(float thr2, uint32_t ni, uint32_t ns) {
    constexpr uint32_t min_ni = QUAD ? 16 : 64;
    constexpr uint32_t min_pairs = QUAD ? 40000 : 80000;
    return thr2 >= 0.0f && ni >= min_ni && (uint64_t)ni * ns >= min_pairs;
}

// field of the summed polynomial at a member (x, y, z scaled offset from the centre): adds to
// the acceleration and the potential
__host__ __device__ inline void far_eval(const FarCoef &c, double inv_h, float x, float y,
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
