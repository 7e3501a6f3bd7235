// CPU check of the far-field polynomial (far_field.h): random superparticles around a group, summed by
// FarAcc, folded and evaluated at random members, against the pair terms in FP64.  Prints for every
// kind the largest error over its bound, of the acceleration and of the potential.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "far_field.h"

using namespace fdx;

static std::mt19937_64 rng(5);
static double uni(double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); }
static void direction(double *d) {
    double n;
    do {
        for (int k = 0; k < 3; k++) d[k] = uni(-1, 1);
        n = std::sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    } while (n > 1 || n < 0.1);
    for (int k = 0; k < 3; k++) d[k] /= n;
}

// With h = radius / R and u = 2^-24: of 1 / |X - r| the degrees n >= 5 are omitted, each at most h^n / R,
// its gradient n h^(n-1) / R^2.  The quadrupole's field is sum Q_ij d_i d_j (1 / |X - r|) / 6: at most
// |Q|* (n + 2)(n + 1) h^n / (6 R^3), its gradient n times that over the radius, |Q|* the sum of its
// eigenvalues' sizes, here at most 3 |Q|.  1.1 for a softening of at most R / 20.  Rounding: the
// coordinates' and the formula's, 20 u of the leading terms.
struct Bound { double a, p; };
static Bound bound(double M, double q, double R, double rad) {
    const double h = rad / R, u = std::ldexp(1.0, -24), nuc = 3 * q;
    double a = 0, p = 0;
    for (int n = 5; n < 40; n++) {
        const double c = M / R + nuc * (n + 2) * (n + 1) / (6 * R * R * R);
        p += 1.1 * c * std::pow(h, n);
        a += 1.1 * c * n * std::pow(h, n - 1) / R;
    }
    a += 20 * u * (M / (R * R) + nuc / (R * R * R * R));
    p += 20 * u * (M / R + nuc / (2 * R * R * R));
    return {a, p};
}

template <bool QUAD>
static void run(const char *name, bool mass, double soft, int count) {
    double ra = 0, rp = 0;
    for (int trial = 0; trial < 400; trial++) {
        const double h = std::ldexp(1.0, (int)uni(-20, 4)), rad = uni(0.2, 0.85);   // rad in cells
        double e2 = 0, far = kFarRatio * rad;
        if (soft > 0) { e2 = soft * soft * far * far; }
        FarAcc acc;
        struct S { double X[3], M, Q[6], R; };
        std::vector<S> s(count);
        Bound b{0, 0};
        for (S &c : s) {
            double d[3];
            direction(d);
            const double R = far * std::exp(uni(0.0, 3.0));
            for (int k = 0; k < 3; k++) c.X[k] = d[k] * R * h;
            c.M = mass ? uni(0.1, 10) : 0.0;
            const double size = QUAD ? uni(0.0, 0.3) * R * R * h * h * 10 : 0.0;   // theta up to 1
            for (int k = 0; k < 6; k++) c.Q[k] = size * uni(-1, 1);
            const double tr = (c.Q[0] + c.Q[1] + c.Q[2]) / 3;
            for (int k = 0; k < 3; k++) c.Q[k] -= tr;
            const float x = (float)c.X[0] * (float)(1 / h), y = (float)c.X[1] * (float)(1 / h),
                        z = (float)c.X[2] * (float)(1 / h);
            float q[6];
            double qn = 0;
            for (int k = 0; k < 6; k++) {
                q[k] = (float)(c.Q[k] / (h * h));
                qn += (k < 3 ? 1 : 2) * (c.Q[k] / (h * h)) * (c.Q[k] / (h * h));
            }
            const float i = 1.0f / sqrtf(x * x + y * y + z * z + (float)e2);
            acc.add<QUAD>(x, y, z, i, (float)c.M, q);
            const Bound o = bound(c.M, std::sqrt(qn), std::sqrt(R * R + e2), rad);
            b.a += o.a;
            b.p += o.p;
        }
        acc.fold();
        FarCoef c;
        c.c0 = acc.c0;
        for (int k = 0; k < 3; k++) c.c1[k] = acc.c1[k];
        for (int k = 0; k < 6; k++) c.c2[k] = acc.c2[k];
        for (int k = 0; k < 10; k++) c.c3[k] = acc.c3[k];
        for (int k = 0; k < 15; k++) c.c4[k] = acc.c4[k];
        for (int m = 0; m < 20; m++) {
            double d[3], r[3];
            direction(d);
            const double len = m < 10 ? rad : uni(0, rad);
            for (int k = 0; k < 3; k++) r[k] = d[k] * len;
            double a[4] = {0, 0, 0, 0}, e[4] = {0, 0, 0, 0};
            far_eval(c, 1 / h, (float)r[0], (float)r[1], (float)r[2], a[0], a[1], a[2], a[3]);
            for (const S &p : s) {
                const double x[3] = {(float)r[0] * h - p.X[0], (float)r[1] * h - p.X[1],
                                     (float)r[2] * h - p.X[2]};
                const double R2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + e2 * h * h;
                const double R = std::sqrt(R2), R5 = R2 * R2 * R;
                const double Qx[3] = {p.Q[0] * x[0] + p.Q[3] * x[1] + p.Q[4] * x[2],
                                      p.Q[3] * x[0] + p.Q[1] * x[1] + p.Q[5] * x[2],
                                      p.Q[4] * x[0] + p.Q[5] * x[1] + p.Q[2] * x[2]};
                const double xQx = x[0] * Qx[0] + x[1] * Qx[1] + x[2] * Qx[2];
                for (int k = 0; k < 3; k++)
                    e[k] += -p.M * x[k] / (R2 * R) + Qx[k] / R5 - 2.5 * xQx * x[k] / (R5 * R2);
                e[3] -= p.M / R + 0.5 * xQx / R5;
            }
            double da = 0;
            for (int k = 0; k < 3; k++) da += (a[k] - e[k]) * (a[k] - e[k]);
            ra = std::fmax(ra, std::sqrt(da) * h * h / b.a);
            rp = std::fmax(rp, std::fabs(a[3] - e[3]) * h / b.p);
        }
    }
    std::printf("%s %.4f %.4f\n", name, ra, rp);
}

int main() {
    run<false>("mono", true, 0, 1);
    run<false>("mono_soft", true, 0.05, 1);
    run<false>("mono_many", true, 0.01, 50);
    run<true>("quad_only", false, 0, 1);
    run<true>("quad", true, 0, 1);
    run<true>("quad_soft", true, 0.05, 1);
    run<true>("quad_many", true, 0.01, 50);
    return 0;
}
