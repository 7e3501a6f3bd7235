// Short-range interaction on the tree: SPH density from candidate neighbour lists.
//
// The same tree is traversed for short-range interactions with four kinds of cutoff
// (section "Interaction calculation"): fixed, j-dependent ("scatter", r < h_j), i-dependent
// ("gather", r < h_i) and symmetric (r < max(h_i, h_j)).  The walk (k_walk.hip) gives each
// group the particles of every leaf within reach; this file gives the walk its radii (the
// largest h of every cell, bottom-up, and of every group) and evaluates, per i-particle,
//   rho_i = sum_j m_j W(|r_ij|, H) over pairs with |r_ij| < H (j = i included),
//   H = r_cut (fixed), h_j (scatter), h_i (gather); symmetric: the mean of the gather and
//   scatter sums; n_i = number of such j (symmetric: |r_ij| < max(h_i, h_j)),
// with the Wendland C6 kernel of the paper's SPH application (section "Giant impact
// simulation"; Dehnen & Aly 2012), q = r / H < 1:
//   W(r, H) = 1365 / (64 pi H^3) (1 - q)^8 (1 + 8 q + 25 q^2 + 32 q^3).
// |r_ij|^2 = dx*dx + dy*dy + dz*dz is rounded as written (no contraction) and compared with
// H*H, so which pairs count is exact.  FP64 throughout; a wave takes runs of a group's members and
// the candidates near them, partial sums combined in a fixed order (deterministic).
#include "bottom_up.h"
#include "dev_util.h"
#include "fdx_internal.h"
#include "sift.h"

namespace fdx {

namespace {

constexpr int kThreads = 256;
constexpr double kWendlandC6 = 1365.0 / (64.0 * 3.14159265358979323846);

inline unsigned grid_for(size_t n, unsigned cap = 8192) {
    size_t b = (n + kThreads - 1) / kThreads;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

// support radius of every particle in sorted order (h given) or the fixed cutoff
__global__ void k_sph_radius(size_t n, const uint32_t *perm, const double *h, double r_fixed,
                             double *sh, DevStatus *st) {
    for (size_t r = gtid(); r < n; r += gstride()) {
        const double v = h ? h[perm[r]] : r_fixed;
        if (!(v > 0.0) || !isfinite(v)) atomicOr(&st->bad_input, 1u);
        sh[r] = v;
    }
}

// largest support radius in every cell, from the leaves up (bottom_up.h)
__device__ __forceinline__ void cell_hmax(const double *sh, double *hmax, const UpCell &u) {
    double v = 0.0;
    const double *p = u.nch ? hmax : sh;
    const uint32_t e = u.first + (u.nch ? u.nch : u.count);
    for (uint32_t i = u.first; i < e; i++) v = fmax(v, p[i]);
    hmax[u.id] = v;
}
__global__ void __launch_bounds__(kUpThreads)
k_cell_hmax(Cells c, const double *sh, double *hmax, UpBlocks u) {
    up_inside(c, u, [&](const UpCell &k) { cell_hmax(sh, hmax, k); });
}
__global__ void __launch_bounds__(kUpThreads)
k_cell_hmax_across(Cells c, const double *sh, double *hmax, UpBlocks u, uint32_t fan) {
    up_across(c, u, fan, [&](const UpCell &k) { cell_hmax(sh, hmax, k); });
}

// largest support radius of every group (one wave per group)
__global__ void __launch_bounds__(kThreads)
k_group_hmax(const uint32_t *ngroups, Groups g, const double *sh, double *rg) {
    const uint32_t G = min(*ngroups, g.cap);
    const int lane = lane_id();
    const size_t wave0 = gtid() / kWave, nwaves = gstride() / kWave;
    for (size_t gi = wave0; gi < G; gi += nwaves) {
        const uint32_t b = g.begin[gi], e = b + g.count[gi];
        double v = 0.0;
        for (uint32_t r = b + lane; r < e; r += kWave) v = fmax(v, sh[r]);
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) v = fmax(v, __shfl_xor(v, d, kWave));
        if (lane == 0) rg[gi] = v;
    }
}

// |r|^2 rounded as written, ((dx dx + dy dy) + dz dz), with no fused multiply-add, so the
// comparison with H^2 decides exactly as the plain definition does
__device__ __forceinline__ double dist2_as_written(double dx, double dy, double dz) {
#pragma clang fp contract(off)
    return (dx * dx + dy * dy) + dz * dz;
}

// W / norm at |r|^2 = r2, 1 / H = invh (the particle itself, r2 = 0, gets q = 1e-140)
__device__ __forceinline__ double wendland(double r2, double invh) {
    const double q = sqrt_pos(fma(r2 * invh, invh, 1e-280));
    const double u = 1.0 - q, u2 = u * u, u4 = u2 * u2, u8 = u4 * u4;
    return u8 * fma(q, fma(q, fma(q, 32.0, 25.0), 8.0), 1.0);
}

struct DensArgs {
    const uint32_t *ngroups;
    const uint32_t *gbegin, *gcount;
    const uint64_t *seg;
    const uint32_t *cnt_e, *list;
    const double4 *jp;
    const double *sh;
    double *rho;
    uint32_t *nngb;
    uint32_t parts, run;          // waves per group; consecutive blocks per XCD
};

// One wave per group, or several where groups are few (group_items.h), so nothing waits for other waves
// (half of the particles of a uniform set sit in groups of about eight).  The members are taken in runs of up to 16, neighbours along the
// curve; for each run the wave reads the candidates 64 at a time, keeps those within reach of
// the run's box in LDS (farther ones lie outside every support radius that could make a pair
// count), and lets the kept ones meet the run, js at a time.  FP64 VALU bound: 9 instructions
// decide a pair, about 25 evaluate one within the support (and some lane nearly always holds
// one).  2^24 uniform particles, 306 neighbours, 1540 candidates per member: 25.0 -> 18.6 ms
// (0.86 of the cycles issue a VALU instruction); runs of up to 8, 12, 20 members: 19.4, 18.7, 18.6 ms;
// a workgroup per group with the tile sifted by four waves: 24.0 ms, waiting at barriers.
constexpr uint32_t kHold = 2 * kWave;      // a block of 64 on top of up to 64 kept

template <int MODE>   // 0 fixed, 1 scatter, 2 gather, 3 symmetric
__global__ void __launch_bounds__(kSiftThreads) k_density(DensArgs a) {
    constexpr bool HJ = MODE == 1 || MODE == 3;          // the candidate's own radius counts
    __shared__ double4 kept_all[kSiftWaves][kHold];
    __shared__ double3 kepth_all[HJ ? kSiftWaves : 1][HJ ? kHold : 1];   // h, 1 / h, norm
    __shared__ double red_all[kSiftWaves][kWave];
    __shared__ uint32_t redn_all[kSiftWaves][kWave];
    const uint32_t G = *a.ngroups;
    const uint32_t lane = (uint32_t)lane_id(), w = uniform_u32(threadIdx.x / kWave);
    const uint64_t lt = lanemask_lt();
    double4 *kept = kept_all[w];
    double3 *kepth = kepth_all[HJ ? w : 0];
    const uint32_t vblocks = xcd_run_blocks(((size_t)G * a.parts + kSiftWaves - 1) / kSiftWaves, a.run);
    for (uint32_t vb = blockIdx.x; vb < vblocks; vb += gridDim.x) {
        const uint32_t item = uniform_u32(xcd_run_block(vb, a.run) * kSiftWaves + w);
        const uint32_t part = item / G, gi = item - part * G;
        if (part >= a.parts) continue;
        const uint32_t gb = uniform_u32(a.gbegin[gi]), ni = uniform_u32(a.gcount[gi]),
                       ne = uniform_u32(a.cnt_e[gi]);
        const uint32_t *cand = a.list + uniform_u64(a.seg[gi]);
        const uint32_t nrun = (ni + kRunMax - 1) / kRunMax, bs = (ni + nrun - 1) / nrun;
        const uint32_t js = kWave / bs, slot = lane / bs;
        for (uint32_t r0 = part * bs; r0 < ni; r0 += bs * a.parts) {
            const uint32_t n = min(bs, ni - r0), li = lane % bs;
            const bool active = slot < js && li < n;
            const uint32_t i = gb + r0 + (active ? li : 0u);
            const double4 pi = a.jp[i];
            const double hi = a.sh[i];
            const double hi2 = __dmul_rn(hi, hi), invhi = 1.0 / hi;
            double bc[3], bh[3], reach2 = hi2 * kSiftMargin<double>;
            sift_box<double>(pi.x, active, bc[0], bh[0]);
            sift_box<double>(pi.y, active, bc[1], bh[1]);
            sift_box<double>(pi.z, active, bc[2], bh[2]);
            if (MODE >= 2) {                             // the run's largest radius, or a bit more
                double hc, hh;
                sift_box<double>(hi, active, hc, hh);
                reach2 = (hc + hh) * (hc + hh) * kSiftMargin<double>;
            }
            double acc = 0.0, accj = 0.0;
            uint32_t cnt = 0, nk = 0;
            // the kept candidates meet the run
            auto meet = [&]() {
                wave_barrier();
                if (active) {
#pragma unroll 2
                    for (uint32_t k = slot; k < nk; k += js) {
                        const double4 pj = kept[k];
                        const double dx = __dsub_rn(pj.x, pi.x), dy = __dsub_rn(pj.y, pi.y),
                                     dz = __dsub_rn(pj.z, pi.z);
                        const double r2 = dist2_as_written(dx, dy, dz);
                        if (MODE == 0 || MODE == 2) {
                            if (r2 < hi2) { acc = fma(pj.w, wendland(r2, invhi), acc); cnt++; }
                        } else if (MODE == 1) {
                            const double3 hj = kepth[k];
                            if (r2 < __dmul_rn(hj.x, hj.x)) {
                                acc = fma(pj.w * hj.z, wendland(r2, hj.y), acc);
                                cnt++;
                            }
                        } else {
                            const double3 hj = kepth[k];
                            const bool in_i = r2 < hi2, in_j = r2 < __dmul_rn(hj.x, hj.x);
                            if (in_i) acc = fma(pj.w, wendland(r2, invhi), acc);
                            if (in_j) accj = fma(pj.w * hj.z, wendland(r2, hj.y), accj);
                            const double H = fmax(hi, hj.x);
                            if (r2 < __dmul_rn(H, H)) cnt++;
                        }
                    }
                }
                nk = 0;
                wave_barrier();
            };
            // indices are read two blocks ahead, positions one
            double4 p = make_double4(0, 0, 0, 0);
            double h = 1.0;
            uint32_t j1 = 0;
            if (ne) {
                j1 = cand[min(lane, ne - 1)];
                p = a.jp[j1];
                if (HJ) h = a.sh[j1];
                j1 = cand[min(lane + kWave, ne - 1)];
            }
            for (uint32_t t0 = 0; t0 < ne; t0 += kWave) {
                const double4 J = p;
                const double hj = h;
                p = a.jp[j1];
                if (HJ) h = a.sh[j1];
                j1 = cand[min(t0 + lane + 2 * kWave, ne - 1)];
                double lim = reach2;
                if (HJ) {
                    const double r2j = hj * hj * kSiftMargin<double>;
                    lim = MODE == 1 ? r2j : fmax(reach2, r2j);
                }
                const bool keep =
                    t0 + lane < ne && sift_dist2<double>(J.x, J.y, J.z, bc, bh) <= lim;
                const uint64_t b = __ballot(keep);
                if (keep) {
                    const uint32_t o = nk + (uint32_t)__popcll(b & lt);
                    kept[o] = J;
                    if (HJ) kepth[o] = make_double3(hj, 1.0 / hj, kWendlandC6 / (hj * hj * hj));
                }
                nk += (uint32_t)__popcll(b);
                if (nk >= (uint32_t)kWave) meet();
            }
            if (nk) meet();
            // the factors that are the same for every pair of a member
            const double normi = kWendlandC6 * invhi * invhi * invhi;
            double sum = acc;
            if (MODE == 0 || MODE == 2) sum = acc * normi;
            if (MODE == 3) sum = 0.5 * fma(acc, normi, accj);
            red_all[w][lane] = active ? sum : 0.0;
            redn_all[w][lane] = active ? cnt : 0u;
            wave_barrier();
            if (lane < n) {
                double s = 0.0;
                uint32_t c = 0;
                for (uint32_t k = 0; k < js; k++) {
                    s += red_all[w][k * bs + lane];
                    c += redn_all[w][k * bs + lane];
                }
                a.rho[gb + r0 + lane] = s;
                a.nngb[gb + r0 + lane] = c;
            }
            wave_barrier();
        }
    }
}

// results back to the caller's order
__global__ void k_sph_unsort(size_t n, const uint32_t *inv, const double *rho_s,
                             const uint32_t *n_s, double *rho, uint32_t *nngb) {
    for (size_t u = gtid(); u < n; u += gstride()) {
        const uint32_t r = inv[u];
        rho[u] = rho_s[r];
        nngb[u] = n_s[r];
    }
}

}  // namespace

hipError_t sph_radius(size_t n, const uint32_t *perm, const double *h, double r_fixed,
                      double *sh, DevStatus *st, hipStream_t s) {
    if (!n) return hipSuccess;
    hipLaunchKernelGGL(k_sph_radius, dim3(grid_for(n)), dim3(kThreads), 0, s, n, perm, h, r_fixed,
                       sh, st);
    return hipGetLastError();
}

hipError_t sph_cell_hmax(size_t n, int nsys, const int64_t *sys_off, const uint32_t *scratch,
                         const Cells c, const double *sh, double *hmax, hipStream_t s) {
    up_launch(up_blocks(n, nsys, sys_off, scratch),
              [&](uint32_t grid, int threads, const UpBlocks &u) {
                  hipLaunchKernelGGL(k_cell_hmax, dim3(grid), dim3(threads), 0, s, c, sh, hmax, u);
              },
              [&](uint32_t grid, int threads, const UpBlocks &u, uint32_t fan) {
                  hipLaunchKernelGGL(k_cell_hmax_across, dim3(grid), dim3(threads), 0, s, c, sh,
                                     hmax, u, fan);
              });
    return hipGetLastError();
}

hipError_t sph_group_hmax(size_t gmax, const Groups g, const double *sh, double *rg,
                          DevStatus *st, hipStream_t s) {
    if (!gmax) return hipSuccess;
    hipLaunchKernelGGL(k_group_hmax, dim3(grid_for(gmax * kWave, 4096)), dim3(kThreads), 0, s,
                       &st->n_groups_c, g, sh, rg);
    return hipGetLastError();
}

hipError_t sph_density(int mode, size_t gmax, int n_group, const Groups g, const uint64_t *seg,
                       const uint32_t *cnt_e, const uint32_t *list, const double4 *jp,
                       const double *sh, double *rho_s, uint32_t *n_s, DevStatus *st,
                       hipStream_t s) {
    if (!gmax) return hipSuccess;
    const GroupItems o = density_items(gmax, n_group);
    DensArgs a{&st->n_groups_c, g.begin, g.count, seg, cnt_e, list, jp, sh, rho_s, n_s, o.parts, o.run};
    const unsigned grid = o.blocks < 65536 ? o.blocks : 65536;   // 8 o.run divides both
    switch (mode) {
        case 0: hipLaunchKernelGGL(k_density<0>, dim3(grid), dim3(kSiftThreads), 0, s, a); break;
        case 1: hipLaunchKernelGGL(k_density<1>, dim3(grid), dim3(kSiftThreads), 0, s, a); break;
        case 2: hipLaunchKernelGGL(k_density<2>, dim3(grid), dim3(kSiftThreads), 0, s, a); break;
        default: hipLaunchKernelGGL(k_density<3>, dim3(grid), dim3(kSiftThreads), 0, s, a); break;
    }
    return hipGetLastError();
}

hipError_t sph_unsort(size_t n, const uint32_t *inv, const double *rho_s, const uint32_t *n_s,
                      double *rho, uint32_t *nngb, hipStream_t s) {
    if (!n) return hipSuccess;
    hipLaunchKernelGGL(k_sph_unsort, dim3(grid_for(n)), dim3(kThreads), 0, s, n, inv, rho_s, n_s,
                       rho, nngb);
    return hipGetLastError();
}

}  // namespace fdx
