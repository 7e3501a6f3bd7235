// Expansion of every group's far superparticles into one polynomial (far_field.h).
//
// One wave per group.  It reads the group's superparticle list in blocks of 128 entries, keeps
// the far ones in an LDS queue, and whenever 64 are queued every lane takes one and adds its
// terms to 46 register accumulators.  The lanes are summed with DPP moves, and every member's
// far field is evaluated and written where the force kernel adds the pairs to it.  The list is
// partitioned in place on the way, near entries first, so the force kernel reads only those.
//
// About 240 instructions per far superparticle, where one pair costs 34.5.  Bound by the gathers of
// 80-byte cell records out of L2, most of them to tell near from far: 2^24 clustered particles,
// n_group 256, 6.7e8 entries, 0.30 of their interactions far: 4.6 ms, and the force kernel 42 -> 31.7 ms.
// The time is the same with 2, 3 or 4 waves per SIMD, 64, 128 or 256 entries per block, with far
// entries at half the instructions, and with records read by pairs of lanes (half the L1
// accesses); L2 requests are what these have in common.
#include <algorithm>
#include <type_traits>

#include "dev_util.h"
#include "far_field.h"
#include "far_partition.h"
#include "fdx_internal.h"

namespace fdx {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kScan = kFarBlock / kWave;          // list entries per lane and block
constexpr uint32_t kQueue = kFarBlock + kWave;    // a block on top of a part-filled round

struct FarArgs {
    const uint32_t *ngroups, *gcount;
    const FarGeom *geom;
    const double *mom;
    const uint64_t *seg;
    const uint32_t *cap, *cnt_s;
    uint32_t *list, *near;
    const uint32_t *gbegin;
    const double4 *jp;
    double4 *fs;
    uint32_t gmax;
};

// sum over the 64 lanes, returned to every lane
__device__ __forceinline__ float wave_sum_f32(float v) {
    auto move = [](float x, auto ctrl, auto mask) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value,
                                                          decltype(mask)::value, 0xf, false));
    };
    using std::integral_constant;
    v += move(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});   // row_shr:1
    v += move(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});   // row_shr:2
    v += move(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});   // row_shr:4
    v += move(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});   // row_shr:8
    v += move(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});   // row_bcast:15
    v += move(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});   // row_bcast:31
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), kWave - 1));
}
template <int CTRL, int MASK>
__device__ __forceinline__ double dpp_add_f64(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, MASK, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, MASK, 0xf,
                                                              false);
    return v + __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double wave_sum_f64(double v) {
    v = dpp_add_f64<0x111, 0xf>(v);
    v = dpp_add_f64<0x112, 0xf>(v);
    v = dpp_add_f64<0x114, 0xf>(v);
    v = dpp_add_f64<0x118, 0xf>(v);
    v = dpp_add_f64<0x142, 0xa>(v);
    v = dpp_add_f64<0x143, 0xc>(v);
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, kWave - 1);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), kWave - 1);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

template <bool QUAD>
__global__ void __launch_bounds__(kThreads, 3)
k_far(FarArgs a) {
    __shared__ float4 qx_all[kWaves][kQueue];          // to be expanded
    __shared__ uint32_t qi_all[QUAD ? kWaves : 1][QUAD ? kQueue : 1];
    __shared__ uint32_t held_all[kWaves][2][kFarHeld];    // ids to be written back: near, far
    const int w = threadIdx.x / kWave, lane = lane_id();
    const uint64_t lt = lanemask_lt();
    const uint32_t G = min(*a.ngroups, a.gmax);
    const double2 *mom = reinterpret_cast<const double2 *>(a.mom);
    // The four waves of a block take four consecutive groups, whose lists begin with the same
    // cells of the upper tree; blocks of neighbouring groups share an XCD.
    const uint32_t vblocks = xcd_run_blocks((G + kWaves - 1) / kWaves);
    for (uint32_t vb = blockIdx.x; vb < vblocks; vb += gridDim.x) {
    const uint32_t gi = uniform_u32(xcd_run_block(vb) * kWaves + (uint32_t)w);
    if (gi >= G) continue;
    const FarGeom f = a.geom[gi];
    const uint32_t ns = uniform_u32(a.cnt_s[gi]), ni = uniform_u32(a.gcount[gi]);
    if (!far_worth<QUAD>(f.thr2, ni, ns)) {
        if (lane == 0) a.near[gi] = kNone;
        continue;
    }
    uint32_t *spj = a.list + uniform_u64(a.seg[gi]) + (uniform_u32(a.cap[gi]) - ns);
    const double q2 = f.inv_h * f.inv_h;
    FarAcc acc;
    const float inv_h = (float)f.inv_h;            // a power of two: scaling by it is exact
    auto expand = [&](uint32_t slot) {
        const float4 e = qx_all[w][slot];
        float q[6] = {0, 0, 0, 0, 0, 0};
        if (QUAD) {
            const double2 *o = mom + 5 * (size_t)qi_all[w][slot] + 2;
            const double2 u = o[0], v = o[1], t = o[2];
            q[0] = (float)(u.x * q2); q[1] = (float)(u.y * q2); q[2] = (float)(v.x * q2);
            q[3] = (float)(v.y * q2); q[4] = (float)(t.x * q2); q[5] = (float)(t.y * q2);
        }
        const float x = e.x * inv_h, y = e.y * inv_h, z = e.z * inv_h;
        const float i = __builtin_amdgcn_rsqf(fmaf(z, z, fmaf(y, y, fmaf(x, x, f.e2))));
        acc.template add<QUAD>(x, y, z, i, e.w, q);
    };
    FarPartition part(ns);
    using Block = FarPartition::Block;
    auto load_ids = [&](const Block &b, uint32_t (&id)[kScan]) {
#pragma unroll
        for (int k = 0; k < kScan; k++) {
            const uint32_t j = (uint32_t)(k * kWave + lane);
            id[k] = b.len ? spj[b.start + min(j, b.len - 1)] : 0u;
        }
    };
    auto load_com = [&](const uint32_t (&id)[kScan], double2 (&u)[kScan], double2 (&v)[kScan]) {
#pragma unroll
        for (int k = 0; k < kScan; k++) {
            u[k] = mom[5 * (size_t)id[k]];
            v[k] = mom[5 * (size_t)id[k] + 1];
        }
    };
    uint32_t cnt = 0;                              // queued for expansion, the same in every lane
    Block b0 = part.choose(0), b1 = part.choose(0);
    uint32_t id0[kScan], id1[kScan];
    double2 u0[kScan], v0[kScan];
    load_ids(b0, id0);
    load_ids(b1, id1);
    load_com(id0, u0, v0);
    while (b0.len) {
#pragma unroll
        for (int k = 0; k < kScan; k++) {
            const float px = (float)(u0[k].y - f.ex), py = (float)(v0[k].x - f.ey),
                        pz = (float)(v0[k].y - f.ez);
            const float r2 = fmaf(pz, pz, fmaf(py, py, px * px));
            const bool in = (uint32_t)(k * kWave + lane) < b0.len;
            const bool far = r2 > f.thr2 && in;
            const uint64_t m = __ballot(far);
            const uint32_t nf = (uint32_t)__popcll(m), rank = (uint32_t)__popcll(m & lt);
            if (in) {
                // the entries of a block are its first lanes, so the near ones before a lane are
                // the lanes before it less the far ones
                const uint32_t at = far ? part.held[1] + rank : part.held[0] + (uint32_t)lane - rank;
                held_all[w][far ? 1 : 0][at] = id0[k];
            }
            if (far) {
                qx_all[w][cnt + rank] = make_float4(px, py, pz, (float)u0[k].x);
                if (QUAD) qi_all[w][cnt + rank] = id0[k];
            }
            cnt += nf;
            part.held[0] += min(kWave + 0u, b0.len > (uint32_t)(k * kWave) ? b0.len - k * kWave : 0u) - nf;
            part.held[1] += nf;
        }
        const uint32_t back = part.sorted(b0);
        wave_barrier();
        // the next block: ids long arrived, its centres of mass on the way during the expansion
        const Block b2 = part.choose(back);
        b0 = b1;
        b1 = b2;
#pragma unroll
        for (int k = 0; k < kScan; k++) id0[k] = id1[k];
        load_com(id0, u0, v0);
        load_ids(b1, id1);
        // ids back into free slots
#pragma unroll
        for (int c = 0; c < 2; c++) {
            const uint32_t n = part.ready(c);
            for (uint32_t i = (uint32_t)lane; i < n; i += kWave)
                spj[part.slot(c, i)] = held_all[w][c][part.held[c] + i];
            part.written(c, n);
        }
        while (cnt >= (uint32_t)kWave) {
            cnt -= kWave;
            expand(cnt + (uint32_t)lane);
        }
        wave_barrier();
    }
    // every slot is read: what is left goes to the slots in between
#pragma unroll
    for (int c = 0; c < 2; c++)
        for (uint32_t i = (uint32_t)lane; i < part.held[c]; i += kWave)
            spj[part.slot(c, i)] = held_all[w][c][i];
    if (lane == 0) a.near[gi] = part.put[0] + part.held[0];
    if ((uint32_t)lane < cnt) expand((uint32_t)lane);
    acc.fold();
    // the sums over the wave, the same in every lane
    FarCoef c;
    c.c0 = uniform_f64(wave_sum_f64(acc.c0));
#pragma unroll
    for (int u = 0; u < 3; u++) c.c1[u] = uniform_f64(wave_sum_f64(acc.c1[u]));
#pragma unroll
    for (int u = 0; u < 6; u++) c.c2[u] = wave_sum_f32(acc.c2[u]);
#pragma unroll
    for (int u = 0; u < 10; u++) c.c3[u] = wave_sum_f32(acc.c3[u]);
#pragma unroll
    for (int u = 0; u < 15; u++) c.c4[u] = wave_sum_f32(acc.c4[u]);
    // the members' far field, which the force kernel adds its pairs to
    const uint32_t gb = uniform_u32(a.gbegin[gi]);
    for (uint32_t i = (uint32_t)lane; i < ni; i += kWave) {
        const double4 p = a.jp[gb + i];
        double4 o = make_double4(0, 0, 0, 0);
        far_eval(c, f.inv_h, (float)((p.x - f.ex) * f.inv_h), (float)((p.y - f.ey) * f.inv_h),
                 (float)((p.z - f.ez) * f.inv_h), o.x, o.y, o.z, o.w);
        a.fs[gb + i] = o;
    }
    }
}

}  // namespace

hipError_t far_expand(size_t gmax, const ForceArgs &fa, hipStream_t s) {
    if (!gmax) return hipSuccess;
    const size_t blocks = xcd_run_blocks((gmax + kWaves - 1) / kWaves);
    const unsigned grid = (unsigned)std::min<size_t>(blocks, 256 * kXcdRun);
    FarArgs a;
    a.ngroups = &fa.st->n_groups_c;
    a.gcount = fa.g->count; a.geom = fa.g->far; a.mom = fa.mom;
    a.seg = fa.seg; a.cap = fa.cap; a.cnt_s = fa.cnt_s; a.list = fa.list; a.near = fa.near;
    a.gbegin = fa.g->begin; a.jp = fa.jp; a.fs = fa.fs;
    a.gmax = (uint32_t)gmax;
    if (fa.quad) hipLaunchKernelGGL(k_far<true>, dim3(grid), dim3(kThreads), 0, s, a);
    else hipLaunchKernelGGL(k_far<false>, dim3(grid), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace fdx
