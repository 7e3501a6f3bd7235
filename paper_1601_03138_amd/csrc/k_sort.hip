// Stable LSD radix sort of (63-bit key, u32 index) pairs, then stably by system id, so the
// result is ordered by (system, key, original index).  8-bit digits.
//
// Up to 8192 elements are sorted by one workgroup, all passes in LDS.  More are sorted in one
// launch per digit: one kernel histograms every digit place at once (the counts do not
// depend on the order), and each pass takes tiles by ticket, ranks the tile with ballot-based
// multisplit (stable), adds the counts of the tiles before it by looking back over their
// published sums (the single-pass scan with decoupled look-back, Merrill & Garland 2016), and
// writes each digit's run of the tile, laid out in LDS, contiguously.  With several systems
// (at most 2^16) and a carry buffer, a 16-bit copy of each element's system id travels with it
// through the key passes, so the system-id passes read their digit in order instead of
// gathering it through the permutation.
//
// A pass moves 24 B per element (12 read, 12 written) and is bound by HBM and by the latency of
// the chain load -> rank -> look back -> write.  Whole sort of 8 key passes, against a histogram,
// a three-launch scan and a scatter per pass: 2^24 elements 1.58 + 0.16 -> 1.14 ms, 2^20 150 + 60
// -> 167 us, 4096 170 -> 37 us, launches 40 -> 11 (1 up to 8192).  2^24 elements per pass: tiles of
// 4096 by 512 or 1024 threads 136 us, 2048 by 256 threads 201 us; 4, 6, 8, 16 look-back words at a
// time 139, 136, 139, 175 us.
#include "dev_util.h"
#include "fdx_internal.h"

namespace fdx {

namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / kWave;     // 8
constexpr int kItems = 8;                    // rounds of 64 per wave
constexpr int kWaveTile = kItems * kWave;    // 512 elements per wave
constexpr int kTile = kWaves * kWaveTile;    // 4096 elements per block
constexpr int kRadix = 256;
constexpr int kPlaces = 12;                  // digit places: 8 of the key, up to 4 of the system

// digit source: the key, the system id gathered through the index, or the carried system id
enum { kDigitKey = 0, kDigitSysGather = 1, kDigitSysCarried = 2 };

template <int SRC>
__device__ __forceinline__ uint32_t digit_of(uint64_t k, uint32_t v, uint32_t sc,
                                             const uint32_t *sysid, int shift) {
    if (SRC == kDigitSysGather) return (sysid[v] >> shift) & (kRadix - 1);
    if (SRC == kDigitSysCarried) return (sc >> shift) & (kRadix - 1);
    return (uint32_t)(k >> shift) & (kRadix - 1);
}

// the lanes holding the same digit as this one, among the lanes of `valid`
__device__ __forceinline__ uint64_t same_digit(uint32_t d, uint64_t valid) {
    uint64_t m = valid;
#pragma unroll
    for (int b = 0; b < 8; b++) {
        const uint64_t bal = __ballot((d >> b) & 1u);
        m &= ((d >> b) & 1u) ? bal : ~bal;
    }
    return m;
}

// Scratch of the multi-block sort: a ticket per pass, the digit bases of every place, and the
// look-back words of every (tile, digit).
struct Scratch {
    uint32_t *ticket, *base;
    uint64_t *state;
};
constexpr size_t kHeadWords = 64 + (size_t)kPlaces * kRadix;
__host__ __device__ inline Scratch scratch_view(uint32_t *p) {
    return Scratch{p, p + 64, reinterpret_cast<uint64_t *>(p + kHeadWords)};
}

// counts of every digit of every place: `places` of the key from bit 0, then sys_places of the
// system id.  Four copies per block keep lanes with equal digits apart.
__global__ void __launch_bounds__(kThreads)
k_rs_hist(const uint64_t *key, const uint32_t *sysid, size_t n, int places, int sys_places,
          uint32_t *base) {
    __shared__ uint32_t h[8][kRadix][4];
    for (int k = threadIdx.x; k < 8 * kRadix * 4; k += kThreads) (&h[0][0][0])[k] = 0;
    __syncthreads();
    const int c = threadIdx.x & 3;
    for (size_t i = gtid(); i < n; i += gstride()) {
        const uint64_t k = key[i];
#pragma unroll
        for (int p = 0; p < 8; p++)
            if (p < places) atomicAdd(&h[p][(k >> (8 * p)) & (kRadix - 1)][c], 1u);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < places * kRadix; k += kThreads) {
        const uint32_t *q = &h[0][0][0] + 4 * k;
        const uint32_t v = q[0] + q[1] + q[2] + q[3];
        if (v) atomicAdd(&base[k], v);
    }
    if (!sys_places) return;
    __syncthreads();
    for (int k = threadIdx.x; k < 4 * kRadix * 4; k += kThreads) (&h[0][0][0])[k] = 0;
    __syncthreads();
    for (size_t i = gtid(); i < n; i += gstride()) {
        const uint32_t s = sysid[i];
#pragma unroll
        for (int p = 0; p < 4; p++)
            if (p < sys_places) atomicAdd(&h[p][(s >> (8 * p)) & (kRadix - 1)][c], 1u);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < sys_places * kRadix; k += kThreads) {
        const uint32_t *q = &h[0][0][0] + 4 * k;
        const uint32_t v = q[0] + q[1] + q[2] + q[3];
        if (v) atomicAdd(&base[places * kRadix + k], v);
    }
}

// counts -> exclusive sums within each place (one block per place)
__global__ void __launch_bounds__(kRadix) k_rs_base(uint32_t *base) {
    __shared__ uint64_t tmp[kRadix / kWave];
    uint64_t tot;
    uint32_t *b = base + (size_t)blockIdx.x * kRadix;
    const uint32_t e = (uint32_t)block_excl_scan<kRadix>(b[threadIdx.x], tmp, &tot);
    b[threadIdx.x] = e;
}

// Look-back word: value << 8 | pass << 2 | kind (1 the tile's own count, 2 the sum of all tiles
// up to it).  One 64-bit word carries both, so relaxed atomics at device scope do, and a word of an
// earlier pass is never mistaken for this one's.
constexpr uint64_t kOwn = 1, kSum = 2;
__device__ __forceinline__ uint64_t look_word(uint64_t v, int pass, uint64_t kind) {
    return v << 8 | (uint64_t)(pass + 1) << 2 | kind;
}
__device__ __forceinline__ uint64_t look_load(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void look_store(uint64_t *p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One pass.  Tiles are numbered by ticket in the order blocks start, so every tile looked back at
// has started, and a tile publishes its own counts before it waits for anything: every wait ends.
// CARRY moves the 16-bit system ids along (sc_in -> sc_out).
template <int SRC, bool CARRY>
__global__ void __launch_bounds__(kThreads)
k_rs_pass(const uint64_t *key_in, const uint32_t *val_in, const uint16_t *sc_in,
          const uint32_t *sysid, size_t n, int shift, int pass, uint32_t *scratch,
          uint64_t *key_out, uint32_t *val_out, uint16_t *sc_out) {
    static_assert(SRC != kDigitSysCarried || CARRY, "carried digits are staged with the carry");
    __shared__ uint64_t sk[kTile];
    __shared__ uint32_t sv[kTile];
    __shared__ uint16_t ss[CARRY ? kTile : 1];
    __shared__ uint32_t wcnt[kWaves][kRadix];     // per wave and digit: count, then offset
    __shared__ uint32_t lstart[kRadix];           // first LDS slot of each digit
    __shared__ uint32_t gstart[kRadix];           // global position of that slot
    __shared__ uint64_t scan_tmp[kWaves];
    __shared__ uint32_t tile_s;
    const Scratch sc = scratch_view(scratch);
    if (threadIdx.x == 0) tile_s = atomicAdd(&sc.ticket[pass], 1u);
    for (int k = threadIdx.x; k < kWaves * kRadix; k += kThreads) (&wcnt[0][0])[k] = 0;
    __syncthreads();
    const uint32_t tile = tile_s;
    const int w = threadIdx.x / kWave, lane = lane_id();
    const uint64_t lt = lanemask_lt();
    const size_t b0 = (size_t)tile * kTile, base = b0 + (size_t)w * kWaveTile;
    uint64_t kk[kItems];
    uint32_t vv[kItems], rk[kItems], cc[kItems];
#pragma unroll
    for (int r = 0; r < kItems; r++) {
        const size_t i = base + (size_t)r * kWave + lane;
        const size_t j = i < n ? i : n - 1;
        kk[r] = key_in[j];
        vv[r] = val_in[j];
        cc[r] = CARRY ? sc_in[j] : 0u;
    }
#pragma unroll
    for (int r = 0; r < kItems; r++) {
        const bool valid = base + (size_t)r * kWave + lane < n;
        const uint32_t d = digit_of<SRC>(kk[r], vv[r], cc[r], sysid, shift);
        const uint64_t m = same_digit(d, __ballot(valid));
        const uint32_t before = (uint32_t)__popcll(m & lt);
        const uint32_t prev = wcnt[w][d];
        wave_barrier();
        if (valid && before == 0) wcnt[w][d] = prev + (uint32_t)__popcll(m);
        wave_barrier();
        rk[r] = valid ? (d << 16) | (prev + before) : 0xFFFFFFFFu;
    }
    __syncthreads();
    uint32_t tot = 0;
    uint64_t *mine = sc.state + (size_t)tile * kRadix;
    const int d = threadIdx.x;
    if (d < kRadix) {
#pragma unroll
        for (int ww = 0; ww < kWaves; ww++) {
            const uint32_t c = wcnt[ww][d];
            wcnt[ww][d] = tot;
            tot += c;
        }
        look_store(mine + d, look_word(tot, pass, tile ? kOwn : kSum));
    }
    uint64_t btot;
    const uint32_t ls = (uint32_t)block_excl_scan<kThreads>(tot, scan_tmp, &btot);
    if (d < kRadix) lstart[d] = ls;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kItems; r++) {
        if (rk[r] != 0xFFFFFFFFu) {
            const uint32_t dg = rk[r] >> 16;
            const uint32_t slot = lstart[dg] + wcnt[w][dg] + (rk[r] & 0xFFFFu);
            sk[slot] = kk[r];
            sv[slot] = vv[r];
            if (CARRY) ss[slot] = (uint16_t)cc[r];
        }
    }
    if (d < kRadix) {
        // counts of the tiles before this one: kWin words are read together
        constexpr int kWin = 6;
        uint64_t before = 0;
        const uint64_t tag = (uint64_t)(pass + 1) << 2;
        bool found = tile == 0;
        for (int64_t t = (int64_t)tile - 1; !found;) {
            uint64_t s[kWin];
#pragma unroll
            for (int q = 0; q < kWin; q++)
                s[q] = look_load(sc.state + (size_t)(t - q > 0 ? t - q : 0) * kRadix + d);
#pragma unroll
            for (int q = 0; q < kWin; q++) {
                // words are used in order; the first one not published yet is read again
                if (found || t < 0 || (s[q] & 0xFCull) != tag || !(s[q] & 3ull)) break;
                before += s[q] >> 8;
                found = (s[q] & 3ull) == kSum;
                t--;
            }
        }
        if (tile) look_store(mine + d, look_word(before + tot, pass, kSum));
        gstart[d] = sc.base[(size_t)pass * kRadix + d] + (uint32_t)before;
    }
    __syncthreads();
    const uint32_t cnt = (uint32_t)(n - b0 < (size_t)kTile ? n - b0 : (size_t)kTile);
    for (uint32_t j = threadIdx.x; j < cnt; j += kThreads) {
        const uint64_t k = sk[j];
        const uint32_t v = sv[j];
        const uint32_t c = CARRY ? (uint32_t)ss[j] : 0u;
        const uint32_t dg = digit_of<SRC>(k, v, c, sysid, shift);
        const uint32_t pos = gstart[dg] + (j - lstart[dg]);
        key_out[pos] = k;
        val_out[pos] = v;
        if (CARRY) sc_out[pos] = (uint16_t)c;
    }
}

// All passes of a small sort in one workgroup, in place: the elements go through LDS from pass to
// pass.  4096 elements take 37 us, 4.6 us a pass: two thirds of the launches, look-back chains and
// idle CUs of the tiled sort at 8193 (8.4 us a pass), and a single launch.  It ends at the
// 8192 elements (and their counters) that one CU's LDS holds.
constexpr int kBlockThreads = 1024;
constexpr int kBlockWaves = kBlockThreads / kWave;
constexpr size_t kBlockMax = 8192;

template <int ITEMS>
__global__ void __launch_bounds__(kBlockThreads)
k_rs_block(uint64_t *key, uint32_t *val, const uint32_t *sysid, uint32_t n, int places,
           int sys_places) {
    __shared__ uint64_t sk[kBlockThreads * ITEMS];
    __shared__ uint32_t sv[kBlockThreads * ITEMS];
    __shared__ uint32_t wcnt[kBlockWaves][kRadix];
    __shared__ uint32_t lstart[kRadix];
    __shared__ uint64_t scan_tmp[kBlockWaves];
    const int w = threadIdx.x / kWave, lane = lane_id();
    const uint64_t lt = lanemask_lt();
    const uint32_t base = (uint32_t)(w * ITEMS * kWave + lane);
    uint64_t kk[ITEMS];
    uint32_t vv[ITEMS], rk[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
        const uint32_t i = base + (uint32_t)(r * kWave);
        kk[r] = i < n ? key[i] : 0;
        vv[r] = i < n ? val[i] : 0;
    }
    for (int p = 0; p < places + sys_places; p++) {
        for (int k = threadIdx.x; k < kBlockWaves * kRadix; k += kBlockThreads)
            (&wcnt[0][0])[k] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; r++) {
            const bool valid = base + (uint32_t)(r * kWave) < n;
            const uint32_t d =
                p < places ? digit_of<kDigitKey>(kk[r], 0, 0, nullptr, 8 * p)
                           : (valid ? digit_of<kDigitSysGather>(0, vv[r], 0, sysid,
                                                                8 * (p - places)) : 0u);
            const uint64_t m = same_digit(d, __ballot(valid));
            const uint32_t before = (uint32_t)__popcll(m & lt);
            const uint32_t prev = wcnt[w][d];
            wave_barrier();
            if (valid && before == 0) wcnt[w][d] = prev + (uint32_t)__popcll(m);
            wave_barrier();
            rk[r] = valid ? (d << 16) | (prev + before) : 0xFFFFFFFFu;
        }
        __syncthreads();
        uint32_t tot = 0;
        const int d = threadIdx.x;
        if (d < kRadix) {
#pragma unroll
            for (int ww = 0; ww < kBlockWaves; ww++) {
                const uint32_t c = wcnt[ww][d];
                wcnt[ww][d] = tot;
                tot += c;
            }
        }
        uint64_t btot;
        const uint32_t ls = (uint32_t)block_excl_scan<kBlockThreads>(tot, scan_tmp, &btot);
        if (d < kRadix) lstart[d] = ls;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; r++) {
            if (rk[r] != 0xFFFFFFFFu) {
                const uint32_t dg = rk[r] >> 16;
                const uint32_t slot = lstart[dg] + wcnt[w][dg] + (rk[r] & 0xFFFFu);
                sk[slot] = kk[r];
                sv[slot] = vv[r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; r++) {
            const uint32_t i = base + (uint32_t)(r * kWave);
            if (i < n) { kk[r] = sk[i]; vv[r] = sv[i]; }
        }
    }
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
        const uint32_t i = base + (uint32_t)(r * kWave);
        if (i < n) { key[i] = kk[r]; val[i] = vv[r]; }
    }
}

// 16-bit system ids in input order (the carry's starting copy)
__global__ void k_carry_init(size_t n, const uint32_t *sysid, uint16_t *sc) {
    for (size_t i = gtid(); i < n; i += gstride()) sc[i] = (uint16_t)sysid[i];
}

template <int SRC, bool CARRY>
void rs_pass(uint32_t ntiles, hipStream_t s, const uint64_t *kin, const uint32_t *vin,
             const uint16_t *cin, const uint32_t *sysid, size_t n, int shift, int pass,
             uint32_t *scratch, uint64_t *kout, uint32_t *vout, uint16_t *cout) {
    hipLaunchKernelGGL((k_rs_pass<SRC, CARRY>), dim3(ntiles), dim3(kThreads), 0, s, kin, vin, cin,
                       sysid, n, shift, pass, scratch, kout, vout, cout);
}

}  // namespace

size_t radix_scratch_u32(size_t n) {
    if (n <= kBlockMax) return 1;
    return kHeadWords + 2 * (size_t)kRadix * ((n + kTile - 1) / kTile);
}

hipError_t radix_sort(size_t n, uint64_t *key, uint64_t *key_alt, uint32_t *val,
                      uint32_t *val_alt, const uint32_t *sysid, int nsys, int key_bits,
                      uint32_t *scratch, bool *result_in_alt, hipStream_t s, uint16_t *carry) {
    *result_in_alt = false;
    if (n <= 1) return hipSuccess;
    int sys_passes = 0;
    for (int b = 0; (1ll << b) < (long long)nsys; b += 8) sys_passes++;
    const int key_passes = (key_bits + 7) / 8;
    if (key_passes + sys_passes == 0) return hipSuccess;
    if (n <= kBlockMax) {
        // one workgroup: 4096 elements at four per thread, else eight
        if (n <= kBlockMax / 2)
            hipLaunchKernelGGL(k_rs_block<4>, dim3(1), dim3(kBlockThreads), 0, s, key, val, sysid,
                               (uint32_t)n, key_passes, sys_passes);
        else
            hipLaunchKernelGGL(k_rs_block<8>, dim3(1), dim3(kBlockThreads), 0, s, key, val, sysid,
                               (uint32_t)n, key_passes, sys_passes);
        return hipGetLastError();
    }
    const uint32_t ntiles = (uint32_t)((n + kTile - 1) / kTile);
    hipError_t e = fill_u32(scratch, 0u, radix_scratch_u32(n), s);
    if (e != hipSuccess) return e;
    const Scratch sc = scratch_view(scratch);
    const size_t hb = (n + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(k_rs_hist, dim3((unsigned)(hb < 4 * 1024 ? (hb + 3) / 4 : 1024)), dim3(kThreads), 0, s,
                       key, sysid, n, key_passes, sys_passes, sc.base);
    hipLaunchKernelGGL(k_rs_base, dim3(key_passes + sys_passes), dim3(kRadix), 0, s, sc.base);
    uint64_t *kin = key, *kout = key_alt;
    uint32_t *vin = val, *vout = val_alt;
    const int passes = key_passes + sys_passes;  // key bytes, then system id bytes
    const bool carried = sys_passes > 0 && carry && nsys <= 65536;
    uint16_t *cin = carried ? carry : nullptr, *cout = carried ? carry + n : nullptr;
    if (carried) {
        const size_t b = (n + 255) / 256;
        hipLaunchKernelGGL(k_carry_init, dim3((unsigned)(b < 16384 ? b : 16384)), dim3(256), 0, s,
                           n, sysid, cin);
    }
    for (int p = 0; p < passes; p++) {
        const bool sysp = p >= key_passes;
        const int shift = sysp ? 8 * (p - key_passes) : 8 * p;
        if (!sysp && carried)
            rs_pass<kDigitKey, true>(ntiles, s, kin, vin, cin, sysid, n, shift, p, scratch, kout,
                                     vout, cout);
        else if (!sysp)
            rs_pass<kDigitKey, false>(ntiles, s, kin, vin, cin, sysid, n, shift, p, scratch, kout,
                                      vout, cout);
        else if (carried)
            rs_pass<kDigitSysCarried, true>(ntiles, s, kin, vin, cin, sysid, n, shift, p, scratch,
                                            kout, vout, cout);
        else
            rs_pass<kDigitSysGather, false>(ntiles, s, kin, vin, cin, sysid, n, shift, p, scratch,
                                            kout, vout, cout);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        uint64_t *tk = kin; kin = kout; kout = tk;
        uint32_t *tv = vin; vin = vout; vout = tv;
        uint16_t *tc = cin; cin = cout; cout = tc;
    }
    *result_in_alt = (kin == key_alt);
    return hipSuccess;
}

}  // namespace fdx
