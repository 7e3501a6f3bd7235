// CPU check that entry points allocate and launch on their context's device: the HIP runtime is
// replaced by one on host memory with two devices, the kernel launchers by ones that do nothing,
// and each entry point runs on a context of device 1 while device 0 is current.  Prints
// "entry|status|allocations and launches on device 1|on another device".
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "exchange.cpp"           // its state is local to it
#include "mlp.h"

static int current, good, bad;
static hipError_t seen() { (current == 1 ? good : bad)++; return hipSuccess; }

extern "C" {
hipError_t hipSetDevice(int d) { current = d; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = calloc(1, n); return seen(); }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    memcpy(d, s, n);
    return seen();                 // on the current device's stream
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return ""; }
}

namespace fdx {
size_t exchange_subwalks(int nsys) { return (size_t)kExchangeFrontierMax * nsys * (nsys - 1); }
hipError_t exchange_gather(size_t, const uint32_t *, const uint32_t *, const uint64_t *,
                           const uint32_t *, const uint32_t *, const uint32_t *, const uint64_t *,
                           const uint64_t *, const uint32_t *, const uint32_t *, uint32_t *,
                           uint32_t *, hipStream_t) { return seen(); }
hipError_t compact_lists(size_t, const uint64_t *, const uint32_t *, const uint32_t *,
                         const uint32_t *, const uint64_t *, const uint64_t *, const uint32_t *,
                         uint32_t *, uint32_t *, hipStream_t) { return seen(); }
hipError_t iota_u32(uint32_t *, size_t, hipStream_t) { return seen(); }
hipError_t mlp_features(size_t, const Groups, const Cells, const int64_t *, const float *,
                        const float *, float *, DevStatus *, hipStream_t) { return seen(); }
hipError_t mlp_infer(size_t, const uint32_t *, const float *, const float *, float *, hipStream_t) {
    return seen();
}
size_t mlp_train_blocks(size_t) { return 1; }
hipError_t mlp_grad(size_t, const uint32_t *, const float *, const float *, const float *, float *,
                    float *, float *, float *, hipStream_t) { return seen(); }
hipError_t mlp_adam(float *, const float *, float *, float *, int, float, hipStream_t) {
    return seen();
}
}  // namespace fdx

template <class F>
static void entry(const char *name, F f) {
    current = good = bad = 0;
    const int r = f();
    std::printf("%s|%d|%d|%d\n", name, r, good, bad);
}

int main(int, char **argv) {
    using namespace fdx;
    static DevStatus st;
    uint32_t one[2] = {1, 1}, word[8] = {};
    uint64_t off[2] = {0, 1};
    static float P[kMlpParams], m[kMlpParams], v[kMlpParams], g[kMlpParams];
    static float X[64 * kMlpIn], t[64], y[64];
    fdx_ctx *c = new fdx_ctx();
    c->device = 1;
    c->st = &st;
    c->have_counts = c->have_lists = true;
    c->stats.n_groups = 1;
    c->cnt_e.p = c->cnt_s.p = one;
    c->skey = off;                     // a tree is built
    ExchangeState *x = new ExchangeState();
    x->built = true;
    x->nsys = 2;
    x->pairs = 2;
    x->n_epj = x->n_spj = 1;
    c->ext.exch = x;

    entry("fdx_get_exchange_lists", [&] { return fdx_get_exchange_lists(c, word, word + 1); });
    entry("fdx_get_lists", [&] { return fdx_get_lists(c, word, word + 1, word + 2, word + 3); });
    entry("fdx_mlp_forward", [&] { return fdx_mlp_forward(c, P, X, 64, y); });
    entry("fdx_mlp_grad", [&] { return fdx_mlp_grad(c, P, X, t, 64, g, y); });
    entry("fdx_mlp_adam", [&] { return fdx_mlp_adam(c, P, m, v, g, 1, 0, 1e-3); });
    entry("fdx_predictor_features", [&] { return fdx_predictor_features(c, X); });
    entry("fdx_predictor_train",
          [&] { return fdx_predictor_train(c, X, t, 64, 1, 16, 1e-3, 1, nullptr); });
    entry("fdx_predictor_save", [&] { return fdx_predictor_save(c, argv[1]); });
    entry("fdx_predictor_load", [&] { return fdx_predictor_load(c, argv[1]); });
    return 0;
}
