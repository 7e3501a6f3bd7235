// Exchange lists between domains (section "Exchange of particles and superparticles",
// long-range mode): the domains are the systems of the particle set, each with its own local
// tree; every ordered pair (sender, receiver) is a walk of the sender's tree against the
// receiver's particle box, split into sub-walks over the sender's top-level frontier and run
// by the group-walk kernels through their selection arguments.
#include <algorithm>
#include <vector>

#include "ctx.h"

namespace fdx {

namespace {

// largest list buffer sized by the per-sender bound (one fill walk); 16 GiB of the GPU's HBM
constexpr uint64_t kExchangeBudgetBytes = 16ull << 30;

struct ExchangeState {
    DBuf<uint32_t> box, start, sel, ne, ns, cap, list, nsel, front, fcount;
    DBuf<uint64_t> seg, total;
    DBuf<uint64_t> oe, os, sums;     // prefix sums of ne and ns, their totals
    DBuf<uint32_t> pe, ps;           // entries per ordered pair
    DBuf<uint32_t> out_e, out_s;     // lists in pair order (fdx_get_exchange_lists)
    uint64_t list_cap = 0;
    int nsys = 0;
    size_t pairs = 0;
    uint64_t entries = 0, n_epj = 0, n_spj = 0, capacity = 0;
    double ms_tree = 0, ms_lists = 0;
    bool built = false;
    uint64_t gen = 0;            // context generation the lists belong to
    hipEvent_t ev[3] = {};

    void release() {
        for (auto *b : {&box, &start, &sel, &ne, &ns, &cap, &list, &nsel, &front, &fcount})
            b->release();
        for (auto *b : {&seg, &total, &oe, &os, &sums}) b->release();
        for (auto *b : {&pe, &ps, &out_e, &out_s}) b->release();
        for (auto &e : ev)
            if (e) { (void)hipEventDestroy(e); e = nullptr; }
        list_cap = 0;
        built = false;
    }
};

ExchangeState *state(fdx_ctx *c) {
    if (!c->ext.exch) c->ext.exch = new ExchangeState();
    return static_cast<ExchangeState *>(c->ext.exch);
}

int check_built(fdx_ctx *c) {
    ExchangeState *x = static_cast<ExchangeState *>(c->ext.exch);
    if (!x || !x->built || x->gen != c->gen)
        return fail(c, FDX_ESTATE, "no exchange lists built for the current particles");
    return FDX_OK;
}

}  // namespace

void exchange_release(fdx_ctx *c) {
    ExchangeState *x = static_cast<ExchangeState *>(c->ext.exch);
    if (!x) return;
    x->release();
    delete x;
    c->ext.exch = nullptr;
}

}  // namespace fdx

using namespace fdx;

extern "C" {

int fdx_build_exchange_lists(fdx_ctx *c, double theta, int32_t n_leaf) {
    FDX_ABI_TRY
    if (!c) return FDX_EINVAL;
    if (hipSetDevice(c->device) != hipSuccess) return fail(c, FDX_EHIP, "hipSetDevice failed");
    if (!c->have_particles) return fail(c, FDX_ESTATE, "no particles: call fdx_set_particles first");
    if (c->nsys < 2) return fail(c, FDX_EINVAL, "exchange lists need at least two domains");
    for (int s = 0; s < c->nsys; s++)
        if (c->sys_off_h[s + 1] == c->sys_off_h[s])
            return fail(c, FDX_EINVAL, "domain %d is empty", s);
    const size_t P = (size_t)c->nsys * (size_t)(c->nsys - 1);
    if (P > 0x7FFFFFFFull) return fail(c, FDX_EINVAL, "too many domains");
    // the local trees: keys, sort, cells, moments (and groups, unused here); softening is
    // not used by the lists
    const double eps = c->eps_given ? 0.0 : (c->eps_all > 0 ? c->eps_all : 1.0);
    int r = setup_eval(c, theta, n_leaf, kMaxGroup, eps, 0);
    if (r) return r;
    ExchangeState *x = state(c);
    x->built = false;
    hipStream_t s = c->stream;
    for (auto &e : x->ev)
        if (!e) HIPCHK(c, hipEventCreate(&e));
    HIPCHK(c, hipEventRecord(x->ev[0], s));
    r = run_tree(c, true);
    if (r) return r;
    finish_stats(c);
    HIPCHK(c, hipEventRecord(x->ev[1], s));

    const size_t G = exchange_subwalks(c->nsys);
    HIPCHK(c, x->box.ensure(6 * G));
    HIPCHK(c, x->start.ensure(G));
    HIPCHK(c, x->sel.ensure(G));
    HIPCHK(c, x->ne.ensure(G));
    HIPCHK(c, x->ns.ensure(G));
    HIPCHK(c, x->cap.ensure(G));
    HIPCHK(c, x->seg.ensure(G + 1));
    HIPCHK(c, x->total.ensure(1));
    HIPCHK(c, x->oe.ensure(G));
    HIPCHK(c, x->os.ensure(G));
    HIPCHK(c, x->sums.ensure(2));
    HIPCHK(c, x->pe.ensure(P));
    HIPCHK(c, x->ps.ensure(P));
    HIPCHK(c, x->nsel.ensure(1));
    HIPCHK(c, x->front.ensure((size_t)kExchangeFrontierMax * c->nsys));
    HIPCHK(c, x->fcount.ensure(c->nsys));
    const Cells cv = cells_view(c);
    const double th2 = c->theta * c->theta;
    HIPCHK(c, exchange_split(c->nsys, cv, c->bbox_u.p, c->cube.p, th2, x->front.p, x->fcount.p,
                             x->box.p, x->start.p, x->cap.p, x->sel.p, x->nsel.p, s));
    HIPCHK(c, fill_u32(x->ne.p, 0u, G, s));
    HIPCHK(c, fill_u32(x->ns.p, 0u, G, s));
    Groups pg{};
    pg.box = x->box.p;
    pg.sys = x->start.p;
    pg.cap = (uint32_t)std::min<size_t>(G, 0xFFFFFFFFu);
    // every list of sender s holds at most n_s entries (they cover disjoint sets of its
    // particles; so does each sub-walk within its start cell): with room for that bound in
    // every segment, one fill walk does; past the budget a count walk sizes them first
    const uint64_t bound = (uint64_t)(c->nsys - 1) * (uint64_t)c->n;
    const bool one_pass = bound * sizeof(uint32_t) <= kExchangeBudgetBytes;
    if (!one_pass) {
        HIPCHK(c, walk(false, G, pg, cv, th2, nullptr, nullptr, 0, nullptr, x->ne.p, x->ns.p,
                       nullptr, x->sel.p, x->nsel.p, c->st, s));
        HIPCHK(c, exchange_caps(G, x->sel.p, x->nsel.p, x->ne.p, x->ns.p, x->cap.p, s));
    }
    HIPCHK(c, scan_u32_to_u64(x->cap.p, x->seg.p, G, nullptr, nullptr, c->partial.p, x->total.p,
                              s));
    uint64_t total = bound;
    if (!one_pass) {
        HIPCHK(c, hipMemcpyAsync(&total, x->total.p, 8, hipMemcpyDeviceToHost, s));
        HIPCHK(c, hipStreamSynchronize(s));
    }
    if (total > x->list_cap || !x->list.p) {
        HIPCHK(c, x->list.ensure(total));
        x->list_cap = total;
    }
    HIPCHK(c, walk(true, G, pg, cv, th2, x->seg.p, x->cap.p, x->list_cap, x->list.p, x->ne.p,
                   x->ns.p, nullptr, x->sel.p, x->nsel.p, c->st, s));
    HIPCHK(c, hipEventRecord(x->ev[2], s));
    // where every slot's entries go in the pair-ordered lists, and the pairs' counts
    HIPCHK(c, scan_u32_to_u64(x->ne.p, x->oe.p, G, nullptr, nullptr, c->partial.p, x->sums.p, s));
    HIPCHK(c, scan_u32_to_u64(x->ns.p, x->os.p, G, nullptr, nullptr, c->partial.p, x->sums.p + 1,
                              s));
    HIPCHK(c, exchange_pairs(P, x->oe.p, x->os.p, x->sums.p, x->pe.p, x->ps.p, s));
    uint64_t sums[2];
    HIPCHK(c, hipMemcpyAsync(sums, x->sums.p, sizeof sums, hipMemcpyDeviceToHost, s));
    r = read_status(c);
    if (r) return r;
    const DevStatus &h = c->hst->st;
    if (h.walk_error || h.list_overflow)
        return fail(c, FDX_EHIP, "exchange walk did not complete (stack %u, overflow %u)",
                    h.walk_error, h.list_overflow);
    float t0 = 0, t1 = 0;
    HIPCHK(c, hipEventElapsedTime(&t0, x->ev[0], x->ev[1]));
    HIPCHK(c, hipEventElapsedTime(&t1, x->ev[1], x->ev[2]));
    x->n_epj = sums[0];
    x->n_spj = sums[1];
    x->entries = x->n_epj + x->n_spj;
    x->capacity = total;
    x->nsys = c->nsys;
    x->pairs = P;
    x->ms_tree = t0;
    x->ms_lists = t1;
    x->gen = c->gen;
    x->built = true;
    return FDX_OK;
    FDX_ABI_CATCH(c)
}

int fdx_get_exchange_counts(fdx_ctx *c, uint32_t *n_epj, uint32_t *n_spj) {
    FDX_ABI_TRY
    if (!c) return FDX_EINVAL;
    int r = check_built(c);
    if (r) return r;
    ExchangeState *x = static_cast<ExchangeState *>(c->ext.exch);
    const size_t S = (size_t)x->nsys, P = x->pairs;
    std::vector<uint32_t> pe(P), ps(P);
    HIPCHK(c, hipMemcpyAsync(pe.data(), x->pe.p, 4 * P, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipMemcpyAsync(ps.data(), x->ps.p, 4 * P, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    for (size_t s = 0; s < S; s++)
        for (size_t q = 0; q < S; q++) {
            const size_t k = s * (S - 1) + (q < s ? q : q - 1);
            if (n_epj) n_epj[s * S + q] = q != s ? pe[k] : 0u;
            if (n_spj) n_spj[s * S + q] = q != s ? ps[k] : 0u;
        }
    return FDX_OK;
    FDX_ABI_CATCH(c)
}

int fdx_get_exchange_lists(fdx_ctx *c, uint32_t *epj, uint32_t *spj) {
    FDX_ABI_TRY
    if (!c) return FDX_EINVAL;
    if (hipSetDevice(c->device) != hipSuccess) return fail(c, FDX_EHIP, "hipSetDevice failed");
    int r = check_built(c);
    if (r) return r;
    ExchangeState *x = static_cast<ExchangeState *>(c->ext.exch);
    // pair order on the device, then one copy per kind
    hipStream_t s = c->stream;
    const bool want_e = epj && x->n_epj, want_s = spj && x->n_spj;
    if (!want_e && !want_s) return FDX_OK;
    if (want_e) HIPCHK(c, x->out_e.ensure(x->n_epj));
    if (want_s) HIPCHK(c, x->out_s.ensure(x->n_spj));
    HIPCHK(c, exchange_gather(exchange_subwalks(x->nsys), x->sel.p, x->nsel.p, x->seg.p, x->cap.p,
                              x->ne.p, x->ns.p, x->oe.p, x->os.p, x->list.p, c->sperm,
                              want_e ? x->out_e.p : nullptr, want_s ? x->out_s.p : nullptr, s));
    if (want_e)
        HIPCHK(c, hipMemcpyAsync(epj, x->out_e.p, 4 * x->n_epj, hipMemcpyDeviceToHost, s));
    if (want_s)
        HIPCHK(c, hipMemcpyAsync(spj, x->out_s.p, 4 * x->n_spj, hipMemcpyDeviceToHost, s));
    HIPCHK(c, hipStreamSynchronize(s));
    return FDX_OK;
    FDX_ABI_CATCH(c)
}

int fdx_get_exchange_stats(fdx_ctx *c, fdx_exchange_stats *out) {
    FDX_ABI_TRY
    if (!c || !out) return FDX_EINVAL;
    int r = check_built(c);
    if (r) return r;
    ExchangeState *x = static_cast<ExchangeState *>(c->ext.exch);
    out->n_domains = x->nsys;
    out->n_pairs = (int64_t)x->pairs;
    out->n_epj = (int64_t)x->n_epj;
    out->n_spj = (int64_t)x->n_spj;
    out->list_capacity = (int64_t)x->capacity;
    out->ms_tree = x->ms_tree;
    out->ms_lists = x->ms_lists;
    return FDX_OK;
    FDX_ABI_CATCH(c)
}

}  // extern "C"
