"""Far superparticles of the FP32 path (one polynomial per group) against the FP64 kernels on
the same lists, per particle, within the FP32 rounding bounds plus the omitted Taylor terms; the
lists stay the oracle's sets."""
import math

import numpy as np
import pytest

import oracle as O
from paper_1601_03138_amd import fdx
from paper_1601_03138_amd import inputs as I

pytestmark = pytest.mark.gpu

RATIO, RATIO3 = 24.0, 64.0      # far, very far: |X| > ratio x the group's radius


def bounds(t, g, k, lists, q, ref):
    """Bound on |da| of the members of group k (lists.group_lists(q) is its list), three parts.

    Pair terms, as parity_util.fp32_error_bound: coordinates relative to the group's centre are
    rounded to FP32 (u = 2^-24), |da| <= sum m / r_eff^2 (3 sqrt(3) u (|x_i - c| + |x_j - c|) / r_eff
    + 8 u).
    Tile sums: a 512-thread workgroup cuts a 512-entry tile into floor(512 / n_i) slices and adds
    at most L = 512 / slices + 1 terms plainly, L u sum m / r_eff^2.
    Omitted terms of the expansion about the box centre of superparticles farther than RATIO radii:
    with h = radius / R, sum over n >= 5 (n >= 4 beyond RATIO3) of n h^(n-1) of M / R^2, and of the
    quadrupole's |Q| / (2 R^4) with the Gegenbauer coefficients C^{5/2}_n <= binomial(n + 4, 4),
    times (1 + h)^2 for its form about the member and 4 for the products it is expanded in."""
    u = 2.0 ** -24
    pos = np.stack([t.sx, t.sy, t.sz], axis=1)
    b, m = int(g.begin[k]), int(g.count[k])
    e, s = (v.astype(np.int64) for v in lists.group_lists(q))
    mom, c = t.mom[s], g.centre[k]
    xj = np.concatenate([pos[e], mom[:, 1:4]]) - c
    mj = np.concatenate([t.sm[e], mom[:, 0]])
    xi = pos[b:b + m] - c
    d = xj[None] - xi[:, None]
    reff = np.sqrt(np.sum(d * d, axis=2) + (t.seps[b:b + m] ** 2)[:, None])
    dd = math.sqrt(3.0) * u * (np.linalg.norm(xi, axis=1)[:, None] + np.linalg.norm(xj, axis=1)[None])
    pair = mj / reff ** 2 * (3.0 * dd / reff + 8.0 * u)
    pair[:, :len(e)][e[None] == np.arange(b, b + m)[:, None]] = 0.0
    total = pair.sum(axis=1) + (512 // (512 // m) + 1) * u * (mj / reff ** 2).sum(axis=1)
    sys = t.csys[g.cell[k]]
    unit = t.cube[sys, 3] / 2.0 ** 21                             # grid unit
    lo = t.cube[sys, :3] + unit * g.qmin[k]
    hi = t.cube[sys, :3] + unit * (g.qmax[k].astype(np.int64) + 1)
    rad = 0.5 * np.linalg.norm(hi - lo)
    R = np.linalg.norm(mom[:, 1:4] - 0.5 * (lo + hi), axis=1)
    for ratio, first in ((RATIO, 5), (RATIO3, 4)):
        far = R > ratio * rad * (1 - 1e-6)
        n = np.arange(first, first + 1 if first == 4 else 40)
        h = rad / R[far]
        qq = mom[far, 4:]
        qn = np.sqrt((qq[:, :3] ** 2).sum(1) + 2 * (qq[:, 3:] ** 2).sum(1))
        pw = h[:, None] ** (n - 1)[None]
        mono = (n * pw).sum(1)
        quad = (n * np.array([math.comb(int(v) + 4, 4) for v in n]) * pw).sum(1) * 4 * (1 + h) ** 2
        total = total + (mom[far, 0] / R[far] ** 2 * mono + 0.5 * qn / R[far] ** 4 * quad).sum()
    return total, int((R > RATIO * rad).sum())


def sets(name):
    if name == "clustered":
        return I.clustered(n_background=80011, n_clusters=6, n_per_cluster=10003, seed=5, eps=1e-3)
    if name == "two":                   # a large system, and one too shallow to be expanded
        return I.concat([I.clustered(n_background=76001, n_clusters=6, n_per_cluster=10001, seed=6,
                                     eps=2e-3), I.plummer(3001, seed=7, eps=0.02)])
    ps = I.clustered(n_background=80000, n_clusters=6, n_per_cluster=10000, seed=8, eps=1e-3)
    ps.eps = ps.eps * np.random.default_rng(9).uniform(0.5, 2.0, ps.n)   # no shared softening
    return ps


@pytest.mark.parametrize("name,n_group,theta,quad", [
    ("clustered", 64, 0.4, True), ("clustered", 256, 0.5, True), ("clustered", 512, 0.7, True),
    ("clustered", 256, 0.4, False), ("two", 200, 0.5, True), ("eps", 256, 0.5, True)])
def test_far_field(name, n_group, theta, quad):
    ps = sets(name)
    t = O.build_tree(ps, 8)
    g = O.make_groups(t, n_group)
    rng = np.random.default_rng(3)
    sel = np.sort(rng.choice(g.n, 150, replace=False, p=g.count / g.count.sum()))
    lists = O.walk(t, g, theta, sel)
    with fdx.Context(0) as ctx:
        ctx.set_particles(ps)
        ctx.calc_force(theta, 8, n_group, 0.0, quad=quad, fp32=False)
        a64 = ctx.forces()[t.perm]
        ctx.calc_force(theta, 8, n_group, 0.0, quad=quad, fp32=True)
        a32 = ctx.forces()[t.perm]
        ne, ns, epj, spj = ctx.lists()
        ctx.calc_force(theta, 8, n_group, 0.0, quad=quad, fp32=True, persistent=True)
        pers = ctx.forces()[t.perm]
    assert np.array_equal(a32, pers)
    # the reordered lists are the same sets
    oe = np.concatenate([[0], np.cumsum(ne.astype(np.int64))])
    os_ = np.concatenate([[0], np.cumsum(ns.astype(np.int64))])
    nfar = 0
    for q, k in enumerate(sel):
        e, s = lists.group_lists(q)
        assert np.array_equal(np.sort(epj[oe[k]:oe[k + 1]]), np.sort(e))
        assert np.array_equal(np.sort(spj[os_[k]:os_[k + 1]]), np.sort(s))
        b, m = int(g.begin[k]), int(g.count[k])
        bound, far = bounds(t, g, k, lists, q, a64)
        nfar += far
        err = np.linalg.norm((a32 - a64)[b:b + m, :3], axis=1)
        assert np.all(err <= bound), (k, float((err / bound).max()))
        assert np.max(np.abs(a32[b:b + m, 3] / a64[b:b + m, 3] - 1)) < 1e-5
    assert nfar > 1000
