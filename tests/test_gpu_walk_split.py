"""Gravity walk at the edges of its split: groups of one particle around the size where a wave per
group becomes a wave per run of four, partial runs, and runs that straddle systems.  Lists against the
oracle's."""
import numpy as np
import pytest

import oracle as O
from paper_1601_03138_amd import fdx
from paper_1601_03138_amd import inputs as I

pytestmark = pytest.mark.gpu


def check(ps, n_group, theta):
    t = O.build_tree(ps, 8)
    g = O.make_groups(t, n_group)
    L = O.walk(t, g, theta)
    with fdx.Context(0) as ctx:
        ctx.set_particles(ps)
        ctx.calc_force(theta, 8, n_group, 0.0, quad=False)
        ne, ns, epj, spj = ctx.lists()
    assert np.array_equal(ne.astype(np.int64), L.n_epj) and np.array_equal(ns.astype(np.int64), L.n_spj)
    oe = np.concatenate([[0], np.cumsum(ne.astype(np.int64))])
    os_ = np.concatenate([[0], np.cumsum(ns.astype(np.int64))])
    for k in np.unique(np.r_[np.arange(min(g.n, 64)), np.linspace(0, g.n - 1, 200).astype(int)]):
        e_ref, s_ref = L.group_lists(int(k))
        assert np.array_equal(np.sort(epj[oe[k]:oe[k + 1]]), np.sort(e_ref))
        assert np.array_equal(np.sort(spj[os_[k]:os_[k + 1]]), np.sort(s_ref))
    return g.n


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 255, 16383, 16384, 16385])
def test_groups_of_one(n):
    assert check(I.uniform_cube(n, n, 1e-2), 1, 0.9) == n


@pytest.mark.parametrize("n_group", [3, 64])
def test_runs_across_systems(n_group):
    check(I.ensemble(9, 5, 301, 1700), n_group, 0.6)
