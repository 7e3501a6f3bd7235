"""The far-field expansion inside captured leapfrog steps: every replay equals the eager step, for one
large system (count walk in the graph) and for several (segments sized per system, lists that
outgrow theirs moved to spare space and expanded there)."""
import numpy as np
import pytest

from paper_1601_03138_amd import fdx
from paper_1601_03138_amd import inputs as I

pytestmark = pytest.mark.gpu

DT = 1.0 / 1024.0


def sets(name):
    one = I.clustered(n_background=80001, n_clusters=8, n_per_cluster=10000, seed=21, eps=1e-3)
    if name == "one":
        return one
    return I.concat([I.plummer(3001, seed=22, eps=0.02), one, I.plummer(20011, seed=23, eps=0.01)])


@pytest.mark.parametrize("name,margin", [("one", 200), ("several", 200), ("several", 60)])
def test_replayed_steps_equal_eager_steps(name, margin):
    ps = sets(name)
    with fdx.Context(0) as a, fdx.Context(0) as b:
        for c in (a, b):
            c.set_particles(ps)
            c.calc_force(0.5, 8, 256, 0.0, quad=True, fp32=True, persistent=True)
        b.set_graph_list_margin(margin)
        for step in range(4):
            a.integrate(DT, 1)
            b.integrate(DT, 1, graph=True)
            near, ns = b.near_counts(), b.list_counts()[1]
            assert np.any(near < ns) and np.array_equal(a.near_counts(), near)
            # the state and forces of this step; eager work of another kind between the replays
            fa, fb = a.forces(), b.forces()
            sa, sb = a.particles(), b.particles()
            if step % 2:
                a.calc_density(fdx.CUT_FIXED, 0.05, None, 8, 64)
                b.calc_density(fdx.CUT_FIXED, 0.05, None, 8, 64)
            for x, y in zip(sa, sb):
                assert np.array_equal(x, y)
            assert np.array_equal(fa, fb)
        if margin < 100:
            assert b.stats()["list_spills"] + b.stats()["graph_recoveries"] > 0
