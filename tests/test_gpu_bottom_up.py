"""Bottom-up sums over the tree at the edges of their blocks: one block, two, the largest count that
one workgroup joins and one more, systems that end at a block boundary, empty systems.  Moments
against the oracle; largest radii per cell through the density with equal radii, which must find what
a fixed radius finds."""
import numpy as np
import pytest

import oracle as O
from paper_1601_03138_amd import fdx
from paper_1601_03138_amd import inputs as I

from parity_util import check_moments, check_tree

pytestmark = pytest.mark.gpu


def systems(sizes, seed):
    rng = np.random.default_rng(seed)
    ps = I.uniform_cube(int(np.sum(sizes)), seed, 1e-2)
    ps.m = rng.uniform(0.5, 1.5, ps.n) / ps.n
    ps.sys_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    return ps


SETS = {
    "1": [1],
    "8192": [8192],
    "8193": [8193],
    "12288": [12288],
    "64 blocks": [64 * 4096],
    "65 blocks": [64 * 4096 + 1],
    "97 blocks": [97 * 4096 - 5],
    "ends at boundaries": [4096, 4096, 1, 4095, 8192, 3],
    "empty systems": [0, 5000, 0, 0, 7288, 0, 4096, 0],
    "many systems": [7] * 3000,
}


@pytest.mark.parametrize("name", list(SETS))
@pytest.mark.parametrize("n_leaf", [1, 8])
def test_moments(name, n_leaf):
    ps = systems(SETS[name], 11)
    t = O.build_tree(ps, n_leaf)
    with fdx.Context(0) as ctx:
        ctx.set_particles(ps)
        ctx.calc_force(0.7, n_leaf, 64, 0.0, fp32=True)
        tree = ctx.tree()
    check_tree(tree, t)
    check_moments(tree["mom"], t)


@pytest.mark.parametrize("name", ["1", "8193", "ends at boundaries", "empty systems", "65 blocks"])
@pytest.mark.parametrize("mode", [1, 3])
def test_largest_radii(name, mode):
    ps = systems(SETS[name], 13)
    r = 0.3 / max(ps.n, 64) ** (1 / 3) * 4
    with fdx.Context(0) as ctx:
        ctx.set_particles(ps)
        ctx.calc_density(0, r, None, n_leaf=8, n_group=64)
        rho0, n0 = ctx.density()
        ctx.calc_density(mode, 0.0, np.full(ps.n, r), n_leaf=8, n_group=64)
        rho, nn = ctx.density()
    assert np.array_equal(nn, n0)
    assert np.max(np.abs(rho - rho0) / rho0) <= 1e-12
