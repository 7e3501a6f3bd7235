"""Short-range kernels at the edges of their work mapping: groups of 1, of the sizes where the
runs of members change (16, 17, 32, 33, 80, 81, 160, 161) and of the largest size, with lists around
the 64- and 256-entry blocks.  TreePM cutoff forces and SPH density against the oracle."""
import numpy as np
import pytest

import oracle as O
from paper_1601_03138_amd import fdx
from paper_1601_03138_amd import inputs as I

from parity_util import F32_RMS_REL_VS_TREE

pytestmark = pytest.mark.gpu

SIZES = [1, 7, 16, 17, 32, 33, 80, 81, 160, 161, 512]


def clump(n, seed):
    """n particles in one leaf-sized clump (one group of n with n_group >= n) and a cloud."""
    rng = np.random.default_rng(seed)
    a = I.uniform_cube(n, seed, 1e-3, side=0.05)
    b = I.uniform_cube(257 + 3 * n, seed + 1, 1e-3, side=1.0)
    ps = I.concat([a, b])
    ps.sys_off = None
    for v in (ps.x, ps.y, ps.z):
        v[:n] += 0.21
    ps.m = rng.uniform(0.5, 1.5, ps.n) / ps.n
    return ps


def pull(ps, r_cut):
    """rms over the particles of the sum of m / (r^2 + eps^2) within r_cut (no cutoff function)."""
    d2 = sum((v[:, None] - v[None, :]) ** 2 for v in (ps.x, ps.y, ps.z))
    w = np.where(d2 < r_cut ** 2, ps.m[None, :] / (d2 + ps.eps[:, None] ** 2), 0.0)
    np.fill_diagonal(w, 0.0)
    return np.sqrt(np.mean(w.sum(axis=1) ** 2))


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("r_cut", [0.02, 0.3])
def test_cutoff_force(n, r_cut):
    ps = clump(n, 3 * n + 1)
    t = O.build_tree(ps, 8)
    g = O.make_groups(t, n)
    ref = np.empty((ps.n, 3))
    ref[t.perm.astype(np.int64)] = O.cutoff_lists(t, g, 0.5, r_cut).force()
    scale = np.sqrt(np.mean(np.sum(ref ** 2, axis=1)))
    f0 = pull(ps, r_cut)
    with fdx.Context(0) as ctx:
        ctx.set_particles(ps)
        out = {}
        for fp32 in (False, True):
            for pers in (False, True):
                ctx.calc_force_cutoff(0.5, 8, n, 0.0, r_cut, fp32=fp32, persistent=pers)
                out[fp32, pers] = ctx.forces()
            assert np.array_equal(out[fp32, False], out[fp32, True])
    # Each pair: g to 8 roundings of the oracle's Horner form, whose terms add to 293 at xi = 2
    # (2.6e-13 of the pull without g); FP32: separations to 3 x 2^-24 of groups of side 0.05, with
    # |xi dg/dxi| <= 2.5.  Then the sums.
    d64 = np.sqrt(np.mean(np.sum((out[False, False][:, :3] - ref) ** 2, axis=1)))
    d32 = np.sqrt(np.mean(np.sum((out[True, False][:, :3] - ref) ** 2, axis=1)))
    assert d64 <= 1e-12 * scale + 2.6e-13 * f0
    assert d32 <= F32_RMS_REL_VS_TREE * scale + 2.0 ** -20 * f0
    assert not out[False, False][:, 3].any() and not out[True, False][:, 3].any()


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("mode", [0, 1, 2, 3])
def test_density(n, mode):
    ps = clump(n, 5 * n + 2)
    h = 0.08 * np.random.default_rng(n).uniform(0.5, 2.0, ps.n) if mode else None
    ref, nref = O.density_brute(ps, h, mode, 0.1)
    with fdx.Context(0) as ctx:
        ctx.set_particles(ps)
        ctx.calc_density(mode, 0.1, h, n_leaf=8, n_group=n)
        rho, nn = ctx.density()
    assert np.array_equal(nn, nref)
    assert np.max(np.abs(rho - ref) / ref) <= 1e-12
