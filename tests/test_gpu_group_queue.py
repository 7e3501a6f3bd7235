"""Queues of the persistent kernels at group counts around their consumers: fewer groups than XCDs,
than workgroups, than waves, and more (groups of one particle), and queues of unequal cost.  Every
group is evaluated exactly as by the direct launch."""
import numpy as np
import pytest

from paper_1601_03138_amd import fdx
from paper_1601_03138_amd import inputs as I

pytestmark = pytest.mark.gpu


def sets(name):
    if name == "clustered":
        return I.clustered(n_background=3000, n_clusters=2, n_per_cluster=6000, seed=5), 4
    return I.uniform_cube(int(name), 3, 1e-2), 1


@pytest.mark.parametrize("name", ["1", "7", "8", "9", "2047", "2049", "5121", "20011", "clustered"])
@pytest.mark.parametrize("fp32", [False, True])
def test_every_group_is_evaluated_once(name, fp32):
    ps, n_group = sets(name)
    with fdx.Context(0) as ctx:
        ctx.set_particles(ps)
        out = {}
        for kw in ("direct", "persistent", "fused"):
            ctx.calc_force(0.8, 8, n_group, 0.0, quad=True, fp32=fp32,
                           persistent=kw == "persistent", fused=kw == "fused")
            out[kw] = ctx.forces()
    assert np.array_equal(out["persistent"], out["direct"])
    # the same interactions in another order: sums of at most 2^15 terms, each rounded to 2^-53
    # (rsqrt 4e-15), or FP32 separations relative to another tile; the potential also has the
    # self term m / eps, added and taken away
    tol = 1e-3 if fp32 else 1e-10
    scale = np.sqrt(np.mean(out["direct"] ** 2, axis=0)) + np.array([0, 0, 0, 1.0]) * np.max(ps.m / ps.eps)
    scale = np.maximum(scale, 1e-300)
    assert np.max(np.abs(out["fused"] - out["direct"]) / scale) <= tol
    if name != "1":
        assert np.all(np.any(out["fused"] != 0.0, axis=1))
