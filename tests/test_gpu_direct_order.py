"""Order of the direct launches over the XCDs at the group counts where the length of a run changes
(128 groups per unit of it, up to 16 or 64) and at counts that are no multiple of it: every group is
evaluated, exactly as by the persistent launch."""
import numpy as np
import pytest

from paper_1601_03138_amd import fdx
from paper_1601_03138_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 9, 255, 256, 257, 1025, 2047, 2048, 2049, 8191, 8193, 20001])
def test_groups_of_one(n):
    ps = I.uniform_cube(n, 7, 1e-2)
    with fdx.Context(0) as ctx:
        ctx.set_particles(ps)
        for kw in (dict(fp32=True), dict(fp32=False)):
            out = []
            for persistent in (False, True):
                ctx.calc_force(0.9, 8, 1, 0.0, quad=True, persistent=persistent, **kw)
                out.append(ctx.forces())
                ctx.calc_force_cutoff(0.9, 8, 1, 0.0, 0.2, persistent=persistent, **kw)
                out.append(ctx.forces())
            assert np.array_equal(out[0], out[2]) and np.array_equal(out[1], out[3])
            if n > 1:
                assert np.all(np.any(out[0] != 0.0, axis=1))
