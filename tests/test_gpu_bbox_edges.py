"""Bounding boxes at the edges of their chunks (1024 particles up to 65536, then 4096): systems that
end at, before and behind a chunk's edge, several in one chunk, empty ones.  Cubes and keys against
the oracle, exact."""
import numpy as np
import pytest

import oracle as O
from paper_1601_03138_amd import fdx
from paper_1601_03138_amd import inputs as I

pytestmark = pytest.mark.gpu

SETS = {
    "one": [1025],
    "edges": [1023, 1, 1024, 1025, 1023],
    "several in a chunk": [5, 300, 0, 300, 2, 400, 900, 3],
    "small maximum": [60000, 5536],
    "past it": [60000, 5537, 4095, 1, 4096, 4097, 0, 2],
}


@pytest.mark.parametrize("name", list(SETS))
def test_cubes_and_keys(name):
    sizes = SETS[name]
    ps = I.uniform_cube(int(np.sum(sizes)), 17, 1e-2)
    ps.sys_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    for k in range(len(sizes)):                  # boxes of different places and sizes
        r = slice(ps.sys_off[k], ps.sys_off[k + 1])
        ps.x[r] = ps.x[r] * (k + 1.0) - 3.0 * k
        ps.y[r] -= 0.25 * k
    t = O.build_tree(ps, 8)
    with fdx.Context(0) as ctx:
        ctx.set_particles(ps)
        ctx.calc_force(0.7, 8, 64, 0.0, fp32=True)
        tree = ctx.tree()
    assert np.array_equal(tree["cube"], t.cube)
    assert np.array_equal(tree["key"], t.skey)
