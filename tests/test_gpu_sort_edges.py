"""The radix sort at the edges of its launches: one workgroup (up to 4096 and 8192 elements, four
and eight per thread), tiles of 4096 with look-back, one and several system-id digits.  Keys
and order against a stable host sort of the keys the tree reports."""
import numpy as np
import pytest

from paper_1601_03138_amd import fdx
from paper_1601_03138_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 65, 4095, 4096, 4097, 8191, 8192, 8193, 12288, 12289,
                               40961, 300007])
@pytest.mark.parametrize("n_sys", [1, 3, 257])
def test_order(n, n_sys):
    rng = np.random.default_rng(n + n_sys)
    ps = I.uniform_cube(n, 5, 0.01)
    if n > 100:                          # many equal keys
        for a in (ps.x, ps.y, ps.z):
            a[: n // 2] = np.round(a[: n // 2] * 8) / 8
    cut = np.sort(rng.integers(0, n + 1, n_sys - 1))
    ps.sys_off = np.concatenate([[0], cut, [n]]).astype(np.int64)
    with fdx.Context(0) as ctx:
        ctx.set_particles(ps)
        ctx.build_tree(8, 64)
        t = ctx.tree()
    sysid = np.repeat(np.arange(n_sys), np.diff(ps.sys_off))
    # quantised coordinates as the library defines them, per system
    key = np.zeros(n, np.uint64)
    for s in range(n_sys):
        a, b = ps.sys_off[s], ps.sys_off[s + 1]
        o, lr = t["cube"][s, :3], t["cube"][s, 3]
        q = [np.clip(np.floor((v[a:b] - o[k]) * (2097152.0 / lr)), 0, 2097151).astype(np.uint64)
             for k, v in enumerate((ps.x, ps.y, ps.z))]
        for bit in range(21):
            for k in range(3):
                key[a:b] |= ((q[k] >> np.uint64(bit)) & np.uint64(1)) << np.uint64(3 * bit + 2 - k)
    order = np.lexsort((np.arange(n), key, sysid))
    assert np.array_equal(t["perm"], order.astype(np.uint32))
    assert np.array_equal(t["key"], key[order])
