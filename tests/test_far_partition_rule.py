"""The in-place partition of a superparticle list (near entries first, far ones last) that the
far-field kernel makes while it reads the list in blocks from both ends: replayed step by step
on the host for random and adversarial lists."""
import numpy as np
import pytest

BLOCK, HELD = 128, 512              # entries read together; ids waiting per kind


def partition(lst, far):
    """The kernel's schedule: two blocks are chosen ahead; ids go back only into slots of blocks
    that are sorted in.  Returns (list, near count, most ids held of one kind)."""
    lst = list(lst)
    ns = len(lst)
    lo, hi = 0, ns
    held, room, put, most = [[], []], [0, 0], [0, 0], 0
    unread = np.ones(ns, bool)

    def choose(back):
        nonlocal lo, hi
        n = min(BLOCK, hi - lo)
        if back:
            hi -= n
            start = hi
        else:
            start = lo
            lo += n
        # the block's ids are read when it is chosen
        assert unread[start:start + n].all()
        return start, n, back, lst[start:start + n]

    b0, b1 = choose(0), choose(0)
    while b0[1]:
        start, n, back, ids = b0
        for v in ids:
            held[1 if far[v] else 0].append(v)
        unread[start:start + n] = False
        room[back] += n
        most = max(most, len(held[0]), len(held[1]))
        b2 = choose(1 if len(held[1]) > room[1] else 0)
        b0, b1 = b1, b2
        for c in (0, 1):
            k = min(len(held[c]), room[c])
            out = held[c][len(held[c]) - k:]
            del held[c][len(held[c]) - k:]
            for i, v in enumerate(out):
                slot = ns - 1 - (put[1] + i) if c else put[0] + i
                assert not unread[slot]                     # no unread entry is overwritten
                lst[slot] = v
            put[c] += k
            room[c] -= k
    for c in (0, 1):
        for i, v in enumerate(held[c]):
            lst[ns - 1 - (put[1] + i) if c else put[0] + i] = v
    return lst, put[0] + len(held[0]), most


@pytest.mark.parametrize("ns", [1, 63, 64, 127, 128, 129, 255, 256, 257, 511, 1000, 3001])
@pytest.mark.parametrize("kind", ["none", "all", "front", "back", "alternate", "blocks", "random"])
def test_partition(ns, kind):
    rng = np.random.default_rng(ns)
    i = np.arange(ns)
    far = {"none": i < 0, "all": i >= 0, "front": i < ns // 2, "back": i >= ns // 2,
           "alternate": i % 2 == 0, "blocks": (i // BLOCK) % 3 == 0,
           "random": rng.random(ns) < rng.random()}[kind]
    out, near, most = partition(i, far)
    assert sorted(out) == list(range(ns))
    assert near == int((~far).sum())
    assert not far[out[:near]].any() and far[out[near:]].all()
    assert most <= HELD
