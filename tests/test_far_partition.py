"""The schedule by which the far-field kernel partitions a superparticle list in place, compiled from
the library's header for the CPU: random and adversarial lists come out near entries first, no
unread slot is overwritten, and no more ids wait than the kernel's buffer holds."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1601_03138_amd", "csrc")
BLOCK = 128


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_schedule(tmp_path):
    exe = str(tmp_path / "far_partition_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "far_partition_check.cpp"), "-o", exe],
                   check=True)
    rng = np.random.default_rng(1)
    lists = []
    for ns in (1, 63, 64, 127, 128, 129, 255, 256, 257, 383, 384, 385, 511, 512, 513, 1000, 3001, 9999):
        i = np.arange(ns)
        blocks = rng.random(ns // BLOCK + 1) < 0.5
        lists += [i < 0, i >= 0, i < ns // 2, i >= ns // 2, i % 2 == 0, (i // BLOCK) % 2 == 0,
                  (i // BLOCK) % 3 == 0, (i // (2 * BLOCK)) % 2 == 1, blocks[i // BLOCK],
                  (i > BLOCK) & (i < ns - BLOCK), (i <= BLOCK) | (i >= ns - BLOCK)]
        lists += [rng.random(ns) < p for p in (0.01, 0.3, 0.5, 0.9)]
    text = "\n".join("".join("1" if f else "0" for f in far) for far in lists)
    out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout
    rows = out.strip().splitlines()
    assert len(rows) == len(lists)
    for far, row in zip(lists, rows):
        near, ids, most, wrong = row.split("|")
        ids = np.array(ids.split(), dtype=int)
        assert wrong == "0", (len(far), wrong)
        assert np.array_equal(np.sort(ids), np.arange(len(far)))
        assert int(near) == int((~far).sum())
        assert not far[ids[:int(near)]].any() and far[ids[int(near):]].all()
        assert int(most) <= 3 * BLOCK
