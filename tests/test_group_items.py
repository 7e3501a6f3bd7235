"""Work items of the kernels that take groups in a fixed order (group_items.h, compiled for the CPU):
every item is taken once, few groups are split until the chip has work or they cannot be, and
no XCD gets much more of them than the others."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1601_03138_amd", "csrc")
ITEMS = {"density": (16384, lambda n_group: -(-n_group // 16)),
         "cut": (16384, lambda n_group: -(-n_group // 80))}


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_items(tmp_path):
    exe = str(tmp_path / "group_items_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "group_items_check.cpp"), "-o", exe],
                   check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    seen = set()
    for row in out.strip().splitlines():
        head, parts, once, items, spread = row.split("|")
        kernel, groups, n_group = head.split()
        want, most = ITEMS[kernel]
        groups, parts, most = int(groups), int(parts), most(int(n_group))
        assert int(once) == int(items) == groups * parts, row
        assert parts == most or groups * parts >= want, row
        assert 1 <= parts <= most and (parts == 1 or groups * (parts - 1) < want), row
        if int(items) >= 512:
            assert float(spread) < 1.1, row
        seen.add(kernel)
    assert seen == set(ITEMS)
