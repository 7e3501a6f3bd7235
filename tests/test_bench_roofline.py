"""Host-side logic of bench.py's roofline entry (no GPU): it counts the work that is executed, its
traffic includes the far-field kernel, and a change of any source of the force phase retires a
committed traffic figure."""
import os
import shutil
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

CSRC = os.path.join("paper_1601_03138_amd", "csrc")


def test_executed_flops():
    st = {"n_interactions_pp": 1000, "n_interactions_pc": 2 * 30 + 5 * 40 + 7 * 50}
    count, n_spj = [2, 5, 7], [30, 40, 50]
    # nothing expanded: the listed work
    assert bench.executed_flops(st, True, n_spj, n_spj, count) == bench.force_flops(st, True)
    assert bench.executed_flops(st, False, n_spj, n_spj, count) == bench.force_flops(st, False)
    # ten of the second group's and all of the third's superparticles far
    got = bench.executed_flops(st, True, [30, 30, 0], n_spj, count)
    assert got == 1000 * 20 + (2 * 30 + 5 * 30) * 54 + 60 * 374 + 12 * 205
    got = bench.executed_flops(st, False, [30, 30, 0], n_spj, count)
    assert got == 1000 * 20 + (2 * 30 + 5 * 30) * 20 + 60 * 231 + 12 * 205


def test_traffic_includes_the_far_kernel_and_ends_with_its_sources(tmp_path, monkeypatch):
    root = tmp_path / "root"
    shutil.copytree(os.path.join(ROOT, CSRC), root / CSRC)
    (root / "profiles").mkdir()
    monkeypatch.setattr(bench, "ROOT", str(root))
    sha = bench.force_source_sha()
    (root / "profiles" / "force_x_s_traffic.txt").write_text(
        f"hbm bytes per launch: 7.0e9\nfar-field kernel hbm bytes per launch: 2.5e9\nshape: s\n"
        f"launch: persistent\nforce kernel sources sha256: {sha}\n")
    assert bench.read_traffic("force_x", "s", "persistent") == 9.5e9
    for name in ("k_far.hip", "far_field.h", "group_queue.h", "dev_util.h", "k_force.hip"):
        path = root / CSRC / name
        text = path.read_text()
        path.write_text(text + "\n// changed\n")
        assert bench.read_traffic("force_x", "s", "persistent") is None, name
        path.write_text(text)
    assert bench.read_traffic("force_x", "s", "persistent") == 9.5e9
