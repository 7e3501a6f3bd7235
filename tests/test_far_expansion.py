"""The far-field polynomial of the FP32 path (far_field.h, compiled for the CPU) against the pair terms
in FP64: error within the omitted degrees plus rounding, for monopoles, quadrupoles, softened terms
and sums of many."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1601_03138_amd", "csrc")
HIP = "/opt/rocm/include"


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(HIP, "hip")),
                    reason="needs g++ and the HIP headers")
def test_expansion_within_its_bound(tmp_path):
    exe = str(tmp_path / "far_expansion_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I", HIP, "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "far_expansion_check.cpp"), "-o", exe],
                   check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    rows = [r.split() for r in out.strip().splitlines()]
    assert len(rows) == 7
    for name, acc, pot in rows:
        assert float(acc) <= 1.0 and float(pot) <= 1.0, (name, acc, pot)
