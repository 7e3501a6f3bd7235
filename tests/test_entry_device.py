"""Entry points that allocate device memory or launch kernels do so on their context's device,
whichever device the calling thread has current (checked on the CPU, on the host sources linked
to a HIP runtime of host memory)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1601_03138_amd", "csrc")
HIP = "/opt/rocm/include"


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(HIP, "hip")),
                    reason="needs g++ and the HIP headers")
def test_entry_points_use_their_contexts_device(tmp_path):
    exe = str(tmp_path / "entry_device_check")
    srcs = [os.path.join(ROOT, "tests", "native", "entry_device_check.cpp"),
            os.path.join(CSRC, "capi.cpp"), os.path.join(CSRC, "predictor.cpp")]
    # what the tested entry points do not reach stays unresolved
    subprocess.run(["g++", "-std=c++17", "-O0", "-w", "-D__HIP_PLATFORM_AMD__", "-I", HIP, "-I", CSRC]
                   + srcs + ["-Wl,--unresolved-symbols=ignore-all", "-o", exe], check=True)
    out = subprocess.run([exe, str(tmp_path / "weights.bin")], check=True, capture_output=True,
                         text=True).stdout
    rows = [r.split("|") for r in out.strip().splitlines()]
    assert len(rows) == 9
    for name, status, good, bad in rows:
        assert status == "0", name
        assert int(good) > 0 and bad == "0", (name, good, bad)
