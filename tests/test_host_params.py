"""The host-side update's stores of the 16-bit parameters, on the CPU (tests/pins/host_params.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs the ROCm clang++")
@pytest.mark.parametrize("flags", [[], ["-DPT_HOST_NO_CLONES"]], ids=["clones", "plain"])
def test_same_bits_at_every_alignment_and_length(flags, tmp_path):
    exe = str(tmp_path / "host_params")
    cmd = [CLANG, "-std=c++17", "-O3", "-ffp-contract=off", "-fno-math-errno", "-pthread", *flags,
           "-I", os.path.join(ROOT, "paper_2406_08334_amd", "csrc"), os.path.join(ROOT, "tests", "pins", "host_params.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and "held" in run.stdout, run.stderr[-2000:]
