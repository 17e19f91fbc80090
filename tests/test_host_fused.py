"""Which updates take the step's scalar work along in their own launch (tests/pins/host_fused.cpp).  No GPU."""
import os
import subprocess

import pytest

from paper_2406_08334_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2406_08334_amd")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not os.path.exists(binding.LIB_PATH):
        build.build()
    out = str(tmp_path_factory.mktemp("host_fused") / "host_fused")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-rdynamic", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
           os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "pins", "host_fused.cpp"), "-o", out, "-L", PKG, "-lptchunk",
           "-Wl,-rpath," + PKG, "-Wl,--allow-shlib-undefined"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    return out


@pytest.mark.parametrize("check", ["by_size", "not_otherwise", "not_with_host_threads", "sums_it_does_not_take", "failed_launch"])
def test_fused_updates(exe, check):
    res = subprocess.run([exe, check], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, (res.stdout + res.stderr)[-6000:]
