"""What the library asks of the HIP runtime - launches, streams, events, copies - on a stand-in for it that writes the calls
down (tests/pins/fake_hip.h).  No GPU: the kernels don't run."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PINS = os.path.join(ROOT, "tests", "pins")
PKG = os.path.join(ROOT, "paper_2406_08334_amd")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    from paper_2406_08334_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2406_08334_amd import build
        build.build()
    out = str(tmp_path_factory.mktemp("host_calls") / "host_calls")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-rdynamic", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
           os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"), os.path.join(PINS, "host_calls.cpp"), "-o", out, "-L", PKG, "-lptchunk",
           "-Wl,-rpath," + PKG, "-Wl,--allow-shlib-undefined"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    return out


@pytest.mark.parametrize("check", [
    "captured_without_the_pack",
    "put_off_at_most_once",
    "finalize_on_a_stream_that_is_gone",
    "failed_launch_in_place",
    "overlapping_host_arrays",
    "host_update_beside_the_resident_one",
    "norm_occupancy_by_size",
    "unpack_occupancy_by_size",
    "accumulate_occupancy_by_size",
    "launch_shape_options_and_back",
    "plan_destroyed_and_its_reduction_fails",
    "side_streams_are_judged_by_their_own_steps",
    "recompute_and_norm_in_one_launch",
    "step_ends_with_its_constants",
    "step_end_in_a_graph",
    "captured_alone",
    "kept_in_the_cache_by_size",
    "unpack_kept_by_size",
    "norm_counters_of_two_devices",
    "norm_without_a_context_captured",
    "steps_that_go_on_behind_an_update",
    "sequences_at_random",
])
def test_calls(exe, check):
    res = subprocess.run([exe, check], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, (res.stdout + res.stderr)[-6000:]
