"""Build libptchunk.so for gfx950 with hipcc (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libptchunk.so")
PROBE = os.path.join(HERE, "ptchunk_probe")
CALL = os.path.join(HERE, "_ptcall" + sysconfig.get_config_var("EXT_SUFFIX"))      # of this interpreter: no other loads it
SOURCES = ["pt_ctx.hip", "pt_norm.hip", "pt_pack.hip", "pt_accum.hip", "pt_adamw.hip", "pt_stream.hip", "pt_host.hip", "pt_model.hip"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off",                     # the fp32 sequence of the update is written out FMA by FMA
    "-fno-fast-math",
    "-fno-math-errno",                       # lets the host-side update loop vectorise its sqrt
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def build(verbose: bool = False) -> str:
    """Compiles every HIP source into one shared library, every time it is called."""
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    cmd = [hipcc()] + FLAGS + ["-o", LIB] + srcs
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # hipcc's host pass warns that it does not know the packed-fp32 feature: harmless
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed")
    if verbose and err.strip():
        print(err)
    # the Python-free driver of the C ABI (used under rocprofv3 for hardware counters)
    cmd = [hipcc(), "--offload-arch=gfx950", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), os.path.join(CSRC, "pt_probe.cpp"),
           "-o", PROBE, "-L", HERE, "-lptchunk", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed on pt_probe.cpp")
    build_call(verbose)
    return LIB


def build_call(verbose: bool = False):
    """Compiles the step's calls from Python (host code only; the library's entry points are handed to it when it is loaded).  Without a C++
    compiler or CPython's headers there is none, and ctypes takes those calls."""
    include = sysconfig.get_paths()["include"]
    cxx = shutil.which("g++") or shutil.which("/opt/rocm/llvm/bin/clang++")
    if os.path.exists(CALL):
        os.remove(CALL)                      # none rather than an old one
    if cxx is None or not os.path.exists(os.path.join(include, "Python.h")):
        sys.stderr.write("no C++ compiler or no Python.h: without native marshalling\n")
        return None
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-Wextra", "-I", os.path.join(ROOT, "include"),
           "-I", include, os.path.join(CSRC, "pt_call.cpp"), "-o", CALL]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("the C++ compiler failed on pt_call.cpp")
    return CALL


if __name__ == "__main__":
    print(build(verbose=True))
