"""Builds libsigattn.so (HIP, gfx950 only) in-tree with hipcc.  No JIT, no fallback."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsigattn.so")
SOURCES = ["sigattn_api.hip"]
PROBE_LIB = os.path.join(HERE, "libmachine_probes.so")  # measurement aids for the benchmark, a library of their own
PROBE_SOURCES = ["machine_probes.hip"]

FASTCALL = os.path.join(HERE, "_fastcall.so")            # the binding's plain calls in native code (host only)

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed-fp32 VALU forms are switched off for every device function of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found: libsigattn needs the ROCm toolchain")
    return exe


def _compile(lib: str, sources, verbose: bool) -> str:
    cmd = [hipcc(), *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", lib,
           *[os.path.join(CSRC, s) for s in sources]]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if verbose or res.returncode != 0:
        print(" ".join(cmd))
        print(res.stdout)
        print(res.stderr)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed building {os.path.basename(lib)}")
    return lib


def _compile_fastcall(verbose: bool) -> None:
    if os.path.exists(FASTCALL):
        os.remove(FASTCALL)                     # one of other sources or of another torch is worse than none
    import sysconfig
    import torch
    root = os.path.dirname(torch.__file__)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", sysconfig.get_paths()["include"], "-isystem", os.path.join(root, "include"),
           "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-isystem", os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc()))), "include"),
           "-o", FASTCALL, os.path.join(CSRC, "fastcall.cpp"),
           "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if verbose or res.returncode != 0:
        print(" ".join(cmd))
        print(res.stdout)
        print(res.stderr)
    if res.returncode != 0:
        raise RuntimeError("g++ failed building _fastcall.so")


def build_library(verbose: bool = False) -> str:
    """libsigattn.so (the method), _fastcall.so (its plain calls from torch) and libmachine_probes.so (the benchmark's
    measurement aids).  The two libraries need hipcc and nothing else.  _fastcall.so needs torch, its and Python's headers and
    g++: without them the binding makes every call in Python, with the same results and 3 to 5 us more of host work, and
    this function says so and goes on."""
    _compile(PROBE_LIB, PROBE_SOURCES, verbose)
    _compile(LIB, SOURCES, verbose)
    try:
        _compile_fastcall(verbose)
    except (ImportError, OSError, RuntimeError) as e:
        print(f"_fastcall.so was not built ({type(e).__name__}: {e}): plain calls will be made in Python", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
