"""Builds libmpzch.so (gfx950) in-tree with hipcc.  `python -m paper_2602_17050_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "mpzch.hip")
LIB = os.path.join(HERE, "libmpzch.so")
NATIVE_SRC = os.path.join(HERE, "csrc", "native_call.cpp")
NATIVE = os.path.join(HERE, "_native.so")
CEIL_SRC = os.path.join(HERE, "csrc", "memory_ceilings.hip")
CEIL_BIN = os.path.join(HERE, "memory_ceilings.bin")


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def build_library(verbose: bool = False) -> str:
    """Compiles every time it is called (cross-compiles without a GPU)."""
    cmd = [hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Wall", "-Wno-unused-result",
           SRC, "-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(LIB + ".tmp", LIB)
    build_native(verbose)
    return LIB


def build_native(verbose: bool = False) -> str:
    """The module that marshals the repeated calls of the binding (host code; torch's headers, for its tensors and streams)."""
    import sysconfig
    import torch
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    rocm = os.path.dirname(os.path.dirname(hipcc())) if os.path.isabs(hipcc()) else "/opt/rocm"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-fvisibility=hidden",
           "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",               # what torch's stream header asks of a plain host compiler
           "-isystem", os.path.join(os.path.dirname(torch.__file__), "include"), "-isystem", os.path.join(rocm, "include"),
           "-isystem", sysconfig.get_paths()["include"],
           NATIVE_SRC, "-o", NATIVE + ".tmp", "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(NATIVE + ".tmp", NATIVE)
    return NATIVE


def build_memory_ceilings(verbose: bool = False) -> str:
    """Stand-alone tool that measures the random-access ceilings of the GPU it runs on."""
    cmd = [hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-result",
           CEIL_SRC, "-o", CEIL_BIN + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(CEIL_BIN + ".tmp", CEIL_BIN)
    return CEIL_BIN


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv))
    print(build_memory_ceilings(verbose="-v" in sys.argv))
