"""Builds libhermite.so (gfx950) in-tree with hipcc.

    python -m paper_1104_2700_amd.build

Flags: -O3, C++17, --offload-arch=gfx950, and packed-FP32 instructions
disabled (-Xclang -target-feature -Xclang -packed-fp32-ops): every FP32
operation of the mixed-precision sweep is issued as a plain VALU op.
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhermite.so")
SOURCES = ["hermite_lib.hip", "sweep.hip", "pairs.hip", "integrate.hip",
           "smallrun.hip", "midrun.hip"]
ARCH = os.environ.get("HERMITE_OFFLOAD_ARCH", "gfx950")


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def build(verbose: bool = False) -> str:
    """Compile every HIP source into libhermite.so; returns its path."""
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc(), "--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Wall", "-Wno-unused-result",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           "-o", tmp] + [os.path.join(CSRC, s) for s in SOURCES]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
