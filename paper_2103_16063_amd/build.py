"""Builds the HIP shared library in-tree for gfx950 (no JIT, no torch extension machinery):

    python -m paper_2103_16063_amd.build

The library exposes only the C ABI of include/rannc_dp.h."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librannc_dp.so")
SOURCES = ["rannc_dp_kernels.hip", "rannc_dp_split.hip", "rannc_dp_compact.hip", "rannc_dp_reach.hip", "rannc_dp_bound.hip", "rannc_dp_form.hip", "rannc_dp_api.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-fvisibility=hidden", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def build_library(verbose: bool = False, extra=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *extra, "-o", LIB] + [os.path.join(CSRC, s) for s in SOURCES]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    build_library(verbose=True, extra=sys.argv[1:])
    print("built", LIB)
