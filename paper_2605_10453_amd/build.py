"""Compile the HIP sources in csrc/ for gfx950 into libslimspec.so (in-tree, next to this file)."""
from __future__ import annotations

import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libslimspec.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 code generation
    # MFMA results in vector registers.  A condition of correctness, not a preference: head_resident_kernel<32> keeps its row
    # operand in the 128 accumulation registers it has, and without this it also accumulates there and spills 80 bytes per
    # lane; the kernel counts its own vector loads (s_waitcnt vmcnt(N)), which spills would falsify.  A test holds every
    # instance to no scratch memory.  Of the other kernels it changes down_tile_kernel only (no accumulation registers).
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
    # The first words of a kernel's arguments arrive in scalar registers with its blocks instead of by a load that every block
    # waits for: 0.1 to 0.2 us a launch, and a call is two to six launches (one row, d = 4096, r = 512, V = 128256 34.4 -> 33.9 us,
    # 3 rows, d = 5264, r = 496, V = 19072 25.8 -> 24.9).  Only pointers and numbers are taken, up to the first struct.
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build_library(verbose: bool = True, extra_flags=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *extra_flags, "-o", LIB, *sources()]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    build_library(extra_flags=sys.argv[1:])
