"""Compile the HIP sources in csrc/ for gfx950 into libslimspec.so (in-tree, next to this file)."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libslimspec.so")

KERNARG_PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=16"]
# Sources compiled without it.  merge_streams_kernel keeps most of its two dozen arguments to the end, and the registers they arrive in are then
# not the ones the compiler would use: calls of more than 48 rows take 0.3 to 1 % longer with it (183 calls with / without, geometric means: full head 1.003, plain
# low-rank head 1.005, with prepared weights 1.010, in positions 1.008, sampling 1.000 to 1.003).  head_tile.hip without it: 1.002 and 0.999.
WITHOUT_PRELOAD = ("merge_streams.hip",)

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
    *KERNARG_PRELOAD,
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def flags_of(source: str) -> list:
    """The flags that one source is compiled with."""
    if os.path.basename(source) not in WITHOUT_PRELOAD:
        return list(HIPCC_FLAGS)
    at = HIPCC_FLAGS.index(KERNARG_PRELOAD[1])
    return HIPCC_FLAGS[:at - 1] + HIPCC_FLAGS[at + 1:]


def build_library(verbose: bool = True, extra_flags=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as objects:
        def compile_one(source):
            out = os.path.join(objects, os.path.basename(source) + ".o")
            cmd = [hipcc, *(f for f in flags_of(source) if f != "-shared"), *extra_flags, "-c", "-o", out, source]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return out
        with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
            built = list(pool.map(compile_one, sources()))
        link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *built]
        if verbose:
            print(" ".join(link), flush=True)
        subprocess.run(link, check=True)
    return LIB


if __name__ == "__main__":
    build_library(extra_flags=sys.argv[1:])
