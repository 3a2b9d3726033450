"""Asks csrc/plan.hpp, through a small host program built on first use, what a call is planned to run (test-side only)."""
from __future__ import annotations

import functools
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))


@functools.lru_cache(maxsize=1)
def _probe() -> str:
    from paper_2605_10453_amd import binding, build
    binding.load_library()
    exe = os.path.join(tempfile.mkdtemp(prefix="plan_probe_"), "plan_probe")
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", exe, os.path.join(HERE, "plan_probe.cpp"), build.LIB,
                    "-Wl,-rpath," + os.path.dirname(build.LIB), "-Wl,--allow-shlib-undefined"], check=True)
    return exe


def launch_plan(kind: str, rows: int, d: int, r: int, V: int) -> dict:
    """The matrix-core plan of one launch: resident, rows_per_block, gw (column blocks), nsr (records per row)."""
    out = subprocess.run([_probe()], input=f"{kind} {rows} {d} {r} {V}\n", capture_output=True, text=True, check=True).stdout
    return {k: int(v) for k, v in (f.split("=") for f in out.split())}
