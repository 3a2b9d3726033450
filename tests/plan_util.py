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


def plan_of(kind: str, rows: int, d: int, r: int, V: int, k: int, fp32=False, prepared=False, sampling=False) -> dict:
    """What a call runs.  kernel: stream, rows, tile or resident; and, for the last two, f16 (operands), rows_per_block,
    col_blocks, records (per row and column block), parks (rows that wait for their exact columns), parked_offset and
    parked_row_bytes (where in the workspace a row does, its number of columns first); resident_fits; for stream, chunk_cols,
    rows_in_lds (whether a launch's row input fits shared memory), own_input (the kernel makes t itself) and block_tail (all
    wavefronts of a block finish its only row);
    for rows, reads_ahead (MB of the weights that the launches which make t read ahead, at most), slices_meet (how the sums of the slices of the contraction meet: one, at_once, halves or in_turn), sum_slices (slices of t that its blocks add, 0: none) and rows_as_they_lie (the full head's rows are read without a launch that regroups them); for stream and rows, merge (how merge_kernel takes the chunks' lists: short,
    long_ahead or long)."""
    line = f"{kind} {rows} {d} {r} {V} {k} {int(fp32)} {int(prepared)} {int(sampling)}\n"
    out = subprocess.run([_probe()], input=line, capture_output=True, text=True, check=True).stdout
    fields = dict(f.split("=") for f in out.split())
    return {key: v if key in ("kernel", "merge", "slices_meet") else int(v) for key, v in fields.items()}


def assert_plan(kind: str, rows: int, d: int, r: int, V: int, k: int, fp32=False, prepared=False, sampling=False, **expected):
    """A test that is about one kernel or branch says so, and fails when a later rule sends its shape elsewhere."""
    plan = plan_of(kind, rows, d, r, V, k, fp32, prepared, sampling)
    assert {key: plan[key] for key in expected} == expected, plan
