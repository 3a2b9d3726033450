"""The down-projections of several rows (csrc/down_tile.hip, csrc/down_rows.hip) where the hidden size is no multiple of their
32-element stages: the last stage holds 8, 16 or 24 elements, alone or after full ones, in a slice of its own or at the end of
one.  And ranks that are no multiples of a block's columns, rows in one, two and three tiles, groups of rows."""
import numpy as np
import pytest

from paper_2605_10453_amd import synth
from parity_util import compare_with_oracle, to_dev_bf16
from test_gpu_parity import gpu  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu

FP32_TOL = 6e-5      # up to 48 rows t stays in fp32: see test_gpu_rows_head.py
LOGPROB_TOL = 2e-2   # more rows: t travels as 16 bits


@pytest.mark.parametrize("d", [8, 24, 40, 64 + 8, 7 * 32 + 16, 1024 + 24, 4064 + 8])
@pytest.mark.parametrize("rows,r", [(6, 8), (17, 72), (40, 264), (70, 40), (150, 136)])
def test_ragged_hidden_size(gpu, oracle_mod, rows, r, d):
    torch, b = gpu
    print(f"down-projection: rows={rows} d={d} r={r}", flush=True)
    V, k = 1000, 4
    x = synth.make_inputs(synth.small_config(rows, d, r, V, k, peaked_every=4), seed=rows + d)
    # (what lies behind the last row and column of h and A must not matter: both end at an allocation of their own)
    ids, lp = b.slimspec_head_topk(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B), k)
    torch.cuda.synchronize()
    ora = oracle_mod.slimspec_head_topk(x.h, x.A, x.B, k)
    z_at = lambda ri, ci: oracle_mod.slimspec_logits_at(x.h, x.A, x.B, ri, ci)
    tol = dict(tie_tol=FP32_TOL, lp_tol=FP32_TOL) if rows <= 48 else dict(lp_tol=LOGPROB_TOL)
    compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V, **tol)


@pytest.mark.parametrize("r,d", [(72, 104), (256, 1024), (24, 2040), (272, 264)])
@pytest.mark.parametrize("off", [[0, 7, 7, 30, 41], [0, 0, 3], [0, 33, 48]])
def test_ragged_hidden_size_with_a_matrix_per_position(gpu, r, d, off):
    """Every position's rows as a call of their own with that position's matrix (other row tiles, other kernels for one row)."""
    torch, b = gpu
    V, k = 4104, 5
    x = synth.make_inputs(synth.small_config(off[-1], d, r, V, k), seed=3)
    A = [synth.make_inputs(synth.small_config(1, d, r, V, k), seed=10 + p).A for p in range(len(off) - 1)]
    h, B = to_dev_bf16(x.h), to_dev_bf16(x.B)
    stack = torch.stack([to_dev_bf16(a) for a in A]).contiguous()
    ids, lp = b.slimspec_head_topk_positions(h, stack, off, B, k)
    for p in range(len(off) - 1):
        lo, hi = off[p], off[p + 1]
        if lo == hi:
            continue
        want_ids, want_lp = b.slimspec_head_topk(h[lo:hi].contiguous(), stack[p].contiguous(), B, k)
        torch.cuda.synchronize()
        assert np.abs((lp[lo:hi] - want_lp).cpu().numpy()).max() <= FP32_TOL
        assert torch.equal(ids[lo:hi], want_ids)
