"""The lane-owns-columns kernel (stream_topk_kernel) against the CPU fp64 checker, at the edges of its chunks and of the way a block
shares the contraction: chunks of 64 to 512 columns, 1 to 8 rows of the weights at a time, blocks of 4 to 16 wavefronts,
wavefronts and lane groups without rows, row inputs that shared memory does not hold."""
import numpy as np
import pytest

from paper_2605_10453_amd import synth
from parity_util import compare_with_oracle, to_dev_bf16, to_dev_f32
from plan_util import assert_plan
from test_gpu_parity import gpu  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu

FP32_TOL = 6e-5      # fp32 sums of exact products: see test_gpu_rows_head.py


@pytest.mark.parametrize("rows,d,r,V,k", [
    (1, 64, 8, 8, 3), (1, 64, 8, 64, 64), (1, 72, 16, 72, 5), (1, 128, 40, 16384, 7), (1, 128, 72, 16392, 10), (1, 264, 136, 32776, 9),
    (1, 64, 264, 37208, 4), (1, 512, 320, 65544, 12), (1, 96, 104, 103472, 5), (1, 64, 24, 131072, 40), (1, 64, 48, 131080, 6),
    (1, 64, 16, 262152, 5), (1, 64, 8, 530000, 3), (1, 4096, 1032, 2056, 10), (1, 4096, 8, 4104, 33), (1, 64, 5000, 1000, 5),
    (2, 520, 56, 20000, 11), (2, 1000, 1000, 520, 6), (2, 2048, 24, 131072, 9), (3, 64, 264, 9000, 17), (4, 2048, 264, 40008, 64), (4, 64, 264, 8, 8),
])
def test_low_rank(gpu, oracle_mod, rows, d, r, V, k):
    torch, b = gpu
    print(f"stream kernel, low-rank: rows={rows} d={d} r={r} V={V} k={k}", flush=True)
    assert_plan("low", rows, d, r, V, k, kernel="stream")
    x = synth.make_inputs(synth.small_config(rows, d, r, V, k, peaked_every=2), seed=rows + V)
    ids, lp = b.slimspec_head_topk(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B), k)
    torch.cuda.synchronize()
    ora = oracle_mod.slimspec_head_topk(x.h, x.A, x.B, k)
    z_at = lambda ri, ci: oracle_mod.slimspec_logits_at(x.h, x.A, x.B, ri, ci)
    compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)


@pytest.mark.parametrize("rows,d,V,k,fp32", [
    (1, 8, 8, 2, False), (1, 1000, 37208, 4, False), (1, 3208, 4104, 8, False), (1, 72, 131080, 64 - 4, False), (2, 104, 33000, 5, False),
    (1, 40000, 520, 5, False), (1, 80000, 72, 5, False), (1, 80000, 520, 5, False),      # h fits beside the partial sums, does not
    (4, 16384, 200, 9, False), (3, 16384, 1032, 9, False), (6, 8192, 3080, 4, True), (9, 8192, 2056, 40, True),      # ... of several rows; the last group's fits
    (1, 104, 20000, 6, True), (2, 1000, 2056, 6, True), (5, 264, 9000, 10, True), (8, 2048, 1032, 20, True), (8, 6000, 520, 3, True),
    (19, 136, 8200, 5, True), (70, 72, 1544, 5, True),                         # groups of 8 rows; chunks of 512 columns from 65 rows on
])
def test_full_head(gpu, oracle_mod, rows, d, V, k, fp32):
    torch, b = gpu
    print(f"stream kernel, full head: rows={rows} d={d} V={V} k={k} fp32={fp32}", flush=True)
    assert_plan("full", rows, d, 8, V, k, fp32=fp32, kernel="stream", rows_in_lds=0 if d == 80000 or (rows > 1 and d >= 8192) else 1)
    x = synth.make_inputs(synth.small_config(rows, d, 8, V, k, peaked_every=4), seed=rows + d, with_full_head=True)
    W = synth.bf16_bits_to_f32(x.W) + np.float32(1e-4) if fp32 else x.W
    ids, lp = b.full_head_topk(to_dev_bf16(x.h), to_dev_f32(W) if fp32 else to_dev_bf16(W), k)
    torch.cuda.synchronize()
    ora = oracle_mod.full_head_topk(x.h, W, k)
    z_at = lambda ri, ci: oracle_mod.full_logits_at(x.h, W, ri, ci)
    compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)


# one row whose A every block reads: ranks of 1, 2, 4 and 8 pieces per row of A and of two column blocks, hidden sizes below, at and off
# the rows that a block takes per step, the rule's limits in d r, V and wavefronts, and the first shapes beyond them
@pytest.mark.parametrize("d,r,V,k,own", [
    (8, 8, 8, 2, 1), (4096, 8, 4104, 5, 1), (2048, 16, 8192, 64, 1), (1000, 24, 520, 7, 1), (1024, 32, 131072, 10, 1), (816, 40, 33000, 3, 1),
    (512, 64, 8200, 12, 1), (256, 72, 16384, 33, 1), (272, 120, 9000, 4, 1), (256, 128, 40008, 9, 1), (520, 64, 2056, 5, 0), (16, 136, 1032, 5, 0),
    (64, 16, 131080, 5, 0), (64, 128, 131072, 5, 0),
])
def test_input_made_by_every_block(gpu, oracle_mod, d, r, V, k, own):
    torch, b = gpu
    print(f"stream kernel, one row: d={d} r={r} V={V} k={k}", flush=True)
    assert_plan("low", 1, d, r, V, k, kernel="stream", own_input=own)
    x = synth.make_inputs(synth.small_config(1, d, r, V, k), seed=d + r)
    z_at = lambda ri, ci: oracle_mod.slimspec_logits_at(x.h, x.A, x.B, ri, ci)
    h, B = to_dev_bf16(x.h), to_dev_bf16(x.B)
    stack = to_dev_bf16(np.concatenate([x.A[::-1], x.A, x.A[::-1]])).view(3, d, r)      # the second of three positions has the row
    outs = [b.slimspec_head_topk(h, stack[1], B, k), b.slimspec_head_topk_positions(h, stack, [0, 0, 1, 1], B, k),
            b.slimspec_head_sample(h, stack[1], B, k, 5)]
    torch.cuda.synchronize()
    ora = oracle_mod.head_sample(x.h, x.A, x.B, k, 5)
    for out in outs:
        compare_with_oracle(out[0].cpu().numpy(), out[1].cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)
    assert int(outs[2][3][0]) == ora.sample_ids[0]
