"""The tails of few-row calls against the CPU fp64 checker: the merge of short lists (csrc/merge_kernel.hip) at the sizes where its bound can go wrong, fewer
groups of entries than ids, one group more or less, wavefronts whose own lists are longer than a scan or overflow; and a row's tail by one wavefront
(csrc/gemv_parts.hpp: chunk_row_epilogue), chunks of 64 to 320 columns, last chunks of few columns.  Wide chunks, whose tail is the whole block's:
test_gpu_wide_chunk_tails.py."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2605_10453_amd import synth
from parity_util import compare_with_oracle, to_dev_bf16
from test_gpu_heads_next import check_sample_outputs
from test_gpu_merge import FP32_TOL, check
from test_gpu_parity import gpu  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu


# (d, r): all of A by every block; blocks of 4, of 8 and of 16 wavefronts; V: one chunk to a thousand, no multiples of 64 among them
@pytest.mark.parametrize("d,r", [(64, 16), (1040, 48), (520, 264)])
@pytest.mark.parametrize("V,ks", [(8, (1, 8)), (40, (1, 16, 40)), (136, (9, 17, 64)), (1000, (2, 15, 33)), (8200, (1, 8, 10, 16, 64)), (23344, (1, 10, 17, 31)),
                                  (131080, (4, 16, 63)), (151936, (10,)), (262152, (3, 12))])
def test_one_row(gpu, oracle_mod, d, r, V, ks):
    for k in ks:
        print(f"one row: d={d} r={r} V={V} k={k}", flush=True)
        check(gpu, oracle_mod, synth.make_inputs(synth.small_config(1, d, r, V, k), seed=V + k + r), k)


@pytest.mark.parametrize("V", [2056, 20008, 151936])
@pytest.mark.parametrize("rows", [1, 5])
def test_one_region_holds_the_winners(gpu, oracle_mod, rows, V):
    """Columns that rise in steps: every winner in adjacent chunks, then in adjacent columns, then many equal logits."""
    torch, b = gpu
    k = 16
    x = synth.make_inputs(synth.small_config(rows, 64, 16, V, k), seed=V)
    for width, scale in ((24, 4.0), (1024, 4.0), (V // 2, 1.0)):
        lo = (V - min(width, V)) // 16 * 8
        B = (x.B.astype(np.uint32) << 16).view(np.float32)
        if scale == 1.0:
            B[:, lo:lo + width] = B[:, lo:lo + 1]                # equal logits, more than any list has room for
        else:
            B[:, lo:lo + width] *= scale
        print(f"region: rows={rows} V={V} width={width}", flush=True)
        check(gpu, oracle_mod, replace(x, B=(B.view(np.uint32) >> 16).astype(np.uint16)), k)


@pytest.mark.parametrize("d,r,V,k", [(64, 16, 8, 3), (64, 16, 8200, 16), (520, 264, 23344, 9), (640, 640, 151936, 10), (520, 264, 9000, 33)])
def test_one_row_draws(gpu, oracle_mod, d, r, V, k):
    torch, b = gpu
    x = synth.make_inputs(synth.small_config(1, d, r, V, k), seed=V + 1)
    out = b.slimspec_head_sample(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B), k, 99)
    torch.cuda.synchronize()
    ora = oracle_mod.head_sample(x.h, x.A, x.B, k, 99, return_logits=True)
    check_sample_outputs(torch, out, ora, 99, V, ora.z, oracle_mod)


@pytest.mark.parametrize("d,V,f32", [(2056, 1000, False), (264, 20008, False), (264, 1000, True), (1032, 9000, True)])
def test_one_row_of_the_full_head(gpu, oracle_mod, d, V, f32):
    torch, b = gpu
    k = 11
    x = synth.make_inputs(synth.small_config(1, 8, d, V, k), seed=d)      # (its B [d, V] is the full head's W, of logits of about unit variance)
    h = synth.make_inputs(synth.small_config(1, d, 8, 64, k), seed=d).h
    W = to_dev_bf16(x.B)
    ids, lp = b.full_head_topk(to_dev_bf16(h), W.float() if f32 else W, k)
    torch.cuda.synchronize()
    ora = oracle_mod.full_head_topk(h, x.B, k)
    z_at = lambda ri, ci: oracle_mod.full_logits_at(h, x.B, ri, ci)
    compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)
