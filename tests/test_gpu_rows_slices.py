"""Where the contraction's slices meet in rows_topk_kernel (csrc/rows_head.hip) against the CPU fp64 checker: two to eight slices, the last
rows that are added at once and the first that are not, one to six groups of columns per block, slices without a step of their own."""
import pytest

from paper_2605_10453_amd import synth
from parity_util import compare_with_oracle, to_dev_bf16
from plan_util import assert_plan
from test_gpu_parity import gpu  # noqa: F401  (the module's fixture)
from test_gpu_rows_head import FP32_TOL

pytestmark = pytest.mark.gpu


def how(K, V, rows):
    """Groups of 128 columns per block (one round of 256 blocks), what is left of eight wavefronts splits the contraction's steps of 32."""
    n = min(8 // -(-(-(-V // 128)) // 256), -(-K // 32))
    return {1: "one", 2: "halves"}.get(n, "at_once" if rows <= (16 if n > 4 else 8) else "in_turn")


# contraction steps of 32: 2, 3, 5, 9 (a slice of eight stays empty), 16; V: blocks of 1, 2, 3 and 6 groups of 128 columns (8, 4, 2 and 1 slices)
@pytest.mark.parametrize("r", [40, 72, 136, 264, 512])
@pytest.mark.parametrize("V,rows", [(1000, (5, 8, 9, 16, 17, 33)), (8200, (7,)), (33000, (5, 8, 9, 40)), (66000, (5, 18, 48)), (165000, (6,))])
def test_low_rank(gpu, oracle_mod, r, V, rows):
    torch, b = gpu
    d, k = 96, 7
    for n in rows:
        assert_plan("low", n, d, r, V, k, kernel="rows", slices_meet=how(r, V, n))
        print(f"slices meet: rows={n} r={r} V={V}", flush=True)
        x = synth.make_inputs(synth.small_config(n, d, r, V, k, peaked_every=4), seed=n + r)
        ids, lp = b.slimspec_head_topk(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B), k)
        torch.cuda.synchronize()
        ora = oracle_mod.slimspec_head_topk(x.h, x.A, x.B, k)
        z_at = lambda ri, ci: oracle_mod.slimspec_logits_at(x.h, x.A, x.B, ri, ci)
        compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)


@pytest.mark.parametrize("rows,d,V", [(3, 104, 8200), (8, 1032, 1000), (16, 264, 4104), (17, 264, 4104), (6, 136, 40000), (8, 520, 33000), (12, 520, 33000), (20, 72, 66000)])
def test_full_head(gpu, oracle_mod, rows, d, V):
    torch, b = gpu
    k = 11
    assert_plan("full", rows, d, 8, V, k, kernel="rows", slices_meet=how(d, V, rows))
    print(f"slices meet, full head: rows={rows} d={d} V={V}", flush=True)
    x = synth.make_inputs(synth.small_config(rows, d, 8, V, k, peaked_every=4), seed=rows + d, with_full_head=True)
    ids, lp = b.full_head_topk(to_dev_bf16(x.h), to_dev_bf16(x.W), k)
    torch.cuda.synchronize()
    ora = oracle_mod.full_head_topk(x.h, x.W, k)
    z_at = lambda ri, ci: oracle_mod.full_logits_at(x.h, x.W, ri, ci)
    compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)
