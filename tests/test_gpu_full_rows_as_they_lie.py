"""The full head's rows as rows_topk_kernel reads them (csrc/plan.hpp: rows_read_by_rows) against the CPU fp64 checker: on both sides of the line, row counts
around the 16-row tiles, hidden sizes that end inside a step of 32, and an infinite element in the last eight."""
import numpy as np
import pytest

from paper_2605_10453_amd import synth
from parity_util import compare_with_oracle, to_dev_bf16
from plan_util import assert_plan
from test_gpu_parity import gpu  # noqa: F401  (the module's fixture)
from test_gpu_rows_head import FP32_TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,d,V", [(2, 264, 136), (3, 72, 8200), (8, 8184, 1000), (9, 8184, 1000), (15, 4368, 2056), (16, 4088, 2056), (16, 4096, 2056),
                                      (17, 1032, 33000), (32, 2040, 1000), (33, 2040, 1000), (48, 1360, 2056), (48, 1368, 2056)])
def test_both_sides_of_the_line(gpu, oracle_mod, rows, d, V):
    torch, b = gpu
    k = 17                                                       # (a list that every row count sends to this kernel)
    assert_plan("full", rows, d, 8, V, k, kernel="rows")
    print(f"full head, rows as they lie: rows={rows} d={d} V={V}", flush=True)
    x = synth.make_inputs(synth.small_config(rows, d, 8, V, k, peaked_every=4), seed=rows + d, with_full_head=True)
    ids, lp = b.full_head_topk(to_dev_bf16(x.h), to_dev_bf16(x.W), k)
    torch.cuda.synchronize()
    ora = oracle_mod.full_head_topk(x.h, x.W, k)
    z_at = lambda ri, ci: oracle_mod.full_logits_at(x.h, x.W, ri, ci)
    compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)


# blocks of two, three, four and six groups of columns, on either side of what they take
@pytest.mark.parametrize("rows,d,V,by_rows", [(48, 1040, 33000, 1), (48, 1048, 33000, 0), (48, 744, 66000, 1), (48, 752, 66000, 0), (25, 2400, 100000, 0), (48, 1360, 120000, 1),
                                              (33, 1512, 190016, 1), (20, 3000, 33000, 0), (17, 1168, 132008, 1), (17, 1184, 132008, 0)])
def test_blocks_of_several_groups(gpu, oracle_mod, rows, d, V, by_rows):
    torch, b = gpu
    k = 17
    assert_plan("full", rows, d, 8, V, k, kernel="rows", rows_as_they_lie=by_rows)
    print(f"full head, rows as they lie {by_rows}: rows={rows} d={d} V={V}", flush=True)
    x = synth.make_inputs(synth.small_config(rows, d, 8, V, k, peaked_every=4), seed=rows + d, with_full_head=True)
    ids, lp = b.full_head_topk(to_dev_bf16(x.h), to_dev_bf16(x.W), k)
    torch.cuda.synchronize()
    ora = oracle_mod.full_head_topk(x.h, x.W, k)
    z_at = lambda ri, ci: oracle_mod.full_logits_at(x.h, x.W, ri, ci)
    compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)


@pytest.mark.parametrize("rows,d,by_rows", [(3, 40, 1), (18, 72, 1), (16, 4072, 1), (16, 4104, 0), (40, 1608, 1), (40, 1640, 0)])
def test_an_infinite_element(gpu, oracle_mod, rows, d, by_rows):
    """h[1] = +inf in its last element.  Lanes beyond the last element read the row's last eight once more, against weights that were cleared: that must not
    make row 1's logits not-a-numbers.  They are +inf or -inf by the sign of the last weight, so the first k columns with a positive one win; and every
    other row is as before.  On both sides of the line: the row as it lies and regrouped."""
    torch, b = gpu
    V, k = 1000, 5
    assert_plan("full", rows, d, 8, V, k, kernel="rows", rows_as_they_lie=by_rows)
    assert d % 32 == 8                                           # the last step of 32 holds the last eight elements alone
    x = synth.make_inputs(synth.small_config(rows, d, 8, V, k), seed=d, with_full_head=True)
    h, W_bits = x.h.copy(), x.W.copy()
    h[1, d - 1] = 0x7f80
    W_bits[d - 1][(W_bits[d - 1] & 0x7fff) == 0] = 0x3c00        # no zeros: their product with the infinity would be no number
    W = to_dev_bf16(W_bits)
    print(f"an infinite element: rows={rows} d={d}", flush=True)
    ids0, lp0 = b.full_head_topk(to_dev_bf16(x.h), W, k)
    ids1, lp1 = b.full_head_topk(to_dev_bf16(h), W, k)
    torch.cuda.synchronize()
    assert ids1[1].cpu().numpy().tolist() == np.flatnonzero(W_bits[d - 1] < 0x8000)[:k].tolist()
    others = np.arange(rows) != 1
    assert np.array_equal(ids0.cpu().numpy()[others], ids1.cpu().numpy()[others])
    assert np.array_equal(lp0.cpu().numpy()[others], lp1.cpu().numpy()[others])
