"""The weight-streaming matrix-core kernel for a few rows or long lists (csrc/rows_head.hip) against the CPU fp64 checker,
at the edges of its tiles: 16-row tiles, 48 rows per launch, chunks of 128 to 768 columns, contractions that are no
multiple of 32, lists of 1 to 64 ids, more equal logits than a row's candidate buffer holds, infinite weights."""
import numpy as np
import pytest

from paper_2605_10453_amd import synth
from parity_util import compare_with_oracle, to_dev_bf16
from plan_util import assert_plan
from test_gpu_parity import gpu  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu

# Products are exact and sums fp32: logits below 32 in magnitude (peaked rows), 2^-19 apart there; 32 such steps cover
# the roundings of the accumulation, of t and of the log-sum-exp many times over (5e-6 seen).
FP32_TOL = 6e-5


# rows; V in column groups of 128 per block: 1 (up to 32768 columns), 2, 3, 4, 5 (131080), 6 (165000)
@pytest.mark.parametrize("rows,d,r,V,k", [
    (5, 64, 8, 8, 1), (5, 64, 8, 136, 17), (16, 96, 40, 1000, 64), (17, 72, 24, 8200, 33), (32, 128, 64, 32776, 10),
    (33, 256, 72, 32776, 16), (48, 264, 200, 8192, 5), (49, 128, 96, 5000, 20), (97, 64, 32, 2056, 64),
    (6, 128, 64, 65544, 24), (8, 64, 40, 98312, 10), (40, 64, 40, 131080, 32), (3, 512, 104, 131080, 10), (47, 64, 16, 165000, 48),
    (4, 512, 256, 65544, 64),
])
def test_low_rank_at_the_tile_edges(gpu, oracle_mod, rows, d, r, V, k):
    torch, b = gpu
    print(f"rows kernel, low-rank: rows={rows} d={d} r={r} V={V} k={k}", flush=True)
    x = synth.make_inputs(synth.small_config(rows, d, r, V, k, peaked_every=4), seed=rows + V)
    ids, lp = b.slimspec_head_topk(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B), k)
    torch.cuda.synchronize()
    ora = oracle_mod.slimspec_head_topk(x.h, x.A, x.B, k)
    z_at = lambda ri, ci: oracle_mod.slimspec_logits_at(x.h, x.A, x.B, ri, ci)
    compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)


@pytest.mark.parametrize("rows,d,V,k", [(2, 8, 136, 64), (2, 1000, 32776, 10), (15, 136, 8200, 3), (33, 520, 4104, 40), (48, 72, 66000, 16)])
def test_full_head_at_the_tile_edges(gpu, oracle_mod, rows, d, V, k):
    torch, b = gpu
    print(f"rows kernel, full head: rows={rows} d={d} V={V} k={k}", flush=True)
    x = synth.make_inputs(synth.small_config(rows, d, 8, V, k, peaked_every=4), seed=rows + d, with_full_head=True)
    ids, lp = b.full_head_topk(to_dev_bf16(x.h), to_dev_bf16(x.W), k)
    torch.cuda.synchronize()
    ora = oracle_mod.full_head_topk(x.h, x.W, k)
    z_at = lambda ri, ci: oracle_mod.full_logits_at(x.h, x.W, ri, ci)
    compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)


@pytest.mark.parametrize("k", [3, 40])
def test_more_equal_logits_than_the_candidate_buffer(gpu, oracle_mod, k):
    """All columns equal: every logit ties, the ids are 0 .. k - 1 and the log-probability is -ln V."""
    torch, b = gpu
    rows, d, r, V = 6, 64, 16, 165000
    x = synth.make_inputs(synth.small_config(rows, d, r, V, k), seed=4)
    B = np.ascontiguousarray(np.repeat(x.B[:, :1], V, axis=1))
    ids, lp = b.slimspec_head_topk(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(B), k)
    torch.cuda.synchronize()
    assert np.array_equal(ids.cpu().numpy(), np.tile(np.arange(k, dtype=np.int32), (rows, 1)))
    assert np.abs(lp.cpu().numpy() + np.log(V)).max() <= FP32_TOL


def test_infinite_weights_and_hidden_states(gpu):
    """Same ids and the same (possibly not-a-number) log-probabilities as the one-row calls, which multiply in fp32."""
    torch, b = gpu
    rows, d, r, V, k = 7, 128, 48, 8200, 6
    x = synth.make_inputs(synth.small_config(rows, d, r, V, k), seed=9)
    h, A, B = to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B)
    B[5, 777] = float("inf")
    B[11, 8199] = float("-inf")
    h[3, 10] = float("inf")
    ids, lp = b.slimspec_head_topk(h, A, B, k)
    for i in range(rows):
        if i == 3:      # every logit of this row is infinite or not a number: nothing to compare but that it returns
            continue
        want_ids, want_lp = b.slimspec_head_topk(h[i:i + 1].contiguous(), A, B, k)
        torch.cuda.synchronize()
        assert torch.equal(ids[i], want_ids[0]), (i, ids[i], want_ids[0])
        assert torch.allclose(lp[i], want_lp[0], atol=FP32_TOL, rtol=0, equal_nan=True), (i, lp[i], want_lp[0])


@pytest.mark.parametrize("rows", [3, 5, 9, 16, 17, 33])
@pytest.mark.parametrize("k", [16, 17, 32, 33])
@pytest.mark.parametrize("V", [64, 4104, 40000])
def test_rows_in_pairs(gpu, oracle_mod, rows, k, V):
    """Two rows per wavefront: odd numbers of rows, both ways to bound a list, equal logits (columns of period 24: each value 2 to 1700
    times), a row with an infinite weight's logits beside an ordinary one, and a draw per row."""
    from test_gpu_heads_next import check_sample_outputs
    torch, b = gpu
    d, r = 64, 72
    print(f"rows in pairs: rows={rows} k={k} V={V}", flush=True)
    x = synth.make_inputs(synth.small_config(rows, d, r, V, k, peaked_every=3), seed=rows + k)
    h, A = to_dev_bf16(x.h), to_dev_bf16(x.A)
    assert_plan("full", rows, r, 8, V, k, kernel="rows", sampling=True)
    W = x.B                                              # the full head takes rows as they are: every value of z is exact up to fp32 sums
    hr = np.ascontiguousarray(np.tile(x.h, (1, 2))[:, :r])
    out = b.full_head_sample(to_dev_bf16(hr), to_dev_bf16(W), k, 5)
    torch.cuda.synchronize()
    ora = oracle_mod.head_sample(hr, None, W, k, 5, return_logits=True)
    check_sample_outputs(torch, out, ora, 5, V, ora.z, oracle_mod)
    assert np.abs(out[2].cpu().numpy() - ora.lse).max() <= FP32_TOL
    period = np.ascontiguousarray(np.tile(W[:, :24], (1, V // 24 + 1))[:, :V])
    ids, lp = b.full_head_topk(to_dev_bf16(hr), to_dev_bf16(period), k)
    torch.cuda.synchronize()
    ora = oracle_mod.full_head_topk(hr, period, k)
    z_at = lambda ri, ci: oracle_mod.full_logits_at(hr, period, ri, ci)
    compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)
    for row in ids.cpu().numpy():                        # among equal logits the smaller id comes first
        for res in range(24):
            mine = row[row % 24 == res]
            assert np.array_equal(mine, res + 24 * np.arange(len(mine)))
    Bi = to_dev_bf16(x.B)
    Bi[3, V // 2] = float("inf")
    ids, lp = b.slimspec_head_topk(h, A, Bi, k)
    want, want_lp = b.slimspec_head_topk(h[:1].contiguous(), A, Bi, k)
    torch.cuda.synchronize()
    assert torch.equal(ids[0], want[0]) and torch.allclose(lp[0], want_lp[0], atol=FP32_TOL, rtol=0, equal_nan=True)


# up to 8 rows whose slices of t every block adds: ranks that are no multiple of 64 or 32, the largest one, contractions that end in a partial
# stage, all group sizes, chunks of 128 to 768 columns; and the first shapes on the other side of the rule
@pytest.mark.parametrize("rows,d,r,V,k,slices", [
    (3, 2048, 520, 30000, 10, 8), (4, 2056, 264, 50000, 17, 8), (5, 2056, 8, 136, 3, 8), (5, 1032, 264, 8200, 33, 8), (8, 2064, 72, 32776, 64, 8),
    (7, 2600, 136, 65544, 10, 8), (6, 2056, 40, 98312, 16, 8), (8, 2056, 24, 131080, 20, 8), (5, 2056, 200, 165000, 5, 8), (8, 520, 512, 4104, 9, 8),
    (4, 1024, 1024, 16392, 12, 8), (5, 1024, 1024, 1000, 12, 0), (8, 200, 264, 2056, 6, 2), (9, 2056, 72, 2056, 4, 0),
])
def test_input_summed_by_every_block(gpu, oracle_mod, rows, d, r, V, k, slices):
    torch, b = gpu
    print(f"rows kernel, slices: rows={rows} d={d} r={r} V={V} k={k}", flush=True)
    assert_plan("low", rows, d, r, V, k, kernel="rows", sum_slices=slices)
    x = synth.make_inputs(synth.small_config(rows, d, r, V, k, peaked_every=3), seed=rows + d + r)
    h, A, B = to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B)
    ids, lp = b.slimspec_head_topk(h, A, B, k)
    # the same rows as three positions, one of them empty, with the same matrix
    p_ids, p_lp = b.slimspec_head_topk_positions(h, A.expand(3, d, r).contiguous(), [0, 1, 1, rows], B, k)
    torch.cuda.synchronize()
    ora = oracle_mod.slimspec_head_topk(x.h, x.A, x.B, k)
    z_at = lambda ri, ci: oracle_mod.slimspec_logits_at(x.h, x.A, x.B, ri, ci)
    for got in ((ids, lp), (p_ids, p_lp)):
        compare_with_oracle(got[0].cpu().numpy(), got[1].cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)
    if slices:                                           # not-a-number and infinite logits are summed again from the pieces in shared memory
        Bi = B.clone()
        Bi[r - 1, V // 2] = float("inf")
        h2 = h.clone()
        h2[rows - 1, d - 1] = float("nan")
        got, got_lp = b.slimspec_head_topk(h2, A, Bi, k)
        want, want_lp = b.slimspec_head_topk(h[:1].contiguous(), A, Bi, k)
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.allclose(got_lp[0], want_lp[0], atol=FP32_TOL, rtol=0, equal_nan=True)
        assert torch.isnan(got_lp[rows - 1]).all()
