"""The merge of the chunk lists (csrc/merge_kernel.hip) against the CPU fp64 checker: fewer lists than k and many more, lists whose
heads are all equal, one list that holds every winner, more entries than are fetched ahead, short last lists, draws."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2605_10453_amd import synth
from parity_util import compare_with_oracle, to_dev_bf16
from test_gpu_heads_next import check_sample_outputs
from test_gpu_parity import gpu  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu

FP32_TOL = 6e-5      # fp32 sums of exact products: see test_gpu_rows_head.py


def check(gpu, oracle_mod, x, k):
    torch, b = gpu
    V = x.B.shape[1]
    ids, lp = b.slimspec_head_topk(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B), k)
    torch.cuda.synchronize()
    ora = oracle_mod.slimspec_head_topk(x.h, x.A, x.B, k)
    z_at = lambda ri, ci: oracle_mod.slimspec_logits_at(x.h, x.A, x.B, ri, ci)
    compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)
    return ids.cpu().numpy(), lp.cpu().numpy()


@pytest.mark.parametrize("rows", [1, 2, 7])
@pytest.mark.parametrize("V,k", [(64, 64), (72, 33), (264, 64), (520, 64), (1000, 64), (2056, 64), (2056, 30), (4096, 40), (4096, 64), (12096, 39), (33000, 64), (70000, 10), (131080, 63), (300000, 5), (300000, 24)])
def test_lists_of_every_number_and_length(gpu, oracle_mod, rows, V, k):
    print(f"merge: rows={rows} V={V} k={k}", flush=True)
    check(gpu, oracle_mod, synth.make_inputs(synth.small_config(rows, 64, 16, V, k, peaked_every=3), seed=V + k + rows), k)


@pytest.mark.parametrize("rows", [1, 6])
@pytest.mark.parametrize("k", [1, 10, 50])
@pytest.mark.parametrize("V", [2056, 9000, 131080])
def test_equal_heads_and_crowded_lists(gpu, oracle_mod, rows, k, V):
    """Periodic columns: every chunk's list is the same, the first chunks' ids win.  Then one chunk that holds all winners."""
    x = synth.make_inputs(synth.small_config(rows, 64, 16, V, k), seed=k)
    period = np.ascontiguousarray(np.tile(x.B[:, :8], (1, V // 8)))
    ids, _ = check(gpu, oracle_mod, replace(x, B=period), k)
    # the winners of each group of equal logits are the smallest ids of their residue, in order
    for row in ids:
        for res in range(8):
            mine = row[row % 8 == res]
            assert np.array_equal(mine, res + 8 * np.arange(len(mine)))
    crowded = x.B.copy()
    lo = V // 2 // 8 * 8
    big = (crowded[:, lo:lo + 64].astype(np.uint32) << 16).view(np.float32) * 8.0
    crowded[:, lo:lo + 64] = (big.view(np.uint32) >> 16).astype(np.uint16)
    check(gpu, oracle_mod, replace(x, B=crowded), k)


def test_zero_hidden_state(gpu):
    torch, b = gpu
    V, k = 20000, 64
    x = synth.make_inputs(synth.small_config(3, 64, 16, V, k), seed=1)
    h = to_dev_bf16(np.zeros_like(x.h))
    for n in (1, 3):
        ids, lp = b.slimspec_head_topk(h[:n].contiguous(), to_dev_bf16(x.A), to_dev_bf16(x.B), k)
        torch.cuda.synchronize()
        assert np.array_equal(ids.cpu().numpy(), np.tile(np.arange(k, dtype=np.int32), (n, 1)))
        assert np.abs(lp.cpu().numpy() + np.log(V)).max() <= FP32_TOL


@pytest.mark.parametrize("rows,V", [(1, 72), (1, 200000), (1, 600000), (5, 200000)])
def test_draws(gpu, oracle_mod, rows, V):
    torch, b = gpu
    k = 7
    x = synth.make_inputs(synth.small_config(rows, 64, 16, V, k), seed=V)
    out = b.slimspec_head_sample(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B), k, 1234)
    torch.cuda.synchronize()
    ora = oracle_mod.head_sample(x.h, x.A, x.B, k, 1234, return_logits=True)
    check_sample_outputs(torch, out, ora, 1234, V, ora.z, oracle_mod)


@pytest.mark.parametrize("bits", [0x7fc00000, -0x400000, -1])
@pytest.mark.parametrize("V,k", [(1032, 10), (8200, 10), (40008, 16), (200000, 5)])
def test_rows_of_nothing_but_nan(gpu, V, k, bits):
    """Weights that are no numbers, of either sign or with all bits set (fp32 memory that was never written). The logits cannot be
    ordered, but every output is written, the ids are columns of the vocabulary, and other calls are not changed."""
    torch, b = gpu
    x = synth.make_inputs(synth.small_config(1, 64, 16, V, k), seed=V, with_full_head=True)
    h, W = to_dev_bf16(x.h), to_dev_bf16(x.W).float()
    id_map = torch.arange(V, dtype=torch.int32, device="cuda") * 3
    bad = torch.full((64, V), bits, dtype=torch.int32, device="cuda").view(torch.float32)
    before = b.truncated_head_topk(h, W, id_map, k)
    out_ids = torch.full((1, k), -7, dtype=torch.int32, device="cuda")
    out_lp = torch.zeros((1, k), device="cuda")
    b.truncated_head_topk(h, bad, id_map, k, out_ids=out_ids, out_logprobs=out_lp)
    after = b.truncated_head_topk(h, W, id_map, k)
    torch.cuda.synchronize()
    ids = out_ids.cpu().numpy()[0]
    assert np.all((ids >= 0) & (ids < 3 * V) & (ids % 3 == 0)) and len(set(ids)) == k, ids
    assert np.isnan(out_lp.cpu().numpy()).all()
    assert torch.equal(before[0], after[0]) and torch.equal(before[1], after[1])


@pytest.mark.parametrize("rows", [2, 5])
@pytest.mark.parametrize("bits", [0x7fc0, -0x40, -1])
def test_hidden_states_of_nothing_but_nan(gpu, rows, bits):
    torch, b = gpu
    V, k = 9000, 10
    x = synth.make_inputs(synth.small_config(rows, 64, 16, V, k), seed=rows)
    h = to_dev_bf16(x.h)
    h[1] = torch.full((64,), bits, dtype=torch.int16, device="cuda").view(torch.bfloat16)
    out_ids = torch.full((rows, k), -7, dtype=torch.int32, device="cuda")
    b.slimspec_head_topk(h, to_dev_bf16(x.A), to_dev_bf16(x.B), k, out_ids=out_ids)
    torch.cuda.synchronize()
    ids = out_ids.cpu().numpy()[1]
    assert np.all((ids >= 0) & (ids < V)) and len(set(ids)) == k, ids


@pytest.mark.parametrize("infinite", [False, True])
@pytest.mark.parametrize("rows,V,k", [(1, 9000, 10), (1, 128256, 16), (1, 200000, 10), (2, 40008, 40), (7, 128256, 32)])
def test_rows_that_mix_numbers_and_nan(gpu, rows, V, k, infinite):
    """Logits that are no numbers come before every number, in the order of their ids, wherever the chunk boundaries lie and
    however small the numbers beside them (with infinite: although every chunk also holds columns of +infinity)."""
    torch, b = gpu
    x = synth.make_inputs(synth.small_config(rows, 64, 16, V, k), seed=V + k)
    x = replace(x, h=np.repeat(x.h[:1], rows, axis=0))
    B = x.B.copy()
    t0 = synth.bf16_bits_to_f64(x.h[0]) @ synth.bf16_bits_to_f64(x.A[:, 0])
    if infinite:
        B[1:, ::40] = 0
        B[0, ::40] = 0x7f80 if t0 > 0 else 0xff80
    nan_cols = sorted({V // 2 + 1, V - 3, 3 * V // 4, V - 300})[:k]
    B[:, nan_cols] = 0x7fc0
    ids, lp = b.slimspec_head_topk(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(B), k)
    torch.cuda.synchronize()
    ids = ids.cpu().numpy()
    assert np.isnan(lp.cpu().numpy()).all()
    for row in ids:
        assert row[:len(nan_cols)].tolist() == nan_cols, row
        rest = row[len(nan_cols):]
        assert len(set(row.tolist())) == k and np.all((rest >= 0) & (rest < V))
        if infinite:
            assert np.array_equal(rest, [c for c in range(0, V, 40) if c not in nan_cols][:len(rest)]), row
