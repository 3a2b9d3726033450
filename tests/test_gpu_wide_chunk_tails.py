"""One row in wide chunks (csrc/plan.hpp: block_row_takes; csrc/gemv_parts.hpp: block_row_epilogue) against the CPU fp64 checker: chunks of 448 and of 512 columns,
lists on both sides of the line, draws, last chunks of fewer columns than a list has ids, lists that hold every column of a wavefront, winners in one place."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2605_10453_amd import synth
from parity_util import compare_with_oracle, to_dev_bf16
from plan_util import assert_plan, plan_of
from test_gpu_heads_next import check_sample_outputs
from test_gpu_merge import FP32_TOL, check
from test_gpu_parity import gpu  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,r", [(64, 16), (520, 264)])
@pytest.mark.parametrize("V,cols,ks", [(104000, 448, (1, 10, 11)), (128256, 512, (2, 16, 17, 33))])
def test_one_row(gpu, oracle_mod, d, r, V, cols, ks):
    torch, b = gpu
    for k in ks:
        assert plan_of("low", 1, d, r, V, k)["chunk_cols"] == cols
        print(f"wide chunks: d={d} r={r} V={V} k={k}", flush=True)
        x = synth.make_inputs(synth.small_config(1, d, r, V, k), seed=V + k + r)
        check(gpu, oracle_mod, x, k)
        out = b.slimspec_head_sample(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B), k, 99)
        torch.cuda.synchronize()
        ora = oracle_mod.head_sample(x.h, x.A, x.B, k, 99, return_logits=True)
        check_sample_outputs(torch, out, ora, 99, V, ora.z, oracle_mod)


@pytest.mark.parametrize("V,k,tail", [(104000, 13, 1), (104000, 14, 0), (102008, 13, 1), (125000, 13, 1), (125000, 16, 0), (131072, 16, 1)])
def test_lists_on_either_side_of_the_line(gpu, oracle_mod, V, k, tail):
    for d, r in ((64, 16), (520, 264)):
        assert_plan("low", 1, d, r, V, k, block_tail=tail)
        print(f"wide chunks, the line: d={d} r={r} V={V} k={k}", flush=True)
        check(gpu, oracle_mod, synth.make_inputs(synth.small_config(1, d, r, V, k), seed=V + k + r), k)


@pytest.mark.parametrize("V,last,k", [(V, last, k) for V, last in ((128520, 8), (128528, 16), (128576, 64), (128896, 384), (131072, 512)) for k in (1, 8, 9, 16)]
                         + [(104008, 8, k) for k in (1, 8, 9, 13)])
def test_last_chunks_of_few_columns(gpu, oracle_mod, V, last, k):
    """Fewer columns than ids or than groups for a bound, wavefronts without columns; then the winners among them."""
    torch, b = gpu
    assert_plan("low", 1, 64, 16, V, k, block_tail=1)
    cols = plan_of("low", 1, 64, 16, V, k)["chunk_cols"]
    assert V - (V - 1) // cols * cols == last
    x = synth.make_inputs(synth.small_config(1, 64, 16, V, k), seed=V + k)
    print(f"last chunk: V={V} columns={last} k={k}", flush=True)
    check(gpu, oracle_mod, x, k)
    out = b.slimspec_head_sample(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B), k, 99)
    torch.cuda.synchronize()
    ora = oracle_mod.head_sample(x.h, x.A, x.B, k, 99, return_logits=True)
    check_sample_outputs(torch, out, ora, 99, V, ora.z, oracle_mod)
    B = (x.B.astype(np.uint32) << 16).view(np.float32)
    B[:, V - min(last, 16):] *= 8.0
    check(gpu, oracle_mod, replace(x, B=(B.view(np.uint32) >> 16).astype(np.uint16)), k)


@pytest.mark.parametrize("chunk,first,width", [(100, 0, 512), (0, 0, 512), (100, 128, 128), (250, 384, 128), (7, 510, 4), (251, 0, 8)])
def test_winners_in_one_place(gpu, oracle_mod, chunk, first, width):
    """All of them in one chunk, in one wavefront's columns, across two chunks: columns that stand out, then as many equal ones, which fill the lists."""
    V, k = 128520, 16
    assert_plan("low", 1, 64, 16, V, k, block_tail=1, chunk_cols=512)
    x = synth.make_inputs(synth.small_config(1, 64, 16, V, k), seed=chunk + first)
    t = synth.bf16_bits_to_f64(x.h[0]) @ synth.bf16_bits_to_f64(x.A)
    lo = 512 * chunk + first
    scaled = (x.B.astype(np.uint32) << 16).view(np.float32)
    scaled[:, lo:lo + width] *= 8.0
    print(f"winners in one place: columns {lo} to {lo + width}", flush=True)
    check(gpu, oracle_mod, replace(x, B=(scaled.view(np.uint32) >> 16).astype(np.uint16)), k)
    equal = (x.B.astype(np.uint32) << 16).view(np.float32)
    equal[:, lo:lo + width] = (4.0 * np.sign(t) / np.sqrt(16)).astype(np.float32)[:, None]        # (exact in bf16; logit sum |t|)
    ids, _ = check(gpu, oracle_mod, replace(x, B=(equal.view(np.uint32) >> 16).astype(np.uint16)), k)
    n = min(width, k)
    assert np.array_equal(ids[0][:n], lo + np.arange(n))


@pytest.mark.parametrize("V,d", [(128520, 40), (104008, 264), (128256, 1032)])
@pytest.mark.parametrize("f32", [False, True])
def test_one_row_of_the_full_head(gpu, oracle_mod, V, d, f32):
    torch, b = gpu
    for k in (1, 9, 10):
        assert_plan("full", 1, d, 8, V, k, fp32=f32, block_tail=1)
        x = synth.make_inputs(synth.small_config(1, 8, d, V, k), seed=d)      # (its B [d, V] is the full head's W, of logits of about unit variance)
        h = synth.make_inputs(synth.small_config(1, d, 8, 64, k), seed=d).h
        W = to_dev_bf16(x.B)
        print(f"full head: V={V} d={d} k={k} fp32 weights={f32}", flush=True)
        ids, lp = b.full_head_topk(to_dev_bf16(h), W.float() if f32 else W, k)
        torch.cuda.synchronize()
        ora = oracle_mod.full_head_topk(h, x.B, k)
        z_at = lambda ri, ci: oracle_mod.full_logits_at(h, x.B, ri, ci)
        compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V, tie_tol=FP32_TOL, lp_tol=FP32_TOL)
