"""The head kernel with the row operand in registers (csrc/head_resident.hip: more than 128 rows, r <= 512) against the CPU
fp64 checker, at the edges of its tiles: 256-row blocks, 64-column tiles, stages of 128 contraction elements, column
blocks with one tile or none; and the rescan of a record whose stream dropped a candidate."""
import numpy as np
import pytest

from paper_2605_10453_amd import synth
from parity_util import compare_with_oracle, to_dev_bf16
from plan_util import assert_plan
from test_gpu_heads_next import check_sample_outputs
from test_gpu_parity import check_low_rank, gpu  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu


# contractions of one to four stages, full and ragged; vocabularies of one tile, ragged last tiles, odd and even tile counts
@pytest.mark.parametrize("rows,d,r,V,k", [
    (129, 64, 8, 8, 3), (200, 64, 72, 72, 10), (256, 96, 128, 1000, 12), (257, 64, 136, 8200, 10), (300, 128, 256, 4104, 1),
    (513, 64, 264, 2056, 6), (140, 256, 384, 16392, 10), (512, 128, 392, 16456, 7), (260, 512, 512, 32840, 12), (130, 64, 512, 70008, 5),
])
def test_tile_edges(gpu, oracle_mod, rows, d, r, V, k):
    assert_plan("low", rows, d, r, V, k, kernel="resident")
    x = synth.make_inputs(synth.small_config(rows, d, r, V, k, peaked_every=6), seed=rows + r)
    check_low_rank(gpu, oracle_mod, x, k)


@pytest.mark.parametrize("rows,V", [(300, 40960), (200, 70016)])
def test_four_best_logits_in_one_stream(gpu, oracle_mod, rows, V):
    """A stream is a half-wavefront's share of the 64-column tiles col, col + gw, ... (gw = 128 column blocks for two row
    blocks, 256 for one).  A row's four largest logits sit in four groups of 16 of one stream, one more than it lists."""
    gw = 128 if rows > 256 else 256
    assert_plan("low", rows, 64, 64, V, 5, kernel="resident", col_blocks=gw, records=2)
    cfg = synth.small_config(rows=rows, d=64, r=64, V=V, k=5)
    x = synth.make_inputs(cfg, seed=rows + V)
    t = synth.bf16_bits_to_f64(x.h) @ synth.bf16_bits_to_f64(x.A)
    B = synth.bf16_bits_to_f32(x.B)
    planted = {}
    for n, i in enumerate((0, 9, rows - 1)):
        col = 3 + 5 * n
        cols = [64 * (col + gw * tile) + 32 * jj + 4 for tile in (1, 2) for jj in (0, 1)]      # + 4: the upper half-wavefront
        for c, alpha in zip(cols, (12.0, 11.5, 11.0, 10.5)):
            B[:, c] = (alpha * t[i] / (t[i] @ t[i])).astype(np.float32)
        planted[i] = cols
    x.B = synth.f32_to_bf16_bits(B)
    g_ids, _, _, _ = check_low_rank(gpu, oracle_mod, x, cfg.k, exact_rows=list(planted))
    for i, cols in planted.items():
        assert g_ids[i, :4].tolist() == cols, (i, g_ids[i], cols)


# ranks around the two pieces' strides of 16, 32 and 64 elements and the first rank beyond them, for both kernels
@pytest.mark.parametrize("rows,kernel", [(60, "tile"), (140, "resident")])
@pytest.mark.parametrize("r,V", [(8, 520), (16, 2056), (24, 4104), (32, 9000), (40, 8200), (64, 70000), (72, 8200)])
def test_ranks_in_two_pieces(gpu, oracle_mod, rows, kernel, r, V):
    """Ranks up to 64 multiply the sixteen leading bits of t.  What is left of its rounding moves a logit by at most
    2^-17 sum_j |t_j B[j, v]|, which is below 2^-17 sqrt(r) 18 < 1.1e-3 for logits of up to 18 whose terms do not cancel by more than
    sqrt(r); the winners' own values are exact or within 1.2e-5 of the largest logit.  One piece (r = 72) keeps the bar of 2e-2."""
    assert_plan("low", rows, 64, r, V, 7, kernel=kernel, f16=0)
    x = synth.make_inputs(synth.small_config(rows, 64, r, V, 7, peaked_every=3), seed=5 * r + rows)
    _, g_lp, ora, _ = check_low_rank(gpu, oracle_mod, x, 7)
    if r <= 64:
        err = np.abs(g_lp - ora.logprobs).max()
        print(f"r={r} rows={rows} largest error {err:.2e}", flush=True)
        assert err <= 1.1e-3, err


@pytest.mark.parametrize("rows,d,r,V,k", [(513, 64, 264, 2056, 6), (700, 64, 520, 4104, 10), (1100, 64, 264, 2056, 6), (1540, 64, 40, 1032, 12), (600, 64, 1024, 2056, 16)])
def test_two_launches_share_a_down_projection(gpu, oracle_mod, rows, d, r, V, k):
    """More rows than one launch takes: with the workspace that the query names the down-projection serves two launches at once, with what
    512 rows need one; the last launch of a call, and of a pair, has 1 to 512 rows."""
    torch, b = gpu
    x = synth.make_inputs(synth.small_config(rows, d, r, V, k, peaked_every=6), seed=rows + r)
    ora = oracle_mod.slimspec_head_topk(x.h, x.A, x.B, k)
    z_at = lambda ri, ci: oracle_mod.slimspec_logits_at(x.h, x.A, x.B, ri, ci)
    for n in (rows, 512):
        size = b.slimspec_workspace_bytes(n, d, r, V, k)
        ws = torch.full((size + 256,), 0x5a, dtype=torch.uint8, device="cuda")
        print(f"rows={rows} workspace of {n} rows: {size} bytes", flush=True)
        ids, lp = b.slimspec_head_topk(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B), k, workspace=ws[:size])
        torch.cuda.synchronize()
        compare_with_oracle(ids.cpu().numpy(), lp.cpu().numpy(), ora.ids, ora.lse, z_at, V)
        assert (ws[size:] == 0x5a).all()


@pytest.mark.parametrize("sizes,d,r,V,k", [((700,), 1024, 512, 2056, 10), ((600,), 2056, 136, 4104, 7), ((1024,), 1024, 512, 2056, 16), ((1100,), 520, 264, 1032, 12),
                                           ((300, 250, 50), 1024, 264, 2056, 5), ((512, 1, 0, 187), 1024, 512, 2056, 10)])
def test_results_do_not_depend_on_the_workspace(gpu, oracle_mod, sizes, d, r, V, k):
    """A row's down-projection is cut into the same slices, added in the same order, whether two launches share it or not: a workspace
    that fits one launch at a time, the library's own scratch and the query's workspace give the same bits."""
    torch, b = gpu
    rows = sum(sizes)
    x = synth.make_inputs(synth.small_config(rows, d, r, V, k, peaked_every=6), seed=rows + d)
    h, A, B = to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B)
    off = [sum(sizes[:p]) for p in range(len(sizes) + 1)]
    stack = torch.stack([A.roll(p, 0) for p in range(len(sizes))])

    def run(n):
        ws = torch.full((b.slimspec_workspace_bytes(n, d, r, V, k),), 0x5a, dtype=torch.uint8, device="cuda")
        if len(sizes) == 1:
            return b.slimspec_head_topk(h, A, B, k, workspace=ws)
        return b.slimspec_head_topk_positions(h, stack, off, B, k, workspace=ws)

    print(f"workspaces of 512 and {rows} rows, d={d} r={r}", flush=True)
    outs = [run(rows), run(512)]
    if len(sizes) == 1:
        outs.append(b.slimspec_head_topk_static(h, A, B, k))
    torch.cuda.synchronize()
    for ids, lp in outs[1:]:
        assert torch.equal(ids, outs[0][0]) and torch.equal(lp.view(torch.int32), outs[0][1].view(torch.int32))


@pytest.mark.parametrize("rows,d,r,V,k,kernel", [(513, 64, 40, 2056, 5, "resident"), (700, 520, 264, 4104, 10, "resident"), (700, 64, 520, 2056, 7, "tile"), (1100, 64, 72, 1032, 12, "resident")])
def test_draws_of_more_rows_than_one_launch(gpu, oracle_mod, rows, d, r, V, k, kernel):
    """The noise is a function of the row's index in the call, in every launch, with and without a shared down-projection."""
    torch, b = gpu
    assert_plan("low", rows, d, r, V, k, sampling=True, kernel=kernel)
    x = synth.make_inputs(synth.small_config(rows, d, r, V, k, peaked_every=6), seed=rows + r)
    ora = oracle_mod.head_sample(x.h, x.A, x.B, k, 2 ** 35 + 11, return_logits=True)
    outs = []
    for n in (rows, 512):
        ws = torch.full((b.slimspec_workspace_bytes(n, d, r, V, k),), 0x5a, dtype=torch.uint8, device="cuda")
        print(f"draws of {rows} rows, workspace of {n}", flush=True)
        outs.append(b.slimspec_head_sample(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B), k, 2 ** 35 + 11, workspace=ws))
        torch.cuda.synchronize()
        check_sample_outputs(torch, outs[-1], ora, 2 ** 35 + 11, V, ora.z, oracle_mod)
    assert all(torch.equal(p.view(torch.int32), q.view(torch.int32)) for p, q in zip(*outs))
