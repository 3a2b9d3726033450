"""Rows with fewer than k logits above -infinity: finite hidden states and weights whose product overflows to -infinity in
most columns.  The columns that do not overflow come first, then the others by id with a log-probability of -infinity;
every id is a column of the vocabulary (or its image under the id map), whichever kernels the call takes."""
import numpy as np
import pytest

from paper_2605_10453_amd import synth
from parity_util import to_dev_bf16, to_dev_f32
from test_gpu_parity import gpu  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu

BIG = 2.0 ** 66                 # BIG * BIG is beyond fp32
D = 64
# logits of the finite columns are below 16 in magnitude and summed in fp32 from exact products (t: 64 products first);
# 2^-20 is half a step of fp32 there, 64 of them cover both sums and the log-sum-exp
FP32_TOL = 64 * 2.0 ** -20


def _inputs(rows, V, n_finite, seed):
    """h [rows, D], M [D, V]; n_finite columns without the overflowing product, the first and the last column among them."""
    rng = np.random.default_rng(seed)
    h = rng.standard_normal((rows, D)).astype(np.float32)
    M = (rng.standard_normal((D, V)) * D ** -0.5).astype(np.float32)
    finite = sorted({V - 1, 0}) if n_finite == 2 else sorted(rng.choice(V, n_finite, replace=False).tolist())
    h[:, 0] = BIG
    M[0] = -BIG
    M[0, finite] = 0.0
    return synth.f32_to_bf16_bits(h), synth.f32_to_bf16_bits(M), finite


def _check(ids, lp, h_bits, M_bits, finite, k, tol, id_map=None):
    h, M = synth.bf16_bits_to_f64(h_bits), synth.bf16_bits_to_f64(M_bits)
    z = h[:, 1:] @ M[1:][:, finite]
    lse = np.log(np.exp(z).sum(axis=1))
    others = np.setdiff1d(np.arange(M.shape[1]), finite)
    n = min(k, len(finite))
    name = (lambda c: c) if id_map is None else (lambda c: id_map[c])
    for i in range(h.shape[0]):
        order = np.argsort(-z[i], kind="stable")[:n]
        assert ids[i, :n].tolist() == name(np.array(finite)[order]).tolist(), i
        assert np.abs(lp[i, :n] - (z[i, order] - lse[i])).max() <= tol, i
        assert ids[i, n:].tolist() == name(others[:k - n]).tolist(), i
        assert np.all(lp[i, n:] == -np.inf), i


CASES = [(1, 16, 16, 5), (3, 4104, 10, 3), (5, 16, 16, 2), (6, 4104, 10, 2), (40, 33000, 12, 7), (7, 70008, 40, 9), (1, 600008, 10, 2)]


@pytest.mark.parametrize("rows,V,k,n_finite", CASES)
def test_full_head(gpu, rows, V, k, n_finite):
    torch, b = gpu
    h, W, finite = _inputs(rows, V, n_finite, seed=rows + V)
    ids, lp = b.full_head_topk(to_dev_bf16(h), to_dev_bf16(W), k)
    torch.cuda.synchronize()
    _check(ids.cpu().numpy(), lp.cpu().numpy(), h, W, finite, k, FP32_TOL)


@pytest.mark.parametrize("rows,V,k,n_finite", [(64, 16, 16, 5), (64, 16392, 10, 2), (130, 4104, 16, 3)])
def test_both_heads_above_48_rows(gpu, rows, V, k, n_finite):
    """The stream records' merge: it finds its bound infinite and evaluates every logit of the row in fp32."""
    torch, b = gpu
    h, M, finite = _inputs(rows, V, n_finite, seed=rows + V)
    A = to_dev_bf16(synth.f32_to_bf16_bits(np.eye(D, dtype=np.float32)))       # t = h
    hd, Md = to_dev_bf16(h), to_dev_bf16(M)
    for ids, lp in (b.full_head_topk(hd, Md, k), b.slimspec_head_topk(hd, A, Md, k)):
        torch.cuda.synchronize()
        _check(ids.cpu().numpy(), lp.cpu().numpy(), h, M, finite, k, FP32_TOL)


def test_fp32_weights(gpu):
    torch, b = gpu
    h, W, finite = _inputs(6, 4104, 2, seed=8)
    ids, lp = b.full_head_topk(to_dev_bf16(h), to_dev_f32(synth.bf16_bits_to_f32(W)), 10)
    torch.cuda.synchronize()
    _check(ids.cpu().numpy(), lp.cpu().numpy(), h, W, finite, 10, FP32_TOL)


@pytest.mark.parametrize("rows,V,k,n_finite", CASES[:5])
def test_truncated_head(gpu, rows, V, k, n_finite):
    torch, b = gpu
    h, W, finite = _inputs(rows, V, n_finite, seed=rows + V)
    id_map = np.random.default_rng(V).permutation(V).astype(np.int32) * 3
    ids, lp = b.truncated_head_topk(to_dev_bf16(h), to_dev_bf16(W), torch.from_numpy(id_map).cuda(), k)
    torch.cuda.synchronize()
    _check(ids.cpu().numpy(), lp.cpu().numpy(), h, W, finite, k, FP32_TOL, id_map)


@pytest.mark.parametrize("rows,V,k,n_finite", CASES)
def test_low_rank_and_sampling(gpu, rows, V, k, n_finite):
    torch, b = gpu
    h, B, finite = _inputs(rows, V, n_finite, seed=rows + V)
    A = to_dev_bf16(synth.f32_to_bf16_bits(np.eye(D, dtype=np.float32)))       # t = h
    hd, Bd = to_dev_bf16(h), to_dev_bf16(B)
    ids, lp = b.slimspec_head_topk(hd, A, Bd, k)
    torch.cuda.synchronize()
    _check(ids.cpu().numpy(), lp.cpu().numpy(), h, B, finite, k, FP32_TOL)
    s = b.slimspec_head_sample(hd, A, Bd, k, 5)
    torch.cuda.synchronize()
    assert all(int(t) in finite for t in s[3].cpu()), s[3]
    assert torch.isfinite(s[2]).all() and torch.isfinite(s[4]).all()
