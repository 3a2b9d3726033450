"""One row in wide chunks (csrc/plan.hpp: block_row_takes) against the CPU fp64 checker: chunks of 448 and of 512 columns, lists on both sides of the line, draws."""
import pytest

from paper_2605_10453_amd import synth
from parity_util import to_dev_bf16
from plan_util import plan_of
from test_gpu_heads_next import check_sample_outputs
from test_gpu_merge import check
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
