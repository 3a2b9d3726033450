"""Which code of csrc/merge_kernel.hip takes a call's lists (csrc/plan.hpp: merge_short_lists), against the CPU fp64 checker: both sides of every line."""
import pytest

from paper_2605_10453_amd import synth
from parity_util import to_dev_bf16
from plan_util import assert_plan
from test_gpu_heads_next import check_sample_outputs
from test_gpu_merge import check
from test_gpu_parity import gpu  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu


# the most entries that are requested ahead (2560: five a thread), one list and one entry more, and what a last list of few columns leaves of them
@pytest.mark.parametrize("rows,V,k,merge", [(3, 8192, 40, "long_ahead"), (3, 8072, 40, "long_ahead"), (3, 8200, 40, "long"), (3, 19200, 17, "long_ahead"), (3, 19336, 17, "long"),
                                            (1, 8192, 20, "long_ahead"), (1, 8200, 20, "long"), (1, 524288, 2, "long_ahead"), (1, 524288, 3, "long")])
def test_entries_requested_ahead(gpu, oracle_mod, rows, V, k, merge):
    assert_plan("low", rows, 64, 16, V, k, merge=merge)
    print(f"merge lists: rows={rows} V={V} k={k} {merge}", flush=True)
    check(gpu, oracle_mod, synth.make_inputs(synth.small_config(rows, 64, 16, V, k, peaked_every=3), seed=V + k), k)


# short lists: up to 16 ids, up to 10 of more than 24 rows with up to 128 lists each
@pytest.mark.parametrize("rows,V,k,merge", [(24, 8632, 16, "short"), (25, 8632, 10, "short"), (25, 8632, 11, "long_ahead"), (25, 16384, 16, "long_ahead"), (25, 16392, 16, "short"), (48, 8632, 10, "short"),
                                            (48, 8632, 11, "long_ahead"), (33, 128256, 13, "short"), (48, 12000, 14, "long_ahead")])
def test_short_lists_by_rows(gpu, oracle_mod, rows, V, k, merge):
    assert_plan("low", rows, 64, 16, V, k, merge=merge)
    print(f"merge lists: rows={rows} V={V} k={k} {merge}", flush=True)
    check(gpu, oracle_mod, synth.make_inputs(synth.small_config(rows, 64, 16, V, k, peaked_every=3), seed=V + k), k)


def test_draws_of_many_rows_with_more_than_ten_ids(gpu, oracle_mod):
    torch, b = gpu
    rows, V, k = 25, 8632, 12
    x = synth.make_inputs(synth.small_config(rows, 64, 16, V, k), seed=V)
    out = b.slimspec_head_sample(to_dev_bf16(x.h), to_dev_bf16(x.A), to_dev_bf16(x.B), k, 1234)
    torch.cuda.synchronize()
    ora = oracle_mod.head_sample(x.h, x.A, x.B, k, 1234, return_logits=True)
    check_sample_outputs(torch, out, ora, 1234, V, ora.z, oracle_mod)
