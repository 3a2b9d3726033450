"""Which code of csrc/merge_kernel.hip takes a call's lists (csrc/plan.hpp: merge_kind), against the CPU fp64 checker: both sides of every line."""
import pytest

from paper_2605_10453_amd import synth
from plan_util import assert_plan
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
