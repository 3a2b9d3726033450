"""The host-side plan of a call: pure arithmetic, checked without a GPU."""
import ctypes

import pytest

from paper_2605_10453_amd import binding
from plan_util import launch_plan


def test_resident_head_only_where_its_offsets_fit():
    """head_resident_kernel addresses the 128 rows of a stage of the weights with 32-bit byte offsets: 128 * 2 V <= 2^32."""
    assert launch_plan("low", 512, 4096, 512, 128256)["resident"] == 1
    assert launch_plan("low", 512, 4096, 512, 1 << 24)["resident"] == 1
    for V in ((1 << 24) + 8, 1 << 25, 1 << 26):
        assert launch_plan("low", 512, 4096, 512, V)["resident"] == 0, V


@pytest.mark.parametrize("d,r,V,k", [(512, 64, 16384, 10), (4096, 512, 16384, 12), (4096, 512, 128256, 10), (6248, 392, 2789880, 1),
                                     (3112, 40, 18352, 64), (1024, 520, 20000, 16), (64, 8, 8, 8)])
def test_a_workspace_serves_fewer_rows(d, r, V, k):
    """A caller sizes its workspace for the largest batch and runs smaller ones in it: the size never falls as rows are added."""
    lib = binding.load_library()
    queries = {"head": lambda n: binding.slimspec_workspace_bytes(n, d, r, V, k),
               "routed": lambda n: int(lib.routed_workspace_bytes(ctypes.byref(binding.SlimspecShape(n, d, r, V)), k))}
    for name, query in queries.items():
        sizes = [query(n) for n in range(1, 1100)]
        falls = [(n + 1, sizes[n - 1], sizes[n]) for n in range(1, len(sizes)) if sizes[n] < sizes[n - 1]]
        assert sizes[0] > 0 and not falls, (name, falls[:3])
