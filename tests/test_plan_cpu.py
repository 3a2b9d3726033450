"""The host-side plan of a call: pure arithmetic, checked without a GPU."""
from plan_util import launch_plan


def test_resident_head_only_where_its_offsets_fit():
    """head_resident_kernel addresses the 128 rows of a stage of the weights with 32-bit byte offsets: 128 * 2 V <= 2^32."""
    assert launch_plan("low", 512, 4096, 512, 128256)["resident"] == 1
    assert launch_plan("low", 512, 4096, 512, 1 << 24)["resident"] == 1
    for V in ((1 << 24) + 8, 1 << 25, 1 << 26):
        assert launch_plan("low", 512, 4096, 512, V)["resident"] == 0, V
