"""The host-side plan of a call: pure arithmetic, checked without a GPU."""
import ctypes
import random

import pytest

from paper_2605_10453_amd import binding
from plan_util import plan_of


def test_resident_head_only_where_its_offsets_fit():
    """head_resident_kernel addresses the 128 rows of a stage of the weights with 32-bit byte offsets: 128 * 2 V <= 2^32."""
    assert plan_of("low", 512, 4096, 512, 128256, 10)["resident_fits"] == 1
    assert plan_of("low", 512, 4096, 512, 1 << 24, 10)["resident_fits"] == 1
    for V in ((1 << 24) + 8, 1 << 25, 1 << 26):
        assert plan_of("low", 512, 4096, 512, V, 10)["resident_fits"] == 0, V


@pytest.mark.parametrize("d,r,V,k", [(512, 64, 16384, 10), (4096, 512, 16384, 12), (4096, 512, 128256, 10), (6248, 392, 2789880, 1),
                                     (3112, 40, 18352, 64), (1024, 520, 20000, 16), (64, 8, 8, 8), (512, 320, 16384, 10), (4096, 64, 151936, 10)])
def test_a_workspace_serves_fewer_rows(d, r, V, k):
    """A caller sizes its workspace for the largest batch and runs smaller ones in it: the size never falls as rows are added."""
    lib = binding.load_library()
    queries = {"head": lambda n: binding.slimspec_workspace_bytes(n, d, r, V, k),
               "routed": lambda n: int(lib.routed_workspace_bytes(ctypes.byref(binding.SlimspecShape(n, d, r, V)), k))}
    for name, query in queries.items():
        sizes = [query(n) for n in range(1, 1100)]
        falls = [(n + 1, sizes[n - 1], sizes[n]) for n in range(1, len(sizes)) if sizes[n] < sizes[n - 1]]
        assert sizes[0] > 0 and not falls, (name, falls[:3])


def test_a_workspace_serves_fewer_rows_at_random_shapes():
    """... over shapes drawn near and across the lines of the dispatch: a few rows more or less, vocabularies about 131072 columns,
    hidden sizes and ranks of both few-row rules, rows too long for shared memory."""
    lib = binding.load_library()
    rng = random.Random(5)
    steps = [1, 2, 3, 4, 5, 6, 8, 9, 16, 31, 32, 33, 47, 48, 49, 63, 64, 65, 128, 129, 256, 257, 511, 512, 513, 700, 1024, 1025]
    for _ in range(1500):
        d = 8 * rng.choice([rng.randint(1, 64), rng.randint(64, 256), rng.randint(256, 1024), rng.randint(1024, 12000)])
        r = 8 * rng.choice([rng.randint(1, 32), rng.randint(33, 64), rng.randint(65, 320)])
        V = 8 * rng.choice([rng.randint(1, 1024), rng.randint(1024, 8192), rng.randint(8192, 16384), rng.randint(16385, 40000)])
        k = min(V, rng.choice([1, 4, 10, 16, 17, 40, 64]))
        for query in (lambda n: binding.slimspec_workspace_bytes(n, d, r, V, k),
                      lambda n: int(lib.routed_workspace_bytes(ctypes.byref(binding.SlimspecShape(n, d, r, V)), k))):
            sizes = [query(n) for n in steps]
            falls = [(b, x, y) for b, x, y in zip(steps[1:], sizes, sizes[1:]) if y < x and y != 0]
            assert not falls, (d, r, V, k, falls[:3])


@pytest.mark.parametrize("r,V", [(256, 8192), (256, 32000), (512, 32000), (512, 128256), (1024, 128256)])
def test_prepared_weights_decide_between_33_and_48_rows(r, V):
    """With the column-major copy the stream records' merge is cheap: from 33 rows on such calls were 4 to 15 % slower on the
    kernel for few rows than on head_tile_kernel."""
    for rows in (24, 32):
        assert plan_of("low", rows, 8 * r, r, V, 10, prepared=True)["kernel"] == "rows"
    for rows in (33, 40, 48, 49):
        assert plan_of("low", rows, 8 * r, r, V, 10, prepared=True)["kernel"] == "tile"
        assert plan_of("low", rows, 8 * r, r, V, 10, prepared=True, sampling=True)["kernel"] == ("rows" if rows <= 48 else "tile")
    assert plan_of("low", 40, 8 * r, r, V, 40, prepared=True)["kernel"] == "rows"          # a list the records cannot hold
    assert plan_of("low", 48, 512, 64, V, 10, prepared=True)["kernel"] == "rows"           # the records' merge takes longer than the head kernel


@pytest.mark.parametrize("kind,rows,d,r,V,k,kernel", [
    ("low", 4, 2048, 256, 128256, 10, "stream"), ("low", 4, 3072, 384, 128256, 10, "stream"), ("low", 4, 2560, 320, 64000, 10, "rows"),
    ("low", 3, 4096, 512, 128256, 10, "rows"), ("low", 4, 1024, 128, 151936, 32, "rows"),
    ("low", 4, 4096, 512, 16384, 10, "stream"), ("low", 2, 4096, 512, 128256, 40, "stream"), ("low", 48, 2048, 256, 32000, 3, "rows"),
    ("low", 2, 512, 256, 32768, 10, "rows"), ("low", 2, 512, 264, 32768, 10, "stream"), ("low", 2, 256, 512, 128256, 10, "stream"),
    ("low", 2, 512, 1024, 8192, 64, "stream"), ("low", 2, 512, 512, 151936, 10, "rows"), ("low", 2, 4096, 64, 151936, 10, "stream"), ("low", 2, 4096, 128, 151936, 10, "rows"), ("low", 2, 1024, 16, 151936, 10, "rows"),
    ("low", 2, 4096, 512, 196608, 10, "rows"), ("low", 2, 4096, 512, 196616, 10, "stream"), ("low", 2, 512, 64, 200000, 10, "stream"), ("low", 2, 520, 64, 16384, 10, "stream"),
    ("full", 2, 256, 8, 32000, 10, "stream"), ("full", 2, 264, 8, 32000, 10, "rows"),
    ("full", 33, 512, 8, 64000, 1, "tile"), ("full", 48, 1024, 8, 64000, 1, "rows"), ("full", 48, 768, 8, 8192, 4, "rows"),
    ("full", 40, 512, 8, 128256, 10, "tile"), ("full", 40, 512, 8, 128256, 16, "rows"), ("full", 32, 256, 8, 8192, 1, "rows"),
    ("full", 33, 256, 8, 8192, 1, "tile"), ("full", 36, 512, 8, 8192, 6, "rows"), ("full", 36, 640, 8, 8192, 1, "rows"),
])
def test_few_rows_take_the_kernel_that_measures_faster(kind, rows, d, r, V, k, kernel):
    assert plan_of(kind, rows, d, r, V, k)["kernel"] == kernel


@pytest.mark.parametrize("rows,d,r,V,slices", [
    (8, 4096, 256, 128256, 8), (8, 4096, 256, 196608, 8), (8, 4096, 256, 196616, 0), (8, 4096, 128, 1048576, 0), (5, 4096, 64, 524288, 0),
    (8, 5120, 128, 128256, 8), (8, 5128, 128, 128256, 0), (8, 8192, 24, 8192, 0), (4, 4096, 1024, 128256, 8), (9, 4096, 128, 128256, 0),
])
def test_blocks_add_the_slices_only_where_that_is_less_work(rows, d, r, V, slices):
    """Every block adds them: not with more than one round of blocks, nor with slices so long that halving their number costs more than
    the launch that adds them."""
    plan = plan_of("low", rows, d, r, V, 10)
    assert (plan["kernel"], plan["sum_slices"]) == ("rows", slices), plan


@pytest.mark.parametrize("d,r,V,plain,sampling", [
    (256, 32, 8192, 1, 1), (512, 64, 131072, 1, 1), (256, 128, 40960, 1, 1), (264, 120, 60000, 0, 1), (256, 128, 40968, 0, 1), (336, 96, 60000, 0, 1),
    (256, 128, 128256, 0, 0), (512, 64, 131080, 0, 0), (264, 128, 8192, 0, 0),
])
def test_blocks_make_the_input_only_where_that_is_less_work(d, r, V, plain, sampling):
    """Two trips for A against a launch: beyond r = 64 only with few columns, or where the call waits for the host anyway."""
    assert plan_of("low", 1, d, r, V, 10)["own_input"] == plain
    assert plan_of("low", 1, d, r, V, 10, sampling=True)["own_input"] == sampling


@pytest.mark.parametrize("rows,d,V,in_lds,chunk_cols", [
    (1, 80000, 8192, 0, 64), (2, 24000, 8192, 1, 64), (4, 12288, 8192, 1, 64), (4, 16384, 8192, 0, 256), (3, 16384, 16384, 0, 256), (4, 16384, 16392, 0, 128),
    (8, 6144, 8192, 1, 64), (8, 8192, 8192, 0, 256), (64, 8192, 8192, 0, 256), (65, 8192, 8192, 0, 512), (8, 8192, 65536, 0, 256),
])
def test_rows_read_from_memory_have_no_narrow_chunks(rows, d, V, in_lds, chunk_cols):
    """Rows of the full head that shared memory does not hold leave all lanes beyond a chunk's width idle."""
    plan = plan_of("full", rows, d, 8, V, 10, fp32=True)
    assert (plan["kernel"], plan["rows_in_lds"], plan["chunk_cols"]) == ("stream", in_lds, chunk_cols), plan


@pytest.mark.parametrize("rows,V,k,merge", [
    (4, 20480, 16, "short"), (4, 20480, 17, "long"), (4, 19328, 17, "long"), (4, 19200, 17, "long_ahead"), (4, 8192, 40, "long_ahead"), (4, 8192, 41, "long"),
    (4, 32768, 16, "short"), (1, 262144, 8, "short"), (1, 262144, 9, "long"), (1, 524288, 2, "long_ahead"), (1, 524288, 3, "long"),
])
def test_entries_are_requested_ahead_only_where_that_is_faster(rows, V, k, merge):
    """Long lists: up to five entries per thread of the merge's block (2560); with eight, as short ones have them, calls took 1 to 4 % longer."""
    assert plan_of("low", rows, 1024, 128, V, k)["merge"] == merge


@pytest.mark.parametrize("rows,V,k,merge", [(1, 8632, 16, "short"), (24, 8632, 16, "short"), (25, 8632, 10, "short"), (25, 8632, 11, "long_ahead"), (48, 8632, 10, "short"),
                                            (48, 8632, 11, "long_ahead"), (32, 16384, 16, "long_ahead"), (32, 16392, 16, "short"), (48, 128256, 16, "short")])
def test_many_rows_of_few_short_lists_have_at_most_ten_ids(rows, V, k, merge):
    """The slowest of a launch's rows decides, and with many ids in few lists the short lists' bound now and then admits far too many entries: 42 rows, k = 11,
    V = 8632 8 % slower."""
    assert plan_of("low", rows, 1024, 128, V, k)["merge"] == merge


@pytest.mark.parametrize("rows,d,V,by_rows", [
    (8, 8184, 50000, 1), (8, 8192, 50000, 0), (48, 1360, 32768, 1), (16, 4088, 20000, 1), (16, 4096, 20000, 0), (48, 1360, 120000, 1), (48, 1368, 120000, 0), (24, 2496, 50000, 1),
    (24, 2504, 50000, 0), (16, 4088, 50000, 0), (48, 1200, 60000, 1), (48, 1216, 60000, 0), (48, 1040, 50000, 1), (48, 1048, 50000, 0), (32, 1800, 50000, 0), (40, 1024, 151936, 1),
    (48, 1360, 151936, 0), (33, 1024, 80000, 1), (33, 1096, 80000, 0), (48, 800, 140000, 0), (48, 1024, 100000, 0), (48, 1360, 140000, 0), (32, 1800, 140000, 0), (48, 744, 100000, 1),
    (32, 1120, 110000, 1), (32, 1080, 151936, 1), (32, 1080, 151752, 0), (24, 2216, 131704, 0), (8, 2216, 131704, 1), (16, 1248, 190008, 1), (16, 1256, 190008, 0),
])
def test_full_rows_are_regrouped_where_reading_them_as_they_lie_is_slower(rows, d, V, by_rows):
    """48 rows, d = 1360, V = 140000 took 10 % longer when only rows * d decided."""
    plan = plan_of("full", rows, d, 8, V, 10)
    assert (plan["kernel"], plan["rows_as_they_lie"]) == ("rows", by_rows), plan


@pytest.mark.parametrize("V,cols,most", [(131072, 512, 16), (128256, 512, 16), (125000, 496, 13), (110000, 432, 13), (102400, 448, 13), (102000, 400, 13), (97920, 384, 0), (32768, 128, 0),
                                         (151936, 320, 0), (262144, 512, 16)])
def test_a_single_rows_tail_by_the_block(V, cols, most):
    """Wide chunks and lists of up to 16 ids, 13 in chunks of 400 to 504 columns; k = 11 to 13 took 3 % longer there by one wavefront."""
    for k in range(1, 20):
        plan = plan_of("low", 1, 2048, 256, V, k)
        assert (plan["chunk_cols"], plan["block_tail"]) == (cols, int(k <= most)), plan


@pytest.mark.parametrize("rows,d,r,V,megabytes", [
    (8, 512, 64, 65536, 0), (8, 512, 128, 60000, 9), (3, 256, 32, 128256, 0), (8, 256, 128, 128256, 0), (8, 384, 128, 128256, 0), (8, 768, 128, 30000, 0), (8, 1024, 128, 30000, 9),
    (16, 2048, 128, 16384, 9), (16, 2048, 64, 16384, 0), (17, 512, 32, 60000, 9), (17, 504, 128, 60000, 9), (17, 504, 32, 60000, 0), (40, 256, 128, 128256, 0),
    (8, 4096, 256, 128256, 8), (8, 512, 320, 20000, 8), (12, 4096, 512, 60000, 4), (40, 4096, 512, 128256, 4),
])
def test_weights_are_read_ahead_where_the_launch_has_the_time(rows, d, r, V, megabytes):
    """A down-projection of one launch and little work took longer for it than the projection gained: up to 5 % with the weights in the last-level cache, 10 % without."""
    plan = plan_of("low", rows, d, r, V, 10)
    assert (plan["kernel"], plan["reads_ahead"]) == ("rows", megabytes), plan


def test_bench_names_the_kernel_the_library_runs():
    import os
    import sys
    sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    import bench
    from paper_2605_10453_amd import synth
    shapes = [(c.rows, c.d, c.r, c.V, c.k) for c in synth.CONFIGS.values()] + [(n, 4096, 512, 128256, 10) for n in (2, 16, 40, 64, 200)]
    for rows, d, r, V, k in shapes:
        for prepared in (False, True):
            name = bench.projection_kernel(rows, r, V, k, prepared=prepared)[0]
            assert name == {"stream": "stream_topk", "rows": "rows_topk", "tile": "head_tile", "resident": "head_resident"}[
                plan_of("low", rows, d, r, V, k, prepared=prepared)["kernel"]] + "_kernel", (rows, d, r, V, k, prepared)
        name = bench.projection_kernel(rows, d, V, k, full=True)[0]
        if d >= 1024:
            assert name.split("_kernel")[0] == {"stream": "stream_topk", "rows": "rows_topk", "tile": "head_tile"}[
                plan_of("full", rows, d, r, V, k)["kernel"]], (rows, d, V, k)
