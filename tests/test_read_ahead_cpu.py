"""What the launches before rows_topk_kernel read ahead (csrc/plan.hpp: rows_read_ahead), followed on the host: every load lies inside the
weights, in the columns of the XCD that will ask for them, and together they cover the beginning of every slice of the contraction."""
import os
import subprocess

import pytest

from paper_2605_10453_amd import build

PROGRAM = r"""
#define __host__
#define __device__
#include "%s/plan.hpp"
#include <cstdio>
#include <vector>
using namespace slimspec;
int main() {
    int K, V, bytes, nw, groups;
    while (std::scanf("%%d %%d %%d %%d %%d", &K, &V, &bytes, &nw, &groups) == 5) {
        const RowsGeom g = make_rows_geom(K, V);
        const ReadAhead a = rows_read_ahead(reinterpret_cast<const uint16_t *>(16), K, V, g, bytes, nw);
        std::vector<char> seen((size_t)K * (V / 8));
        long bad = 0, loads = 0;
        const int each = ahead_blocks_each(a, groups);
        for (int b = 0; b < groups * each; ++b)             // row b / each of the grid; a block's XCD is its place in its row by 8
            for (int w = 0; w < nw; ++w) {
                AheadSlot s = ahead_slot(a, b & 7, (b >> 3) * nw + w);
                for (int n = 0; s.on && n < kAheadLoads; ++n, ahead_next(a, s))
                    for (int lane = 0; lane < 64; ++lane) {
                        const int kp = lane / a.lanes, col = s.col0 + 8 * (lane %% a.lanes), row = ahead_row(a, s) + kp;
                        if (kp >= a.rows_step || col >= V) continue;
                        ++loads;
                        if (row < 0 || row >= K || col < 0 || col + 8 > V || (col / (128 * g.G)) %% 8 != (b & 7)) ++bad;
                        else seen[(size_t)row * (V / 8) + col / 8] = 1;
                    }
            }
        const long fits = bytes / (2l * V * a.n_ranges), rows = fits < a.per ? fits : a.per;
        long missed = 0;
        for (int range = 0; range < a.n_ranges; ++range)
            for (int t = 0; t < rows; ++t) {
                const int row = range * a.per + t;
                for (int c = 0; row < K && c < V / 8; ++c) missed += !seen[(size_t)row * (V / 8) + c];
            }
        long distinct = 0;
        for (char c : seen) distinct += c;
        std::printf("%%ld %%ld %%ld %%ld %%d %%d\n", bad, missed, loads, distinct, a.blocks, each);
    }
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    where = tmp_path_factory.mktemp("ahead")
    (where / "walk.cpp").write_text(PROGRAM % os.path.join(build.HERE, "csrc"))
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(where / "walk"), str(where / "walk.cpp")], check=True)
    return lambda line: [int(x) for x in subprocess.run([str(where / "walk")], input=line, capture_output=True, text=True, check=True).stdout.split()]


@pytest.mark.parametrize("K", [8, 40, 136, 264, 520, 2048])
@pytest.mark.parametrize("V", [8, 136, 8200, 20000, 33000, 66008, 98312, 131080, 165000, 196616])
def test_loads_lie_inside_and_cover(walk, K, V):
    # the geometry of rows_topk_kernel: G groups of 128 columns per block, slices of the contraction
    cols = -(-V // 128)
    G = -(-cols // 256)
    G = 4 if G > 6 else G
    steps = -(-K // 32)
    per = -(-steps // min(8 // G, steps))
    ranges = -(-steps // per)
    lanes = 16 * G if G <= 4 else 8 * G                          # of a unit; a wavefront's load covers 64 / lanes rows of it
    rows_at_once, units = 64 // lanes, -(-(V // 8) // lanes)
    for nbytes in (1 << 20, 4 << 20, 9 << 20):
        for nw in (4, 16):
            bad, missed, loads, distinct, blocks, each = walk(f"{K} {V} {nbytes} {nw} 1\n")
            assert bad == 0 and missed == 0, (nbytes, nw, bad, missed)
            assert blocks % 8 == 0 and each == blocks
            # no more than asked for, but for the rows that a load at the end of a range covers besides
            assert 16 * distinct <= nbytes + ranges * (rows_at_once - 1) * 2 * V, (nbytes, nw, distinct)
            # loads that repeat another: of a unit's last wavefront at most all but one, and what of the last range lies beyond K
            rows = min(nbytes // (2 * V * ranges), 32 * per)
            beyond = sum(1 for t in range(0, rows, rows_at_once) if (ranges - 1) * 32 * per + t > K - rows_at_once) + 1 if rows else 0
            assert loads - distinct <= 64 * units * (11 + beyond), (nbytes, nw, loads, distinct)


@pytest.mark.parametrize("groups", [2, 3, 5, 16])
@pytest.mark.parametrize("K,V", [(64, 128256), (128, 32768), (256, 60000), (40, 136)])
def test_several_groups_share_the_blocks(walk, groups, K, V):
    """down_rows_kernel has a row of blocks per group: they read the same as one row does, and no more blocks than that takes."""
    one, shared = walk(f"{K} {V} {9 << 20} 16 1\n"), walk(f"{K} {V} {9 << 20} 16 {groups}\n")
    assert shared[:4] == one[:4] and shared[5] % 8 == 0
    assert one[4] <= groups * shared[5] < one[4] + 8 * groups


def test_nothing_where_a_row_of_each_slice_is_more(walk):
    assert walk(f"512 {1 << 23} {4 << 20} 4 3\n")[2:] == [0, 0, 0, 0]
