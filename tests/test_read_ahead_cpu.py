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
    int K, V, bytes, nw;
    while (std::scanf("%%d %%d %%d %%d", &K, &V, &bytes, &nw) == 4) {
        const RowsGeom g = make_rows_geom(K, V);
        const ReadAhead a = rows_read_ahead(reinterpret_cast<const uint16_t *>(16), K, V, g, bytes, nw);
        std::vector<char> seen((size_t)K * (V / 8));
        long bad = 0, loads = 0;
        for (int b = 0; b < a.blocks; ++b)
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
        std::printf("%%ld %%ld %%ld %%d\n", bad, missed, loads, a.blocks);
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
    for nbytes in (1 << 20, 4 << 20, 9 << 20):
        for nw in (4, 16):
            bad, missed, loads, blocks = walk(f"{K} {V} {nbytes} {nw}\n")
            assert bad == 0 and missed == 0, (nbytes, nw, bad, missed)
            assert blocks % 8 == 0 and 16 * loads <= 4 * nbytes + 64 * 1024 * blocks, (nbytes, nw, loads, blocks)


def test_nothing_where_a_row_of_each_slice_is_more(walk):
    assert walk(f"512 {1 << 23} {4 << 20} 4\n")[2:] == [0, 0]
