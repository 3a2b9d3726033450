// Prints, for every line "kind rows d r V k fp32 prepared sampling" of standard input (kind: low or full; the last three
// 0 or 1), what csrc/plan.hpp plans for the call and its first launch.  Host arithmetic only; linked with the library for
// the rules it keeps in its sources.
#define __host__
#define __device__
#include "../paper_2605_10453_amd/csrc/plan.hpp"
#include <cstdio>
#include <cstring>

using namespace slimspec;

int main()
{
    char kind_name[16];
    int rows, d, r, V, k, fp32, prepared, sampling;
    while (std::scanf("%15s %d %d %d %d %d %d %d %d", kind_name, &rows, &d, &r, &V, &k, &fp32, &prepared, &sampling) == 9) {
        const HeadKind kind = std::strcmp(kind_name, "full") == 0 ? HeadKind::Full : HeadKind::LowRank;
        const bool low_rank = kind == HeadKind::LowRank;
        const MfmaPlan p = make_mfma_plan(kind, mfma_max_rows_per_launch(rows), d, r, V);
        const bool f16 = low_rank && tile_operand_f16(k, prepared != 0), resident = resident_takes(p, f16);
        const bool rows_path = !fp32 && rows_path_takes(kind, rows, d, r, V, k, prepared != 0, sampling != 0);
        const char *kernel = rows_path ? "rows" : fp32 || !tile_path_takes(rows, k) ? "stream" : resident ? "resident" : "tile";
        const ChunkGeom g = make_chunk_geom(kind, rows, low_rank ? r : d, V);
        const RowsGeom rg = make_rows_geom(low_rank ? r : d, V);
        const int chunks = rows_path ? rg.chunks : g.chunks, chunk_cols = rows_path ? 128 * rg.G : 8 * g.lanes;
        const int launch_rows = rows_path && rows > kRowsMaxRows ? kRowsMaxRows : rows;
        const int sum_slices = low_rank && rows_path ? rows_sum_slices(make_rows_plan(kind, launch_rows, d, r, V, k).down, rows, d, r, V) : 0;
        const RowsPlan rp = make_rows_plan(kind, launch_rows < kRowsMaxRows ? launch_rows : kRowsMaxRows, d, r, V, k);
        const int most = sum_slices ? kAheadSlices : !down_rows_takes(rp.down, d, r) ? kAheadFinish : down_rows_reads_ahead(rp.down, d, r, V) ? kAheadDownRows : 0;
        const int reads_ahead = low_rank && rows_path && rows_read_ahead(nullptr, r, V, rg, most, 16).blocks > 0 ? most >> 20 : 0;
        const int last_len = merge_last_len(chunks, chunk_cols, V, k);
        const bool short_lists = merge_short_lists(launch_rows, chunks, last_len, k);
        const int gw = resident ? p.res.gw : p.gw, nsr = resident ? p.res.nsr : p.nsr;
        std::printf("kernel=%s resident_fits=%d f16=%d rows_per_block=%d col_blocks=%d records=%d parks=%d parked_offset=%zu parked_row_bytes=%zu chunk_cols=%d rows_in_lds=%d own_input=%d sum_slices=%d merge=%s rows_as_they_lie=%d block_tail=%d slices_meet=%s reads_ahead=%d\n", kernel, p.resident ? 1 : 0,
                    f16 ? 1 : 0, p.rt, gw, nsr / gw, p.defer && merge_parks_rows(low_rank ? r : d, !low_rank || f16) && !prepared && !sampling ? 1 : 0,
                    p.off_defer, merge_defer_bytes(1), 8 * g.lanes, low_rank || stream_rows_fit(rows < kGemvMaxRows ? rows : kGemvMaxRows, g, d) ? 1 : 0,
                    low_rank && !std::strcmp(kernel, "stream") && own_input_takes(g, rows, d, r, V, sampling != 0) ? 1 : 0,
                    sum_slices,
                    short_lists ? "short" : (chunks - 1) * k + last_len <= kMergeAheadLong * kRowMergeThreads ? "long_ahead" : "long",
                    !low_rank && rows_path && rows_read_by_rows(launch_rows, d, V, rg) ? 1 : 0,
                    rows == 1 && !std::strcmp(kernel, "stream") && block_row_takes(8 * g.lanes, k) ? 1 : 0,
                    rg.KS == 1 ? "one" : rows_lds(launch_rows, low_rank ? r : d, rg, k, sum_slices > 0).meet_at ? "at_once" : rg.KS == 2 ? "halves" : "in_turn", reads_ahead);
    }
    return 0;
}
