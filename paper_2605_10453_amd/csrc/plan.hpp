// Host-side launch plan: which kernels a call runs and where each scratch
// array sits in the caller's workspace.  Pure arithmetic, no HIP calls, so the
// argument checks and the workspace query work on a machine without a GPU.
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <initializer_list>

namespace slimspec {

constexpr int kChunkCols = 512;      // vocabulary columns per partial at most: one wavefront x 8 columns per lane
constexpr int kGemvMaxRows = 8;      // rows handled by one pass of the streaming (lane-owns-columns) path
constexpr int kMergeThreads = 512;    // threads of the stream-merge block of one row
constexpr int SLIMSPEC_KMAX_INTERNAL = 64;
constexpr size_t kAlign = 256;

enum class HeadKind { LowRank, Full };

// How the few-row down-projection is shared out: n_cb column blocks of 64 columns of A x nds slices of d.
struct DownPlan { int n_items = 0, n_cb = 0, nds = 0, slice = 0; };
inline DownPlan make_down_plan(bool low_rank, int d, int r) {
    DownPlan p;
    if (low_rank) {
        p.n_cb = (r + 63) / 64;
        // about 240 items in all (one round of blocks on 256 CUs), at most 32 slices, slices a multiple of 8 rows
        int want = 240 / p.n_cb;
        if (want > 32) want = 32;
        if (want < 1) want = 1;
        int slice = ((d + want - 1) / want + 7) / 8 * 8;
        if (slice < 64) slice = 64;
        p.slice = slice;
        p.nds = (d + slice - 1) / slice;
        p.n_items = p.n_cb * p.nds;
    }
    return p;
}

// Geometry of the streaming kernel: a block owns one chunk of 8 * lanes adjacent columns (8 <= lanes <= 64).  A wavefront's
// lanes cover k_parts rows of the weights at a time, and the block's wavefronts split the contraction (nw1 of them for a single
// row; the launcher's choice otherwise).  The chunks are made so narrow that every CU gets one, and all of them are resident
// together: up to 131072 columns as 256 blocks of 16 wavefronts, beyond (297 chunks of 512 at 151936 columns would be two
// on 41 CUs) for a single row as 512 of 8 or 1024 of 4.  Multiples of 64 columns: whole cache lines wherever the rows are; where they are not
// (V no multiple of 64) a single row's chunks come in units of 16, closer to one per CU (d = 2680, V = 19120, 152 / 239 chunks: 30.9 / 27.5 us a call, d = 7984,
// V = 37208 110.9 / 106.0; several rows keep few lane groups: 8 fp32 rows, d = 440, V = 19192 18.3 / 20.2).
// (With 512 columns whatever V, 66 to 90 CUs of 256 had a block at V = 33184 to 45856: 3.0-3.3 TB/s where 5.5-6.2 are reached now.)
// Short contractions take smaller blocks: wavefronts without rows only lengthen the barriers.
constexpr int kNarrowChunkRows = 64;     // more rows (fp32 weights) keep chunks of 512 columns: their lists would fill the workspace
struct ChunkGeom { int lanes = 64, k_parts = 1, nw1 = 16, chunks = 0; };
inline ChunkGeom make_chunk_geom(int rows, int K, int V) {
    ChunkGeom g;
    const int n16 = (V + 7) / 8;                             // 16-byte column groups
    const int full = (V + kChunkCols - 1) / kChunkCols;
    int slots = 256;
    if (rows == 1 && full > 256) {
        slots = full <= 512 ? 512 : 1024;
        g.nw1 = full <= 512 ? 8 : 4;
    }
    if (rows <= kNarrowChunkRows) {
        const int unit = rows > 1 || V % 64 == 0 ? 8 : 2;
        g.lanes = ((n16 + slots - 1) / slots + unit - 1) / unit * unit;
        g.lanes = g.lanes < 8 ? 8 : g.lanes > 64 ? 64 : g.lanes;
    }
    g.k_parts = 64 / g.lanes;
    g.chunks = (n16 + g.lanes - 1) / g.lanes;
    while (g.nw1 > 4 && g.nw1 * g.k_parts * 4 >= K) g.nw1 /= 2;
    return g;
}

// How a block's nw wavefronts of k_parts lane groups share the contraction: `per` rows per wavefront, n partial sums in all.
struct StreamParts { int per, n; };
constexpr __host__ __device__ StreamParts stream_parts(int nw, int k_parts, int K) {
    const int step = 8 * k_parts, per = ((K + nw - 1) / nw + step - 1) / step * step;
    return {per, (K + per - 1) / per * k_parts};
}
constexpr int kDirectParts = 16;         // partial sums that a row's epilogue adds by itself; more are first added kSumParts ways
constexpr int kSumParts = 8;
// Shared memory of a block for R rows: partial sums, the epilogues' candidates, and the contraction input of x_bytes per element (0: none).
inline size_t stream_lds_bytes(int R, int nw, const ChunkGeom &g, int K, int x_bytes) {
    const int n = stream_parts(nw, x_bytes ? g.k_parts : 1, K).n, cw = 8 * g.lanes;
    return 4 * (size_t)R * cw * (n + (n > kDirectParts ? kSumParts : 0)) + 8 * (size_t)(R < nw ? R : nw) * cw + (size_t)x_bytes * R * K;
}
// A single row's tail by the whole block (gemv_parts.hpp: block_row_epilogue) instead of by one wavefront: wide chunks and short lists, whose elements are
// many and whose candidates few.  Chunks of 512 columns have 32 groups for the bound, two for each of 16 ids; narrower ones have fewer, the bound admits more, and
// more than 64 candidates take the wavefronts a second round.  (One wavefront / the block, us a call, d = 2048, r = 256: chunks of 512, V = 128256 k = 4 21.2 / 19.7,
// k = 10 21.3 / 20.4, k = 16 22.1 / 21.6, k = 24 22.8 / 23.9; of 496, V = 125000 k = 10 20.5 / 19.7, k = 13 21.7 / 21.0, k = 15 21.4 / 21.5; of 464 k = 13 20.5 / 19.8, k = 14
// 20.4 / 19.7, k = 15 20.6 / 21.4; of 448 k = 13 19.7 / 19.3, k = 15 19.6 / 20.7; of 432, V = 110000 k = 10 19.4 / 18.8, k = 13 19.9 / 19.3, k = 14 20.0 / 20.5, k = 16 20.2 / 20.9; of 400,
// V = 102400 k = 10 19.0 / 18.5, k = 13 19.7 / 19.0, k = 15 19.7 / 20.5; of 352, V = 90000, k = 10 18.1 / 18.4; of 128, V = 32768, k = 10 14.3 / 14.8, k = 24 15.0 / 17.1; d = 512, r = 40,
// V = 20000 11.3 / 12.2; full head, d = 1688, V = 87960, k = 38 57.7 / 60.0.)
constexpr __host__ __device__ bool block_row_takes(int cw, int k) { return cw >= 400 && k <= (cw == kChunkCols ? 16 : 13); }
constexpr size_t kStreamLdsLimit = 150 * 1024;      // of the CU's 160 KB
// Do the bf16 rows of a launch (at most kGemvMaxRows) fit beside what its smallest block needs?
inline bool stream_rows_fit(int rows, const ChunkGeom &g, int K) {
    const int R = rows <= 1 ? 1 : rows <= 2 ? 2 : rows <= 4 ? 4 : 8;
    return stream_lds_bytes(R, R == 8 ? 2 : 4, g, K, 2) <= kStreamLdsLimit;
}
// Full head: rows that do not fit are read from memory as fp32, and a wavefront's lanes then cover one row of the weights only.  Chunks of 64 columns
// leave 56 lanes idle there: 256 columns instead (4 rows, d = 16384, V = 8192 524 / 344 us a call, V = 16384 470 / 358, 8 rows, fp32, d = 8192, V = 8192
// 1380 / 1028; 128 columns from V = 16392 on are as good as these: V = 32000 364 / 361 and 1470 / 1504).
constexpr int kWideChunkLanes = 32;
inline ChunkGeom make_chunk_geom(HeadKind kind, int rows, int K, int V) {
    ChunkGeom g = make_chunk_geom(rows, K, V);
    if (kind == HeadKind::Full && rows > 1 && g.lanes < 16 && !stream_rows_fit(rows < kGemvMaxRows ? rows : kGemvMaxRows, g, K)) {
        g.lanes = kWideChunkLanes;
        g.k_parts = 64 / g.lanes;
        g.chunks = ((V + 7) / 8 + g.lanes - 1) / g.lanes;
    }
    return g;
}

// A single row whose A is so small (64 KB) that every block of the streaming kernel makes all of t itself: one launch less.  Two launches
// / one, us a call: d = 256, r = 32, V = 8192 13.1 / 9.5; d = 512, r = 64, V = 8192 14.1 / 13.1, V = 50000 13.7 / 11.9, V = 128256 13.8 / 12.9; d = 4096, r = 8,
// V = 8192 13.4 / 10.6; d = 256, r = 128, V = 8192 13.7 / 11.5; d = 336, r = 96, V = 60000, sampling 20.5 / 16.5.  Not with twice as much (d = 1024, r = 64, V = 16384
// 12.4 / 12.7, d = 512, r = 128, V = 50000 13.2 / 13.9), not where a CU has several blocks that read A (d = 512, r = 64, V = 151936 15.2 / 16.8), and not in
// blocks of 16 wavefronts, whose registers the weights and A do not share (d = 256, r = 128, V = 128256 16.8 / 25.5).  Ranks beyond 64, whose columns of A
// come in two trips, only while the weights are short (r = 120, d = 264: V = 8192 13.5 / 12.6, V = 20000 13.5 / 13.0, V = 40000 12.9 to 13.1 / 13.5, V = 60000
// 13.4 / 14.3; r = 128, d = 256: V = 40000 13.4 / 13.4, V = 60000 13.6 / 14.6; r = 72 level from V = 24000 to 131072) or with draws, whose calls wait for the
// host, for every launch (r = 72 to 128, V = 24000 to 60000 20.2 to 20.6 / 16.5 to 16.9).
constexpr int kOwnShortV = 40960;
inline bool own_input_takes(const ChunkGeom &g, int rows, int d, int r, int V, bool sampling) {
    return rows == 1 && r <= 128 && (int64_t)d * r <= 32768 && V <= 256 * kChunkCols && g.nw1 <= 8 && (r <= 64 || V <= kOwnShortV || sampling);
}

// ---- reading weights ahead (read_ahead.hpp) ------------------------------------------------------------------------
// The launches that make t for rows_topk_kernel leave the memory idle.  Further blocks of them read the weights that its blocks ask for
// first into the L2 (4 MB) of the XCD that will ask: a launch's blocks are dealt to the XCDs in turn, always from the first one on, and
// a line stays there from one launch to the next.  (Nothing / read into the next XCD's L2 / into the right one, us a call: 5 rows, d = 1024, r = 128, V = 128256
// 17.6 / 17.5 / 16.5, 7 rows, r = 256, V = 30000 15.9 / 15.5 / 14.3, 12 rows, d = 4096, r = 512, V = 60000 27.7 / 28.7 / 27.3.  Counters do not show it: a run that
// collects them empties the caches between launches.)
constexpr int kAheadLoads = 12;          // of a wavefront, a kilobyte each (16: a CU with such a block takes longer than the others; 8: more blocks)
struct ReadAhead {
    const uint16_t *M = nullptr;         // [K, V]
    int K = 0, V = 0;
    int lanes = 64, halves = 0;          // a unit is 8 lanes adjacent columns, a chunk of rows_topk_kernel 1 << halves units
    int n_units = 0, chunks = 0;         // units per XCD, chunks in all
    int n_ranges = 1, per = 0;           // its slices of the contraction, `per` rows each
    int rows_step = 1, n_t = 0;          // the first n_t steps of 64 / lanes rows of each
    int q_n = 0, q_div = 0, q_mod = 0;   // wavefronts per unit, and that number by n_ranges
    uint32_t units_inverse = 0, ranges_inverse = 0;      // 2^32 / n, rounded up
    int blocks = 0;                      // of the launch, a multiple of 8; 0: nothing to read
};
// A wavefront's place: unit and first (range, step); slot: its number among those of its XCD.
struct AheadSlot { bool on; int col0, t, range; };
constexpr __host__ __device__ int ahead_quotient(int n, int by, uint32_t inverse) { return by == 1 ? n : (int)(((uint64_t)(uint32_t)n * inverse) >> 32); }
constexpr __host__ __device__ AheadSlot ahead_slot(const ReadAhead &a, int xcd, int slot) {
    const int q = ahead_quotient(slot, a.n_units, a.units_inverse), unit = slot - q * a.n_units;
    const int chunk = xcd + 8 * (unit >> a.halves);
    const int t = ahead_quotient(q, a.n_ranges, a.ranges_inverse);
    return {q < a.q_n && chunk < a.chunks, 8 * a.lanes * ((chunk << a.halves) + (unit & ((1 << a.halves) - 1))), t, q - t * a.n_ranges};
}
// The first of the rows_step rows of a load; a wavefront's loads beyond the last step repeat it.
constexpr __host__ __device__ int ahead_row(const ReadAhead &a, const AheadSlot &s) {
    const int row = s.range * a.per + (s.t < a.n_t ? s.t : a.n_t - 1) * a.rows_step;
    return row < a.K - a.rows_step ? row : a.K - a.rows_step;
}
constexpr __host__ __device__ void ahead_next(const ReadAhead &a, AheadSlot &s) {
    s.t += a.q_div;
    s.range += a.q_mod;
    if (s.range >= a.n_ranges) { s.range -= a.n_ranges; ++s.t; }
}

// ... where a launch's grid has n_groups rows of blocks: how many of them in each (the last ones may find nothing left to read), a multiple of 8.  (All in
// the first row left as many empty blocks in every other: 16 rows in eight positions, d = 512, r = 64, V = 128256 18.0 / 17.3 us a call.)
inline int ahead_blocks_each(const ReadAhead &a, int n_groups) { return (a.blocks + 8 * n_groups - 1) / (8 * n_groups) * 8; }

struct Plan {
    bool ok = false;
    int rows = 0, d = 0, r = 0, V = 0, k = 0;
    int K = 0;                 // contraction length of the vocabulary projection (r or d)
    ChunkGeom geom;
    int chunks = 0;            // partials per row
    // byte offsets into the workspace
    size_t off_x = 0;          // fp32 [kGemvMaxRows, K]: t (low-rank) or widened h (full)
    size_t off_tpart = 0;      // fp32 [nds, kGemvMaxRows, r]  slices of t
    size_t off_part_ms = 0;    // float2 [rows, chunks]      running max, sum of exp
    size_t off_part_val = 0;   // float  [rows, chunks, k]   per-chunk top-k logits
    size_t off_part_id = 0;    // int32  [rows, chunks, k]   per-chunk top-k ids
    size_t off_part_smp = 0;   // float4 [rows, chunks]      per-chunk Gumbel-max winners (sampling calls)
    size_t bytes = 0;
};

inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

inline Plan make_plan(HeadKind kind, int rows, int d, int r, int V, int k) {
    Plan p;
    p.rows = rows; p.d = d; p.r = r; p.V = V; p.k = k;
    p.K = (kind == HeadKind::LowRank) ? r : d;
    p.geom = make_chunk_geom(kind, rows, p.K, V);
    p.chunks = p.geom.chunks;
    size_t off = 0;
    p.off_x = off;          off = align_up(off + sizeof(float) * kGemvMaxRows * (size_t)p.K);
    {
        const DownPlan dp = make_down_plan(kind == HeadKind::LowRank, d, r);
        p.off_tpart = off;  off = align_up(off + sizeof(float) * (size_t)dp.nds * kGemvMaxRows * (size_t)r);
    }
    p.off_part_ms = off;    off = align_up(off + 2 * sizeof(float) * (size_t)rows * p.chunks);
    p.off_part_val = off;   off = align_up(off + sizeof(float) * (size_t)rows * p.chunks * k);
    p.off_part_id = off;    off = align_up(off + sizeof(int32_t) * (size_t)rows * p.chunks * k);
    p.off_part_smp = off;   off = align_up(off + 16 * (size_t)rows * p.chunks);
    p.bytes = off;
    p.ok = true;
    return p;
}

// The largest vocabulary a call may have: a row's lists, counted in chunks of 512 columns (for a single row beyond 131072 columns
// in 512 or 1024 chunks), at 8 bytes for every list and 4 for each of its entries, and 8 k k for the winners', within 159 KB.
inline bool lists_supported(int rows, int V, int k) {
    size_t chunks = ((size_t)V + kChunkCols - 1) / kChunkCols;
    if (rows == 1 && chunks > 256 && chunks <= 1024) {
        const size_t n16 = ((size_t)V + 7) / 8, slots = chunks <= 512 ? 512 : 1024, lanes = (n16 + slots - 1) / slots;
        chunks = (n16 + lanes - 1) / lanes;
    }
    return 8 * (chunks + (size_t)k * k) + 4 * chunks * k <= 159 * 1024;
}

// ---- matrix-core path -------------------------------------------------------------------
constexpr int kPlanSlotsPerXcd = 32;     // blocks per XCD of the persistent kernel (256 CUs / 8 XCDs)
constexpr int kStreamsPerBlock = 4;      // lane streams of a row in one block of the head kernel: two half-wavefronts x two column halves
// Records a block of the head kernel leaves per row: all four lane streams while a row then has at most 512 records
// (many rows: few column blocks, where three listed groups per folded record would often be too few), two or one
// where there are more column blocks (the merge's time grows with the number of records).
inline int streams_per_block(int gw) { return gw <= 128 ? kStreamsPerBlock : gw <= 256 ? 2 : 1; }
constexpr int kStreamListPlan = 3;       // must equal kStreamList (launch.hpp)
constexpr int kStreamRecPlan = 3 + 3 * kStreamListPlan + 8;      // sized for sampling calls (kStreamRecSample, launch.hpp)

int head_tile_rows_per_block(int rows);
size_t merge_defer_bytes(int rows);
// Rows whose exact re-evaluations are parked for exact_cols_kernel: worth two more launches when a few rows with long
// column gathers would otherwise hold the merge up.  Always from K = 2048 (the full head: 127 -> 35 us at 512 rows);
// from K = 1024 when the kernel ran on f16 operands, where few rows need any re-evaluation (C5: 42.7 -> 34.3 us).
// With bf16 operands most rows re-evaluate something and the gathers are bound by the memory side's bandwidth, not by
// one CU's latency: parked or not measures the same at K = 1024 (58 us) and worse at K = 512 (32 -> 43 us).
constexpr int kDeferMinK = 2048, kDeferMinKFine = 1024;
inline bool merge_parks_rows(int K, bool fine_operand) { return K >= kDeferMinK || (fine_operand && K >= kDeferMinKFine); }

// Many-row down-projection: tiles of 64 x 64 of t, the contraction in `slices` slices (a power of two): enough
// blocks for every CU, at least two stages of 32 contraction elements per block.  The rows come in groups that share
// a down-projection matrix (one group unless the call names one matrix per drafted position); a row tile never
// crosses a group, and the rows of padding [rows, rows_pad) form one more group that is only zero-filled.
constexpr int kMaxPositions = 16;
template <int G>                         // groups at most, without the padding
struct DownGridOf {
    int n_rt = 0;                        // row tiles that hold rows, over all groups
    int n_rt_all = 0;                    // ... with the tiles of the padding group
    int n_ct = 0, slices = 1;
    int n_groups = 0;                    // groups with rows; group n_groups is the padding
    int g_row0[G + 2] = {};              // first row of group g; g_row0[n_groups] = rows, g_row0[n_groups + 1] = rows_pad
    int g_tile0[G + 2] = {};             // first row tile of group g; g_tile0[n_groups + 1] = n_rt_all
    int g_mat[G + 1] = {};               // which matrix of the stack the group uses
};
using DownGrid = DownGridOf<kMaxPositions>;
// Two launches' rows at once: the second launch's row tiles stand behind the first's, and either keeps its number of slices, so that a
// row's sums are the same, in the same order, as when every launch has its own down-projection.  A type of its own, with kernels of its own: five
// more words of arguments and the choice between the two cost the calls of one launch 0.4 us (23 rows 42.4 / 42.8 us).
struct JointDownGrid : DownGridOf<kMaxPositions + 1> {      // (a position that both launches hold rows of counts twice)
    int rt_second = 0, slices_second = 1;     // row tiles from rt_second on are the second launch's, with its slices
    int blocks_first = 0;                     // blocks of down_tile_kernel that work for the first
};
static_assert(sizeof(DownGrid) == sizeof(int) * (5 + 2 * (kMaxPositions + 2) + kMaxPositions + 1), "nothing of it is an argument of one launch's kernels");
// group g covers rows [g_first[g], g_first[g + 1]) of the launch (g_first[n_groups] = rows), all groups non-empty
inline DownGrid make_down_grid(int rows, int rows_pad, int d, int r, int n_groups = 1, const int *g_first = nullptr,
                               const int *g_mat = nullptr) {
    DownGrid g;
    g.n_groups = n_groups;
    int tile = 0;
    for (int q = 0; q < n_groups; ++q) {
        const int lo = g_first ? g_first[q] : 0, hi = g_first ? g_first[q + 1] : rows;
        g.g_row0[q] = lo; g.g_tile0[q] = tile; g.g_mat[q] = g_mat ? g_mat[q] : 0;
        tile += (hi - lo + 63) / 64;
    }
    g.n_rt = tile;
    g.g_row0[n_groups] = rows; g.g_tile0[n_groups] = tile;
    tile += (rows_pad - rows + 63) / 64;
    g.g_row0[n_groups + 1] = rows_pad; g.g_tile0[n_groups + 1] = tile;
    g.n_rt_all = tile;
    g.n_ct = (r + 63) / 64;
    const int tiles = g.n_rt * g.n_ct, n_stages = (d + 31) / 32;
    // (two blocks per CU, i.e. twice the slices, measured slower: 10.7 + 4.6 against 8.9 + 4.5 us at 512 rows)
    // (at most 16 slices: with 32, at 16 and 64 rows, the tile kernel measures the same and the sum of the slices 1.1 us more)
    while (g.slices < 16 && tiles * g.slices < 256 && n_stages / (2 * g.slices) >= 2) g.slices *= 2;
    return g;
}
// Blocks of down_tile_kernel.  slices >= 8: every XCD has slices / 8 slices of every tile; fewer: 8 / slices XCDs share a slice and split the
// tiles.  A multiple of 8.
inline int down_tile_blocks(const DownGrid &g) {
    const int tiles = g.n_rt * g.n_ct;
    return g.slices >= 8 ? tiles * g.slices : 8 * ((tiles + 8 / g.slices - 1) / (8 / g.slices));
}
// a: the first launch's rows, no padding; b: the second's
inline JointDownGrid join_down_grids(const DownGrid &a, const DownGrid &b) {
    JointDownGrid g;
    const int rows = a.g_row0[a.n_groups];
    for (int q = 0; q < a.n_groups; ++q) { g.g_row0[q] = a.g_row0[q]; g.g_tile0[q] = a.g_tile0[q]; g.g_mat[q] = a.g_mat[q]; }
    g.n_ct = a.n_ct;
    g.slices = a.slices;
    g.slices_second = b.slices;
    g.rt_second = a.n_rt;
    g.blocks_first = down_tile_blocks(a);
    g.n_rt = a.n_rt + b.n_rt;
    g.n_rt_all = a.n_rt + b.n_rt_all;
    g.n_groups = a.n_groups + b.n_groups;
    for (int q = 0; q <= b.n_groups + 1; ++q) {
        g.g_row0[a.n_groups + q] = rows + b.g_row0[q];
        g.g_tile0[a.n_groups + q] = a.n_rt + b.g_tile0[q];
        if (q < b.n_groups) g.g_mat[a.n_groups + q] = b.g_mat[q];
    }
    return g;
}
// Partial tiles of t, in 64 x 64 tiles of floats, for any grouping of `rows` rows into at most kMaxPositions groups:
// slices * tiles stays below 512 while the contraction is split, and is the tile count itself when it is not.
inline size_t down_part_tiles_bound(int rows, int r) {
    const size_t tiles = ((size_t)(rows + 63) / 64 + kMaxPositions - 1) * (size_t)((r + 63) / 64);
    return tiles > 512 ? tiles : 512;
}

// ---- row operand resident in registers (head_resident.hip) -------------------------------------------------------
constexpr int kResidentTileCols = 64;
constexpr int kResidentMaxK = 512;       // 32 rows x 512 elements: 128 of a wavefront's 256 registers per lane
constexpr int kResidentMaxV = 1 << 24;   // the kernel's 32-bit offsets reach over the 128 rows of a stage of the weights
// Blocks of n_rb row blocks (256 rows) x gw column blocks; n_t tiles of 64 columns; two records (half-wavefronts) per
// block and row, of up to 32 groups at 128 column blocks.  (Four records of 16 groups each make a crowded record, i.e. an
// exact rescan of its columns, eight times rarer than the one 512-row call in a hundred it is at k = 10, and half as long,
// but cost every call 4 us.  A call with one such row: 179 us plain, 128 with prepared weights, against 115 and 96 without;
// head_tile_kernel with four records 148 and 117 against 126 and 105.  With four planted columns 182 and 151 against 119 and 97, and with
// draws, for which such a row is as likely, 222 and 189 against 160 and 136.)
struct ResidentGrid { int n_rb = 1, gw = 8, n_t = 0, nsr = 0; };
inline ResidentGrid make_resident_grid(int n_rb, int V) {
    ResidentGrid g;
    g.n_rb = n_rb;
    g.n_t = (V + kResidentTileCols - 1) / kResidentTileCols;
    int colgroups = kPlanSlotsPerXcd / n_rb;
    if (colgroups < 1) colgroups = 1;
    const int need = (g.n_t + 7) / 8;
    if (colgroups > need) colgroups = need;
    g.gw = 8 * colgroups;
    g.nsr = 2 * g.gw;
    return g;
}

constexpr int kTwoPiecesMaxRank = 64;    // ranks whose t the many-row kernels take in two bf16 pieces (tile_operand below)
// elements between the two pieces: the least that head_tile_kernel's stages of 32 allow
constexpr __host__ __device__ int two_pieces_stride(int r) { return r <= 16 ? 16 : r <= 32 ? 32 : 64; }

struct MfmaPlan {
    int rows = 0, rows_pad = 0, rt = 0, n_rb = 0, gw = 0, nsr = 0, n_vt = 0;
    bool resident = false;               // the row operand fits a wavefront's registers (bf16 operands)
    ResidentGrid res;
    DownGrid down, down_second;          // (the second of two launches)
    size_t off_down_part = 0;            // fp32 [slices][n_rt][n_ct][4][16][64] of each launch: partial tiles of t (sized for any grouping of the rows)
    size_t off_t32 = 0;                  // fp32 [rows_pad, r]
    size_t off_t16 = 0;                  // 16-byte vectors [8 ceil(K / 64), rows_pad]: the head kernel's row operand (two of them for two pieces)
    size_t off_stat = 0;                 // float2 [2 ceil(r / 64), rows_pad]: per row and 32 columns of t, (sum of dt^2, sum of t dt), dt = t - rounded t
    size_t off_tilescale = 0;            // float2 [n_vt]: (column scale, mean square) of B per vocabulary tile
    size_t off_streams = 0;              // fp32 [rows, nsr, kStreamRec] of one launch
    size_t records = 0;                  // ... records there is room for
    size_t off_defer = 0;                // parked rows of the merge (long contractions only; bytes 0 otherwise)
    bool defer = false;
    size_t bytes = 0;
};

// rows here is the number of rows of ONE launch (at most kPlanSlotsPerXcd row blocks), or of two that share a down-projection: the grids
// are then of no use, but the scratch serves both.
constexpr int kMaxLaunchRows = 512;
// The largest hidden size and rank of the low-rank head: down_tile_kernel's 32-bit byte offsets reach over the rows of h of two launches
// and over the 32 rows of a stage of A.
constexpr int kMaxHidden = 1 << 21, kMaxRank = 1 << 24;
static_assert(2ll * kMaxLaunchRows * 2 * kMaxHidden <= 1ll << 32, "offsets into the rows of h");
static_assert(32ll * 2 * kMaxRank <= 1ll << 32, "offsets into a stage of A");
inline MfmaPlan make_mfma_plan(HeadKind kind, int rows, int d, int r, int V) {
    MfmaPlan p;
    p.rows = rows;
    p.rt = head_tile_rows_per_block(rows);
    p.n_rb = (rows + p.rt - 1) / p.rt;
    p.rows_pad = p.n_rb * p.rt;
    p.n_vt = (V + 255) / 256;
    int colgroups = (p.rt == 128 ? 2 : 1) * kPlanSlotsPerXcd / p.n_rb;      // 128-row blocks: two per CU
    if (colgroups < 1) colgroups = 1;
    const int need = (p.n_vt + 7) / 8;
    if (colgroups > need) colgroups = need;
    p.gw = 8 * colgroups;
    p.nsr = streams_per_block(p.gw) * p.gw;
    size_t off = 0;
    if (kind == HeadKind::LowRank) {
        p.off_t32 = off;       off = align_up(off + sizeof(float) * (size_t)p.rows_pad * r);
        p.off_t16 = off;       off = align_up(off + 2 * (size_t)p.rows_pad * ((r + 63) / 64 * 64) * (r <= kTwoPiecesMaxRank ? 2 : 1));
        p.off_stat = off;      off = align_up(off + 2 * sizeof(float) * (size_t)p.rows_pad * 2 * ((r + 63) / 64));
        const int first = rows < kMaxLaunchRows ? rows : kMaxLaunchRows;
        p.down = make_down_grid(first, rows == first ? p.rows_pad : first, d, r);
        if (rows > first) p.down_second = make_down_grid(rows - first, p.rows_pad - first, d, r);
        size_t tiles = down_part_tiles_bound(first, r);
        if (rows > first) tiles += down_part_tiles_bound(rows - first, r);
        p.off_down_part = off; off = align_up(off + sizeof(float) * 4096 * tiles);
        p.off_tilescale = off; off = align_up(off + 2 * sizeof(float) * (size_t)p.n_vt);
    } else {
        p.off_t16 = off;       off = align_up(off + 2 * (size_t)p.rows_pad * ((d + 63) / 64 * 64));      // h regrouped for the kernel
    }
    p.resident = kind == HeadKind::LowRank && p.rt == 256 && r <= kResidentMaxK && V <= kResidentMaxV;
    if (p.resident) p.res = make_resident_grid(p.n_rb, V);
    // (room for the records of one row block, the most a row has: a workspace then serves fewer rows as well)
    const int nsr_res = p.resident ? make_resident_grid(1, V).nsr : 0;
    p.records = (size_t)rows * (p.nsr > nsr_res ? p.nsr : nsr_res);
    if (rows > kMaxLaunchRows)           // (of one launch at a time, and fewer rows have more records each)
        for (const int of_launch : {kMaxLaunchRows, rows - kMaxLaunchRows}) {
            const size_t n = make_mfma_plan(kind, of_launch, d, r, V).records;
            if (n > p.records) p.records = n;
        }
    p.off_streams = off;       off = align_up(off + sizeof(float) * p.records * kStreamRecPlan);
    p.defer = (kind == HeadKind::Full ? d : r) >= kDeferMinKFine;      // room for it; the call decides (merge_parks_rows)
    if (p.defer) { p.off_defer = off; off = align_up(off + merge_defer_bytes(rows < kMaxLaunchRows ? rows : kMaxLaunchRows)); }
    p.bytes = off;
    return p;
}
// Rows of one launch of the matrix-core kernels.  More rows per launch would leave fewer column blocks (gw), hence
// fewer stream records per row, and a row whose top-k crowd into one record pays an exact rescan of that record's
// columns: at 512 rows a row still has 128 column blocks, with two or four records each.
inline int mfma_max_rows_per_launch(int rows) { return rows > kMaxLaunchRows ? kMaxLaunchRows : rows; }
// Rows that share a down-projection: those of two launches.
inline int mfma_joint_rows(HeadKind kind, int rows) {
    return kind == HeadKind::LowRank && rows > kMaxLaunchRows ? (rows < 2 * kMaxLaunchRows ? rows : 2 * kMaxLaunchRows) : mfma_max_rows_per_launch(rows);
}

// ---- few rows or long lists on the matrix cores, fp32-exact products (rows_head.hip) ----------------------------
constexpr int kRowsMaxRows = 48;         // rows per launch: three 16-row MFMA tiles (their accumulators: 96 registers)
constexpr int kRowsMaxColGroups = 6;     // 128-column groups per block at most (their logits: 149 KB of LDS at 48 rows)
constexpr int kRowsOneRoundCols = 256 * 128 * kRowsMaxColGroups;     // columns that 256 blocks cover, one per CU
// Floats between two rows of logits in shared memory; a row's place is reused for its candidates' 64-bit keys.
constexpr __host__ __device__ int rows_lds_stride(int G) { return (128 * G > 512 ? 128 * G : 512) + 8; }
// A block covers G groups of 128 columns in KS slices of the contraction (at most 8 wavefronts).  G is the
// smallest that needs at most 256 blocks, one round on the chip's CUs; what is left of the 8 wavefronts splits the
// contraction (more loads in flight, shorter chains of additions).  Wavefronts beyond G KS (a contraction of fewer
// steps than slices) only take their share of the rows' epilogues.
struct RowsGeom { int G = 1, KS = 1, waves = 8, chunks = 0; };
inline RowsGeom make_rows_geom(int K, int V) {
    RowsGeom g;
    const int groups = (V + 127) / 128, steps = (K + 31) / 32;
    g.G = (groups + 255) / 256;
    if (g.G > kRowsMaxColGroups) g.G = 4;
    g.KS = 8 / g.G;
    g.waves = g.G * g.KS;
    if (g.KS > steps) g.KS = steps;
    g.chunks = (groups + g.G - 1) / g.G;
    return g;
}
// The slices of the contraction are added at once, from a place of their own each, by all threads: the more slices and the fewer rows (only rows
// that exist are written), the more that saves.  (One after the other / at once, us a call: 8 slices, d = 4096, r = 512, V = 20000 8 rows 22.4 / 21.6,
// 16 rows 22.9 / 22.1, 32 rows 29.2 / 29.4, V = 32768 28.9 / 29.5; 4 slices, d = 1024, r = 128, V = 65536 3 rows 15.6 / 15.3, 8 rows 16.0 / 15.9, 16 rows 17.1 / 17.3.)
constexpr int kRowsMaxKS = 8;
constexpr size_t kRowsLdsLimit = 156 * 1024;
inline bool rows_meet_at_once(int KS, int rows) { return KS > 2 && KS <= kRowsMaxKS && rows <= (KS > 4 ? 16 : 8); }
constexpr __host__ __device__ int rows_meet_stride(int G) { return 128 * G + 4; }      // floats between two rows of a slice's sums
// What the epilogue of two rows needs in shared memory beside their logits, per wavefront: each row's candidates.
constexpr int kPairCand = 64;
constexpr int kPairMaxK = 32;            // longer lists take one row per wavefront
constexpr int kPairKeys = kPairCand + 2; // (the two rows' candidates in different banks)
// Bytes before the pieces of t that a block keeps: the rows' logits, the candidates.
constexpr __host__ __device__ size_t rows_x_offset(int NT, int G, int waves, int k) {
    return sizeof(float) * 16 * NT * (size_t)rows_lds_stride(G) + (k <= kPairMaxK ? sizeof(uint64_t) * 2 * kPairKeys * waves : 0);
}
// Shared memory of a block of rows_topk_kernel; meet_at: floats before the place where the slices' sums meet at once, 0: they meet otherwise
// (sum: the block keeps t's pieces, see rows_sum_slices).
struct RowsLds { size_t bytes = 0; int meet_at = 0; };
inline RowsLds rows_lds(int rows, int K, const RowsGeom &g, int k, bool sum) {
    const int NT = (rows + 15) / 16;
    RowsLds l;
    l.bytes = rows_x_offset(NT, g.G, g.waves, k) + (sum ? 3 * 16 * 16 * (size_t)((K + 63) / 64 * 8) : 0);
    const size_t meet = sizeof(float) * (size_t)(g.KS - 1) * rows * rows_meet_stride(g.G);
    if (NT == 1 && rows_meet_at_once(g.KS, rows) && l.bytes + meet <= kRowsLdsLimit) { l.meet_at = (int)(l.bytes / sizeof(float)); l.bytes += meet; }
    return l;
}
// What a launch before rows_topk_kernel reads ahead: the beginning of every slice of the contraction, in blocks of nw wavefronts.  How much: what
// comes while the launch's own blocks work; more makes it longer.  (Nothing / this, us a call: down_rows_kernel, 9 MB: 7 rows, d = 1024, r = 256, V = 30000
// 16.7 / 15.2; 5 rows, r = 128, V = 128256 18.0 / 17.0 (6 MB 17.2, 16 MB 17.0); 16 rows, d = 2048, r = 256, V = 65536 21.5 / 20.3 (6 MB 20.7, 16 MB 20.5); 12 rows in four
// positions, r = 200, V = 60000 18.7 / 17.9 (16 MB 18.4).  The slices of up to 8 rows, 8 MB: d = 4096, r = 256, V = 128256 25.0 / 24.4 (4 MB 25.1); 4 rows
// of the router 51.5 / 50.3.  The kernel that adds the slices, 4 MB: 12 rows, d = 4096, r = 512, V = 60000 28.4 / 27.2, 30 rows, d = 3000, r = 400, V = 20000 28.1 / 27.6, 23 rows
// 41.1 / 40.8, 40 rows, k = 32 52.1 / 51.7; not the tile kernel before it, which its loads delay: 40 rows, d = 6000, r = 1000, V = 100000 69.7 / 70.2, and 69.4
// with the former alone.  Nor the down-projection of one row, whose blocks fill the CUs: 32.2 / 32.1, 45.7 / 45.6.  Over 84 calls of 9 to 48 rows with the kernel that
// adds the slices 0.996 of the time.  With more than one round of blocks, V = 200000 to 1000000, what the later rounds' blocks find is less, and nothing is lost:
// 5 rows, d = 512, r = 64 0.93 (V = 262144) to 0.99, 7 rows, d = 1024, r = 256 0.98 to 1.00, 12 and 40 rows, d = 4096, r = 512 0.996 to 1.007, noise.)
constexpr int kAheadDownRows = 9 << 20, kAheadSlices = 8 << 20, kAheadFinish = 4 << 20;
inline ReadAhead rows_read_ahead(const uint16_t *M, int K, int V, const RowsGeom &g, int bytes, int nw) {
    ReadAhead a;
    const int steps = (K + 31) / 32, per = (steps + g.KS - 1) / g.KS;
    a.n_ranges = (steps + per - 1) / per;
    a.per = 32 * per;
    const int64_t fits = bytes / (2 * (int64_t)V * a.n_ranges);
    const int rows = fits < a.per ? (int)fits : a.per;       // of every slice
    if (rows < 1) return a;
    a.M = M; a.K = K; a.V = V;
    a.lanes = 16 * g.G;
    while (a.lanes > 64) { a.lanes /= 2; ++a.halves; }
    a.rows_step = 64 / a.lanes;
    a.n_t = (rows + a.rows_step - 1) / a.rows_step;
    a.chunks = g.chunks;
    a.n_units = (a.chunks + 7) / 8 << a.halves;
    a.q_n = (a.n_ranges * a.n_t + kAheadLoads - 1) / kAheadLoads;
    a.q_div = a.q_n / a.n_ranges; a.q_mod = a.q_n % a.n_ranges;
    const auto inverse = [](int n) { return (uint32_t)(((uint64_t(1) << 32) + n - 1) / n); };
    a.units_inverse = inverse(a.n_units); a.ranges_inverse = inverse(a.n_ranges);
    a.blocks = 8 * ((a.n_units * a.q_n + nw - 1) / nw);
    return a;
}
// Its down-projection in one launch (down_rows.hip) or in two (down_tile.hip).  One block per 16 columns of t reads all of h and
// of its columns of A, 32 bytes of every row: that takes longer than the second launch once there are many rows of either, and
// from 1 KB per row of A on they come from few of the L2's channels.  Calls at V = 32768 (one / two launches, us; rows of the largest
// group with one matrix): d = 1024, r = 128 5 rows 14.8 / 18.2, 23 rows 19.7 / 21.2, 40 rows 24.0 / 25.0; d = 2048, r = 256 5 rows 20.8 / 21.9, 16 rows
// 22.3 / 22.5, 23 rows 26.1 / 25.6, 12 rows in four groups 21.1 / 23.5; d = 4096, r = 512, V = 128256 5 rows 50.6 / 42.0.
inline int largest_group(const DownGrid &g) {
    int most = 0;
    for (int q = 0; q < g.n_groups; ++q) most = g.g_row0[q + 1] - g.g_row0[q] > most ? g.g_row0[q + 1] - g.g_row0[q] : most;
    return most;
}
inline bool down_rows_takes(const DownGrid &g, int d, int r) { return r <= 256 && (d <= 1024 || (d <= 2048 && largest_group(g) <= 16)); }
// Does that one launch read weights ahead?  It takes longer for it, the less it has to do itself (512 elements of d are one step of its wavefronts) and the
// longer the weights' way is: what is gained must be more.  (Nothing / 9 MB, us a call, the weights in the last-level cache and, in brackets, 600 MB of copies in
// turn: 8 rows, d = 256, r = 128, V = 30000 5 % (8) slower, d = 512 5 % (5), d = 768 2 % (3), d = 1024 1 % (0) faster; d = 512, r = 64, V = 65536 1 % (3)
// slower, r = 128, V = 60000 4 % faster (4 slower), d = 1024 7 % (2) faster; d = 384, r = 128, V = 128256 2 % faster (5 slower), d = 256 1 % faster (6 slower); 40 rows, d = 512,
// r = 64, V = 65536 1 % (1) faster, d = 384, r = 128, V = 60000 6 % faster (level).  Over 312 such calls 1.5 % (0.2) faster with these lines; without them 1.3 % faster
// (1.4 slower), 44 (141) of them by more than 1.5 % slower, up to 5 % (10), now none (30, up to 5 %).)
inline bool down_rows_reads_ahead(const DownGrid &g, int d, int r, int V) {
    const int64_t weights = (int64_t)r * V;
    return largest_group(g) > 16 ? d >= 512 || (d > 256 && weights >= 7000000) : d > 384 && d * weights >= 3500000000;
}

// Up to 8 rows: down_tile_kernel leaves 8 slices of t row by row (or fewer, where the contraction has no more), which every block of
// rows_topk_kernel adds itself, instead of a launch that does it once.  The number of slices, 0: not so.  (A launch / every block, us a call: 6 rows, d = 2056,
// r = 136, V = 8192 18.0 / 15.6; 7 rows, d = 1464, r = 288, V = 22984 20.6 / 18.6; 6 rows in six positions, r = 216 22.8 / 20.5; 5 rows, d = 3576, r = 256, V = 74504
// 26.7 / 25.6; 4 rows, d = 3600, r = 520 25.3 / 24.0; 4 rows of the router, d = 4096, r = 512, V = 128256 53.9 / 52.5; 8 rows 40.0 / 39.2.
// Not with 4 slices where 16 blocks' worth of the contraction are cut (4 rows, r = 520 26.7, 8 rows, r = 512 42.0), nor with more rows: 12 rows, r = 256 23.6 / 24.3.
// Not where blocks are more than one round, of which each adds the slices again: 8 rows, r = 256, V = 196608 33.8 / 32.5, V = 262144 48.7 / 51.3, r = 128,
// V = 1048576 101.9 / 110.6, 5 rows, r = 64, V = 524288 41.3 / 42.7; nor with long slices, of which 16 would be summed otherwise: 8 rows, d = 5120, r = 24 to
// 240 1 to 5 % faster, d = 6144 up to 2.5 % faster, r = 128, V = 128256 23.7 / 24.0, d = 8192, r = 24 18.9 / 19.2, r = 128, V = 128256 24.6 / 25.6.)
constexpr int kRowsSumRows = 8, kRowsMaxSlices = 8;
constexpr int kRowsSumFloats = 32768;    // of the slices, which every block reads; half of it beyond d = 4096
constexpr int kRowsSumHidden = 5120;
inline int rows_sum_slices(const DownGrid &g, int rows, int d, int r, int V) {
    if (rows > kRowsSumRows || r > 1024 || d > kRowsSumHidden || V > kRowsOneRoundCols || down_rows_takes(g, d, r)) return 0;
    const int n = g.slices < kRowsMaxSlices ? g.slices : kRowsMaxSlices;
    return rows * r * n <= (d <= 4096 ? kRowsSumFloats : kRowsSumFloats / 2) ? n : 0;
}

// The full head's rows as they lie in memory, or regrouped by a launch of their own (2 to 4 us).  A load of 16 rows touches 16 lines instead of 8, which are
// half used: a block waits longer for its rows, the more the more elements they have.  Nobody sees that where a block has one group of columns, or where
// the weights' way from HBM is the bound (four groups in a round that fills the chip).  It costs most where one wavefront takes a whole contraction
// (five and six groups) and V is no multiple of 64, so that the weights' loads touch more lines as well.  (Regrouped / as they lie, us a call, k = 10: 8 rows,
// d = 512, V = 8192 14.7 / 12.0, d = 8184, V = 50000 158.0 / 156.2; one group: 48 rows, d = 1360, V = 32000 32.5 / 31.5; four that fill: 48 rows, d = 1360, V = 120000
// 71.6 / 71.1; five, V = 151752: 32 rows, d = 1080 74.3 / 78.9, 24 rows, d = 2216, V = 131704 119.7 / 126.1; 16 rows, d = 4088, V = 50000 84.5 / 87.8; two: 32 rows, d = 1800, V = 50000
// 48.1 / 50.7, 40 rows, d = 1024, V = 41000 31.5 / 30.1; 40 rows, d = 1024, V = 151936 68.8 / 67.1, 48 rows, d = 1360 87.0 / 90.0; others: 33 rows, d = 1024, V = 80000 45.2 / 44.0,
// 48 rows, d = 1024, V = 100000 54.5 / 56.7, d = 1360, V = 140000 85.0 / 94.3.  Of 3467 calls of 2 to 48 rows, d = 272 to 8176, V = 8192 to 190016, these lines leave 13 more than
// 0.5 % slower than regrouped, one more than 1 % (1.8 %), the mean 5.4 % faster; rows * d < 65536 alone left 202, up to 10 %.)
constexpr int kFillingChunks = 232;      // blocks from which on the chip counts as full
inline bool rows_read_by_rows(int rows, int d, int V, const RowsGeom &g) {
    const bool fills = g.chunks >= kFillingChunks;
    const int most = rows <= 8 || g.G == 1 || (g.G == 4 && fills) ? 65536
                   : g.G > 4 && V % 64 != 0 ? 20000
                   : rows <= 24 ? 60000
                   : g.G == 2 ? (fills ? 58000 : 50000)
                   : fills ? 50000 : 36000;
    return (int64_t)rows * d < most;
}
// Contractions this path takes: its row operand and partial tiles then fit beside the lists in a few tens of MB.
inline bool rows_path_fits(HeadKind kind, int d, int r) { return kind == HeadKind::LowRank ? r <= 2048 : d <= 8192; }

struct RowsPlan {
    int rows = 0, rows_pad = 0, pieces = 1;
    RowsGeom geom;
    DownGrid down;
    size_t off_down_part = 0;            // fp32 partial tiles of t (low-rank head; sized for any grouping of the rows)
    size_t off_x = 0;                    // 16-byte vectors [pieces][8 ceil(K / 64)][rows_pad]
    size_t off_part_ms = 0, off_part_val = 0, off_part_id = 0, off_part_smp = 0;      // as in Plan, [rows, chunks]
    size_t bytes = 0;
};
// rows: of one launch, at most kRowsMaxRows
inline RowsPlan make_rows_plan(HeadKind kind, int rows, int d, int r, int V, int k) {
    RowsPlan p;
    const int K = kind == HeadKind::LowRank ? r : d;
    p.rows = rows;
    p.rows_pad = (rows + 15) / 16 * 16;
    p.pieces = kind == HeadKind::LowRank ? 3 : 1;
    p.geom = make_rows_geom(K, V);
    size_t off = 0;
    if (kind == HeadKind::LowRank) {
        p.down = make_down_grid(rows, p.rows_pad, d, r);
        p.off_down_part = off; off = align_up(off + sizeof(float) * 4096 * down_part_tiles_bound(rows, r));
    }
    p.off_x = off;         off = align_up(off + 16 * (size_t)p.pieces * p.rows_pad * ((K + 63) / 64 * 8));
    const size_t n = (size_t)rows * p.geom.chunks;
    p.off_part_ms = off;   off = align_up(off + 2 * sizeof(float) * n);
    p.off_part_val = off;  off = align_up(off + sizeof(float) * n * k);
    p.off_part_id = off;   off = align_up(off + sizeof(int32_t) * n * k);
    p.off_part_smp = off;  off = align_up(off + 16 * n);
    p.bytes = off;
    return p;
}

// ---- merge of the chunk lists (merge_kernel.hip) -------------------------------------------------------------------
// Short lists take code of their own as long as the block's threads hold all entries, eight each, and a chunk each: up to 16 ids, and up to 10 in a launch
// of more than 24 rows with up to 128 lists each.  The bound it works with is the smallest maximum of k classes.  A class of few lists has few heads, and
// now and then the bound admits many more than k entries, the more the larger k; the slowest row decides how long the launch takes, and of many rows
// one is such a row.  (The other code / this one, mean over five to eight inputs: d = 512, r = 64, V = 8632, us a call 42 rows k = 10 17.2 / 17.3, k = 11 17.6 / 19.1,
// k = 13 18.2 / 18.4, 32 rows k = 11 15.0 / 15.4, k = 13 15.5 / 15.9, 24 rows k = 11 14.3 / 14.0, 12 rows 12.6 / 12.3; V = 16384, 42 rows, k = 13 18.1 / 18.9.  k = 11 to 16 of 28 to
// 48 rows: 64 lists 0.92 to 0.99 of its time, 100 lists 0.97 to 1.00, 130 to 250 lists 0.97 to 1.03, among them the full head, 32 rows, d = 992, V = 52064, k = 12 32.0 / 31.7.)  Long ones
// are requested before the bound is known up to five entries per thread: with more, fetching what the bound leaves out takes longer than the second
// trip to memory (d = 1024, r = 128, us a call, requested / not: 4 rows, V = 20480, k = 24 13.9 / 13.5, V = 8192, k = 48 15.9 / 15.3, 40 rows, V = 16384,
// k = 30 24.4 / 23.6, one row, V = 20480, k = 24 12.0 / 11.5).
constexpr int kRowMergeThreads = 512;
constexpr int kMergeShort = 16, kMergeShortFewLists = 10;      // ids of a short list at most, and of ...
constexpr int kMergeFewRows = 24, kMergeFewLists = 128;  // ... a launch of more rows than these with up to these lists each
constexpr int kMergeAhead = 8;           // entries per thread of short lists
constexpr int kMergeAheadLong = 5;       // ... of long ones
// ids in the last chunk's list (the others have k)
inline int merge_last_len(int chunks, int chunk_cols, int V, int k) {
    const int last_cols = V - (chunks - 1) * chunk_cols;
    return last_cols < k ? last_cols : k;
}
inline bool merge_short_lists(int rows, int chunks, int last_len, int k) {
    return k <= (rows > kMergeFewRows && chunks <= kMergeFewLists ? kMergeShortFewLists : kMergeShort)
        && chunks <= kRowMergeThreads && (chunks - 1) * k + last_len <= kMergeAhead * kRowMergeThreads;
}

// ---- which kernels a call runs ------------------------------------------------------------------------------------
constexpr int kMfmaMaxK = 16;            // the lane streams keep 3 groups: enough for k <= 16 (larger k: rows_head.hip)
constexpr int64_t kRowsMinWeights = 12 << 20;
constexpr int kMfmaMinRows = 5;          // below, rows whose calls rows_path_takes leaves are streamed in lock step

// Few rows, or lists longer than the lane streams keep (rows_head.hip); the rest is tile_path_takes's or streamed.
// Where the lines lie (us per call at d = 4096, r = 512, V = 128256 unless said otherwise; the other path's time first,
// this one's second):
//   * k > kMfmaMaxK: always; the lane-owns-columns kernel reads the weights once per 8 rows (40 rows, k = 32: 420 / 52).
//   * 3 and 4 rows, low-rank: the streaming kernel needs no kernel that finishes t.  It is level or a little behind up to 256 chunks of 512
//     columns (one round of its blocks) while r is small: r = 256 27.4 / 28.6, 384 33.8 / 35.8, r = 256, V = 64000 25 / 25; behind where t takes one
//     short launch (d = 512, r = 64, V = 16384 15.6 / 13.1, d = 1024, r = 128, V = 32768 16.7 / 14.6, V = 128256 21.5 / 20.2, r = 256, V = 65536 22.0 / 20.3)
//     and beyond 256 chunks (V = 151936: r = 256 39.4 / 29.1, r = 512 57.6 / 39.6; but of the smallest weights r = 16 18.0 / 19.3, r = 64 22.5 / 19.9).
//   * 2 rows, low-rank: level up to 256 chunks (r = 512 39.1 / 41.8, r = 256 26.3 / 28.5, d = 2048, r = 256, V = 32768 17.4 / 20.3, d = 1024,
//     r = 128 14.5 / 14.7).  This kernel from d = 512 down while t takes one launch (r = 16, V = 8192 13.3 / 12.5, r = 64 13.6 / 13.5, r = 256, V = 32768
//     15.1 / 16.3, V = 128256 23.7 / 22.4), not where it takes two (r = 264, V = 32768 15.8 / 19.0, V = 128256 23.1 / 26.5, r = 512 17.3 / 20.5 and 31.4 / 34.2,
//     r = 1024, V = 32768 25.1 / 27.4).  Beyond 256 chunks this kernel (V = 151936: r = 512 53.1 / 42.5, r = 256 33.9 / 28.7, r = 128 25.4 / 23.8, d = 1024,
//     r = 64 19.8 / 16.9), but not with small weights behind two launches (d = 4096, r = 16 17.1 / 18.6, r = 64 20.5 / 21.2), nor where its blocks are
//     more than one round (V = 200000: r = 16 17.6 / 22.5, r = 64 21.3 / 26.1, r = 512 56.0 / 58.5, d = 1024, r = 64 20.8 / 21.8; V = 262144: r = 64
//     22.4 / 28.8, r = 512 62.2 / 70.4).
//   * full head, from 2 rows: 188.9 / 185.3; d = 1024, V = 8192 24.3 / 17.8.  Two rows with d = 256, V = 32000: 15.7 / 16.4.
//   * up to 32 rows, k <= kMfmaMaxK: 23 rows 50.9 / 40.5, 32 rows 51.7 / 41.3 (the weights in the last-level cache; with prepared ones the other path takes
//     51.2 and 51.9).
//   * 33 to 48 rows: a wavefront finishes up to six rows after the weights, which a short contraction does not pay for,
//     while head_tile_kernel's cost stays the same and its merge is cheap with prepared weights or few candidates.
//       prepared: 33 rows 51.0 / 54.4, 48 rows 51.5 / 58.9 (r = 1024: 76.8 / 84.1); this kernel only where few tiles of the
//         vocabulary leave head_tile_kernel long contractions on few CUs (48 rows, r = 2048: V = 32000 74 / 68, V = 8192 68 / 53)
//         and for the smallest ranks, where the head kernel is short beside its merge of 9 us (60 rows, r = 64, V = 14000: 4 + 4 for t, 9, 9) and
//         this kernel's merge takes 4 (33 and 48 rows, d = 512: r = 16, V = 8192 26.3 / 15.9 and 26.5 / 17.1, r = 64, V = 32000 28.0 / 18.1 and
//         29.3 / 19.5, V = 128256 32.5 / 22.2 and 32.7 / 24.1; d = 4096, r = 64, V = 128256 32.6 / 26.6 and 32.7 / 28.0);
//       plain low-rank calls stay, and with them their fp32 t: 48 rows, k = 10 0.99 to 1.4 times as fast; with k = 3 and r = 256
//         they give up a little (40 rows, V = 8192 30.9 / 33.1, 48 rows, V = 32000 34.1 / 36.9);
//       full head, k = 4, 48 rows: d = 256 22.7 / 28.8 at V = 32000, 30.0 / 34.4 at V = 128256; d = 1024 41.8 / 36.0 and 67.3 / 66.3.
//         The other path's re-evaluated columns cost in proportion to k d, this one's epilogue to V: it is behind up to d = 768 while
//         k d stays below about 17 sqrt(V) and k below 16 (V = 8192: k = 4, d = 256 22.8 / 26.9, 36 rows, k = 6, d = 512 31.6 / 26.6; V =
//         128256: k = 10, d = 512 46.1 / 47.0, k = 16 51.8 / 47.4), not with so small a V that head_tile_kernel's blocks are few (d = 768, V = 8192, k = 1 28.3 / 25.3).
//     Sampling calls stay, prepared ones too: the draw is dearer in head_tile_kernel and its merge (48 rows: r = 64, V = 8192 41.0 / 20.9, r = 256, V = 32000
//     47.5 / 32.3, r = 512, V = 128256 73.3 / 58.4, prepared 67.8 / 58.5).
//   * more rows would need a second launch, and lose.
inline bool rows_path_takes(HeadKind kind, int rows, int d, int r, int V, int k, bool prepared, bool sampling) {
    const bool low_rank = kind == HeadKind::LowRank;
    if (rows < 2 || !rows_path_fits(kind, d, r)) return false;
    if (low_rank && rows == 2) {
        if (V <= 256 * kChunkCols) return d <= 512 && r <= 256;
        return V <= kRowsOneRoundCols && ((d < 2048 && r <= 256) || (int64_t)r * V >= kRowsMinWeights);
    }
    if (low_rank && rows <= 4)
        return (d < 2048 && r <= 256) || ((int64_t)r * V >= kRowsMinWeights && (V > 256 * kChunkCols || r > (V > 65536 ? 384 : 256)));
    if (k > kMfmaMaxK) return true;
    if (!low_rank && rows == 2) return d > 256;
    if (rows > kRowsMaxRows) return false;
    if (rows <= 32 || sampling) return true;
    if (!low_rank) return d > 768 || k > 10 || V < 16 * d || (int64_t)k * d * k * d > (int64_t)300 * V;
    return !prepared || r <= 64 || (r >= 1024 && V <= 16 * r);
}

inline bool tile_path_takes(int rows, int k) { return rows >= kMfmaMinRows && k <= kMfmaMaxK; }

// What the many-row kernels multiply the weights with: the bf16 rows of the full head, or t log2(e) rounded to bf16, to f16, or to
// two bf16 pieces (its sixteen leading bits).
enum Operand : int { kOperandExact, kOperandBf16, kOperandF16, kOperandTwoBf16 };

// The direct-to-LDS kernel takes bf16 operands as they are, or turns the weight tiles into f16 inside LDS and takes an f16
// t (8 times finer).  The conversion costs the projection kernel about 12 %; the finer operand saves most of the merge's
// exact re-evaluations, which grow with k: measured break-even at k = 10, 5-9 % of the call in favour of f16 at k = 16.
// With a column-major copy the re-evaluations cost little: bf16 as it is.
inline bool tile_operand_f16(int k, bool prepared) {
#ifdef SLIMSPEC_DIAG_OPERAND_F16      // experiment builds only: force the operand mode (1 f16, 0 bf16)
    return SLIMSPEC_DIAG_OPERAND_F16 != 0 && !prepared;
#endif
    return k > 12 && !prepared;
}
// Ranks up to 64 (kTwoPiecesMaxRank) take two bf16 pieces instead of one: with so few terms the columns' norms differ from each other by
// a tenth and more, the bound on one piece's error does not hold for all of them, and a row that finds out is evaluated exhaustively.
// The second piece costs head_resident_kernel, whose contraction is padded to 128, nothing, and head_tile_kernel a stage or two.  (One
// piece / two, us a call: 375 rows, d = 584, r = 40, V = 64120, prepared 206-289 / 34.7; 129 rows, r = 56, V = 151936, prepared 237.6 / 42.3;
// 512 rows, d = 1024, r = 64, V = 128256 234.3 / 56.1; 100 rows, r = 24, V = 128256, prepared 241.9 / 31.5; 64 rows, r = 16, V = 8192 66.4 / 28.9,
// 27.5 where no row finds out; 60 rows, r = 64, V = 14000, prepared, none finds out, 27.4 / 28.2; 100 rows, r = 64, V = 32000 33.0 / 32.5.  From r = 72
// on none of some 20 calls found out.  Relative error of the log-probabilities against 64 bits, a dozen calls: 1.2e-4 to 2.5e-4 / 4e-7 to 9e-7.)
inline Operand tile_operand(int r, int k, bool prepared) {
    return tile_operand_f16(k, prepared) ? kOperandF16 : r <= kTwoPiecesMaxRank ? kOperandTwoBf16 : kOperandBf16;
}

// head_resident_kernel instead of head_tile_kernel: bf16 operands.
inline bool resident_takes(const MfmaPlan &p, bool f16_operand) { return p.resident && !f16_operand; }

}  // namespace slimspec
