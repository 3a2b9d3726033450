// Streaming ("lane owns columns") kernels for calls with few rows, where the head
// is bound by reading the weight matrix once from HBM (paper section 4.1: the
// O(rd + Vr) low-rank head and the O(Vd) full head).
//
//   down_items_kernel     t = h A as slices over d, one block per (64 columns of A) x (slice of d)
//   stream_topk_kernel    z[:, chunk] = x M[:, chunk] for a chunk of 64 to 512 columns, then the
//                         chunk's running max, sum of exp and top-k, one partial per
//                         (row, chunk); no logit is written to memory
//   widen_rows_kernel     bf16 h -> fp32 (contraction input of a full head whose rows do not fit shared memory)
#include "gemv_parts.hpp"
#include "launch.hpp"
#include <type_traits>

namespace slimspec {

// ---------------------------------------------------------------------------
// t = h A for up to R rows, as slices: block = one item (64 columns of A x a slice of d, read as
// full 128-byte lines); tpart is [nds][R][r] and the consumer adds the nds slices in order.
constexpr int kDownThreads = 1024;

template <int R, bool POS>
__global__ __launch_bounds__(kDownThreads) void down_items_kernel(
    const uint16_t *__restrict__ h, const uint16_t *__restrict__ A, float *__restrict__ tpart,
    int rows_here, int d, int r, int n_cb, int slice, RowMats mats)
{
    __shared__ float redd[kDownThreads / 64][R][kItemCols];
    down_item<R, kDownThreads, POS>(redd, h, A, tpart, blockIdx.x, n_cb, slice, rows_here, d, r, threadIdx.x, mats);
}

__global__ __launch_bounds__(256) void widen_rows_kernel(
    const uint16_t *__restrict__ h, float *__restrict__ x, int n)
{
    int e = blockIdx.x * 256 + threadIdx.x;
    if (e < n) x[e] = bf16_to_float(h[e]);
}

// ---------------------------------------------------------------------------
// One block per chunk of 8 * lanes adjacent columns of the vocabulary.  M is the [K, V] weight matrix (bf16 or fp32).
// A lane owns 8 adjacent columns; a wavefront's 64 lanes are 64 / lanes (`k_parts`) rows of M at a time, so a narrow
// chunk fills the wavefront as well, and the NW k_parts lane groups of a block split the contraction into ranges of
// `per` rows (a multiple of 8).  Their partial sums meet in shared memory in a fixed order, and wavefront i % NW (a single row in a wide chunk: the
// block, block_row_epilogue) reduces row i of the chunk to (max, sum of exp, top-k) and writes the partial.
//
// What bounds it: the weights' way from HBM, as long as every CU has a block and asks for enough of them (plan.hpp chooses
// the chunks for that); with small weights the chain of trips before and after: the contraction input (for one or two
// rows as a rule one trip: all of a thread's loads are requested together, and the first weights right behind them), the weights, the
// epilogue of one wavefront (a single row in a wide chunk: of the block).
//
// Measured, one row (kernel; chunks of 512 columns and x as it comes, before, in brackets): full head, d = 7984, V = 37208 96 us
// (180), d = 3208, V = 33184 38 (70); r = 1568, V = 40248 25.2 (44); r = 72, V = 103472 7.2 (10.5); d = 4096, V = 128256, where
// the chunks are the same, 169.9 (171.3, and 4.7 in a launch that widened the row to fp32).  3 rows, r = 496, V = 19072 15.2 (22.3).
//
// SRC: what x is.  kSlices: nds partial sums of the contraction input, [nds][R][K] fp32 (down_items_kernel's); four
// adjacent lanes add a quarter of the slices each.  kHalfRows: the bf16 rows themselves, [rows_here][K] (full head).  Both
// are put into shared memory.  kGlobal: fp32 [R][K], read from memory (rows too long for that; k_parts is 1).
// kOwn: one row, x_src is h [d], nds is d, and every block makes t = h A itself from A [d, K]: a launch less for what the block waits longer, at
// most a few trips to the L2 (plan.hpp: own_input_takes).
enum { kGlobal = 0, kSlices = 1, kHalfRows = 2, kOwn = 3 };

// t = h A of one row into xs (shared memory), by the whole block: 64 columns at a time, a thread 8 of them in every
// `slots`-th row, `then` (the weights' first loads) behind the last of A's.
template <int NT, class Then>
__device__ __forceinline__ void own_input(const uint16_t *__restrict__ h, const uint16_t *__restrict__ A, float (*redd)[kItemCols],
                                          float *xs, int d, int r, int tid, Then then)
{
    constexpr int NW = NT / 64, U = 8;
    const int lane = tid & 63, wave = tid >> 6;
    const int pl = r > 32 ? 3 : r > 16 ? 2 : r > 8 ? 1 : 0;     // 2^pl adjacent threads cover a row's columns (64 of them at most)
    const int piece = tid & ((1 << pl) - 1), slot = tid >> pl, slots = NT >> pl;
    for (int c0 = 0; c0 < r; c0 += kItemCols) {
        const int col = c0 + piece * 8;
        float acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.f;
        for (int j0 = 0; j0 < d; j0 += U * slots) {
            const int j = j0 + slot;
            uint4 w[U];
            uint16_t hv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (j0 + u * slots >= d) break;                // (the same for the whole block)
                const int row = min(j + u * slots, d - 1);
                w[u] = *reinterpret_cast<const uint4 *>(A + (size_t)row * r + min(col, r - 8));
                hv[u] = h[row];
            }
            if (c0 + kItemCols >= r && j0 + U * slots >= d) then();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (j + u * slots >= d) continue;
                const float f[8] = {bf16_lo(w[u].x), bf16_hi(w[u].x), bf16_lo(w[u].y), bf16_hi(w[u].y),
                                    bf16_lo(w[u].z), bf16_hi(w[u].z), bf16_lo(w[u].w), bf16_hi(w[u].w)};
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] = fmaf(bf16_to_float(hv[u]), f[e], acc[e]);
            }
        }
        // the lanes that hold the same columns
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float v = acc[e];
            if (pl < 1) v += dpp_f32<0xB1>(v);
            if (pl < 2) v += dpp_f32<0x4E>(v);
            if (pl < 3) v += dpp_f32<0x141>(dpp_f32<0x1B>(v));  // lane ^ 4
            v += dpp_f32<0x128>(v);                             // lane ^ 8
            uint32_t a, b;
            swap_pair<16>(__float_as_uint(v), a, b);
            v = __uint_as_float(a) + __uint_as_float(b);
            swap_pair<32>(__float_as_uint(v), a, b);
            v = __uint_as_float(a) + __uint_as_float(b);
            if (lane < (1 << pl)) redd[wave][lane * 8 + e] = v;
        }
        __syncthreads();
        if (tid < kItemCols && c0 + tid < r) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) s += redd[w][tid];     // fixed order
            xs[c0 + tid] = s;
        }
        if (c0 + kItemCols < r) __syncthreads();
    }
}

template <int R, int NW, typename WT, int SRC>
__global__ __launch_bounds__(NW * 64) void stream_topk_kernel(
    const void *__restrict__ x_src, int nds, const uint16_t *__restrict__ A, const WT *__restrict__ M,
    float2 *__restrict__ part_ms, float *__restrict__ part_val, int *__restrict__ part_id,
    int rows_here, int row0, int K, int V, int chunks, int lanes, int k_parts, StreamParts sp, int k,
    float4 *__restrict__ part_smp, uint32_t seed_lo, uint32_t seed_hi)
{
    constexpr int NT = NW * 64, EW = (R < NW) ? R : NW;
    extern __shared__ __align__(16) unsigned char dyn[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Blocks are dealt round-robin to the 8 XCDs: adjacent chunks, which share a cache line per row of M wherever the rows
    // are no multiples of 128 bytes, go to one XCD.
    const int per_xcd = (chunks + 7) >> 3;
    const int chunk = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (chunk >= chunks) return;
    int kp = 0;                                             // lane / lanes
    for (int first = lanes; first < 64; first += lanes) kp += lane >= first ? 1 : 0;
    const int g = lane - kp * lanes;
    const int cw = 8 * lanes, chunk_col = chunk * cw, col = chunk_col + 8 * g;
    const bool active = kp < k_parts && col < V;          // V is a multiple of 8: all 8 columns valid or none

    __shared__ std::conditional_t<R == 1, BlockRowLds, char> one_row;
    BlockRowPlan row_plan;
    const auto plan_row = [&]() {                               // (behind the first loads)
        if constexpr (R == 1) {
            if (!block_row_takes(cw, k)) return;
            row_plan = make_block_row_plan(cw, chunk_col, V, k);
            if (tid < kBoundGroups && tid >= row_plan.bound.n_groups) one_row.groups[tid] = 0u;
        }
    };

    float acc[R][8];
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[i][e] = 0.f;

    // Rows [j0, j1) of M for this wavefront, 8 k_parts at a time of which lane group kp takes the eight from 8 kp on: the
    // rows' addresses are the same in all lanes but for an offset kept in one register.  K is a multiple of 8.
    const int n_parts = sp.n, step = 8 * k_parts;
    const int j0 = min(K, wave * sp.per), j1 = min(K, j0 + sp.per);
    float *red = reinterpret_cast<float *>(dyn);                              // [n_parts][R][cw]
    float *red2 = red + n_parts * R * cw;                                     // [kSumParts][R][cw] if n_parts > kDirectParts
    uint64_t *sel = reinterpret_cast<uint64_t *>(red2 + (n_parts > kDirectParts ? kSumParts * R * cw : 0));      // [EW][cw]
    unsigned char *xs_raw = reinterpret_cast<unsigned char *>(sel + EW * cw);                                   // x: [R][K], fp32 (kSlices) or bf16
    constexpr int U = (sizeof(WT) == 2 && R <= 2) ? 16 : 8, UG = U / 8;
    using RawT = decltype(load_raw8(static_cast<const WT *>(nullptr)));
    const uint32_t off = active ? (uint32_t)(8 * kp) * (uint32_t)V + (uint32_t)col : 0u;      // (8 k_parts rows of at most 2^17 columns when k_parts > 1)
    const auto load_row = [&](int j) { return load_raw8(M + (size_t)j * V + off); };          // row j + 8 kp

    if constexpr (SRC != kGlobal) {
        RawT q[U];
        const auto load_batch = [&](int j) {
#pragma unroll
            for (int u = 0; u < U; ++u) q[u] = load_row(j + (u >> 3) * step + (u & 7));
        };
        // (where the wavefront's range ends inside it, a lane group without rows reads the first group's)
        const bool in_first = active && j0 < j1;
        const auto load_first = [&]() {
            if (!in_first) return;
#pragma unroll
            for (int g8 = 0; g8 < UG; ++g8) {
                if (g8 > 0 && j0 + g8 * step >= j1) continue;   // (the same for the whole wavefront)
                const bool have = j0 + g8 * step + 8 * kp < j1;
                const uint32_t o = have ? off : (uint32_t)col;
#pragma unroll
                for (int u = 0; u < 8; ++u) q[8 * g8 + u] = load_raw8(M + (size_t)(j0 + g8 * step + u) * V + o);
            }
        };
        if constexpr (SRC == kOwn) {
            __shared__ float redd[NW][kItemCols];
            own_input<NT>(static_cast<const uint16_t *>(x_src), A, redd, reinterpret_cast<float *>(xs_raw), nds, K, tid, load_first);
        } else if constexpr (SRC == kSlices) {
            const float4 *x = static_cast<const float4 *>(x_src);
            float4 *xs = reinterpret_cast<float4 *>(xs_raw);
            const uint32_t n4 = (uint32_t)(R * K) / 4u, sg = tid & 3u, last = (uint32_t)nds - 1u;
            constexpr uint32_t SL = 8;                          // slices of a lane: sg, sg + 4, ... (at most 32 in all: make_down_plan)
            float4 v[SL];
            const auto load_slices = [&](uint32_t e) {
                if (e >= n4) return;                            // (a wavefront of none goes on to its weights)
#pragma unroll
                for (uint32_t u = 0; u < SL; ++u) {
                    if (4u * u > last) { v[u] = make_float4(0.f, 0.f, 0.f, 0.f); continue; }      // few slices: not the last one again and again
                    v[u] = x[min(sg + 4u * u, last) * n4 + e];
                }
            };
            const auto add_slices = [&](uint32_t e) {
                float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (uint32_t u = 0; u < SL; ++u) {
                    const uint32_t on = sg + 4u * u <= last ? 0xffffffffu : 0u;      // (a condition becomes a branch per slice)
                    const auto kept = [&](float f) { return __uint_as_float(__float_as_uint(f) & on); };
                    s.x += kept(v[u].x); s.y += kept(v[u].y); s.z += kept(v[u].z); s.w += kept(v[u].w);
                }
                const auto quad = [](float f) { f += dpp_f32<0xB1>(f); return f + dpp_f32<0x4E>(f); };
                s.x = quad(s.x); s.y = quad(s.y); s.z = quad(s.z); s.w = quad(s.w);
                if (sg == 0 && e < n4) xs[e] = s;
            };
            uint32_t e = (uint32_t)tid >> 2;
            for (uint32_t e0 = 0; e0 + NT / 4 < n4; e0 += NT / 4, e += NT / 4) { load_slices(e); add_slices(e); }
            load_slices(e);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (R <= 2) load_first();                 // behind the last of them: vector memory returns in order
            __builtin_amdgcn_sched_barrier(0);
            add_slices(e);
            // More rows have several float4 per lane, and the weights in flight then delay the last of them more than they gain
            // (before / behind the sum: 4 rows, d = 512, r = 264, V = 128256 26.4 / 25.4 us a call, d = 8192, r = 1024, V = 8192 30.9 / 28.8).
            if constexpr (R > 2) load_first();
        } else {
            uint4 *xs = reinterpret_cast<uint4 *>(xs_raw);
            const int n8 = rows_here * K / 8;                   // rows beyond the last stay undefined: nobody reads their sums
            const uint4 *x = static_cast<const uint4 *>(x_src);
            for (int e0 = 0; e0 < n8; e0 += NT) {
                const uint4 v = x[min(e0 + tid, n8 - 1)];
                if (e0 + NT >= n8) load_first();
                if (e0 + tid < n8) xs[e0 + tid] = v;
            }
        }
        plan_row();
        __syncthreads();
        const auto fma_group = [&](const RawT *w, int j) __attribute__((always_inline)) {      // rows j + 8 kp ... of the lane group
            float xv[R][8];
#pragma unroll
            for (int i = 0; i < R; ++i) {
                if constexpr (SRC != kHalfRows) {
                    const float4 *p = reinterpret_cast<const float4 *>(xs_raw) + (i * K + j) / 4 + 2 * kp;
                    const float4 a = p[0], b = p[1];
                    xv[i][0] = a.x; xv[i][1] = a.y; xv[i][2] = a.z; xv[i][3] = a.w;
                    xv[i][4] = b.x; xv[i][5] = b.y; xv[i][6] = b.z; xv[i][7] = b.w;
                } else
                    widen8(Raw8Bf16{reinterpret_cast<const uint4 *>(xs_raw)[(min(i, rows_here - 1) * K + j) / 8 + kp]}, xv[i]);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                float f[8];
                widen8(w[u], f);
#pragma unroll
                for (int i = 0; i < R; ++i)
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[i][e] = fmaf(xv[i][u], f[e], acc[i][e]);
            }
        };
        if (active) {
            int j = j0;
#pragma unroll
            for (int g8 = 0; g8 < UG; ++g8)
                if (j + g8 * step + 8 * kp < j1) fma_group(q + 8 * g8, j + g8 * step);
            j += UG * step;
            for (; j + UG * step <= j1; j += UG * step) {
                load_batch(j);
#pragma unroll
                for (int g8 = 0; g8 < UG; ++g8) fma_group(q + 8 * g8, j + g8 * step);
            }
            for (; j < j1; j += step)
                if (j + 8 * kp < j1) {
                    RawT w[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) w[u] = load_row(j + u);
                    fma_group(w, j);
                }
        }
    } else {
      plan_row();
      if (active) {
        const float *x = static_cast<const float *>(x_src);
        const auto rows_from = [&](int j, auto n_tag) {         // (k_parts is 1)
            constexpr int N = decltype(n_tag)::value;
            RawT q[N];
#pragma unroll
            for (int u = 0; u < N; ++u) q[u] = load_row(j + u);
#pragma unroll
            for (int u = 0; u < N; ++u) {
                float f[8];
                widen8(q[u], f);
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const float xv = x[(size_t)i * K + j + u];
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[i][e] = fmaf(xv, f[e], acc[i][e]);
                }
            }
        };
        int j = j0;
        for (; j + U <= j1; j += U) rows_from(j, std::integral_constant<int, U>{});
        if constexpr (U > 8)
            for (; j < j1; j += 8) rows_from(j, std::integral_constant<int, 8>{});
      }
    }
    const int part = wave * k_parts + kp;
    if (kp < k_parts && part < n_parts) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            float4 *dst = reinterpret_cast<float4 *>(red + (part * R + i) * cw + 8 * g);
            dst[0] = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
            dst[1] = make_float4(acc[i][4], acc[i][5], acc[i][6], acc[i][7]);
        }
    }
    __syncthreads();
    if (R == 1 && block_row_takes(cw, k)) {
        if constexpr (R == 1) block_row_epilogue<NW>(one_row, row_plan, red, n_parts, cw, chunk_col, tid, k, (size_t)row0 * chunks + chunk, part_ms, part_val, part_id, part_smp,
                               gumbel_key(seed_lo, seed_hi, (uint32_t)row0));
        return;
    }
    // many lane groups (narrow chunks): every thread adds some of their sums first
    const float *sums = red;
    int n_sums = n_parts;
    if (n_parts > kDirectParts) {
        const int n2 = R * cw / 2;                              // pairs of columns
        for (int item = tid; item < kSumParts * n2; item += NT) {
            const int p0 = item / n2, c2 = item - p0 * n2;
            float2 s = make_float2(0.f, 0.f);
            for (int p = p0; p < n_parts; p += kSumParts) {
                const float2 v = reinterpret_cast<const float2 *>(red)[p * n2 + c2];
                s.x += v.x; s.y += v.y;
            }
            reinterpret_cast<float2 *>(red2)[item] = s;
        }
        __syncthreads();
        sums = red2;
        n_sums = kSumParts;
    }
    const auto finish = [&](auto e_tag, auto topk_tag, auto draw_tag, int i) {
        chunk_row_epilogue<decltype(e_tag)::value, decltype(topk_tag)::value, decltype(draw_tag)::value>(
            sums + i * cw, n_sums, R * cw, cw, chunk_col, V, lane, k, sel + (wave % EW) * cw, (size_t)(row0 + i) * chunks + chunk,
            part_ms, part_val, part_id, part_smp, gumbel_key(seed_lo, seed_hi, (uint32_t)(row0 + i)));
    };
    const auto finish_row = [&](auto topk_tag, auto draw_tag, int i) {
        if (cw <= 128) finish(std::integral_constant<int, 2>{}, topk_tag, draw_tag, i);
        else if (cw <= 256) finish(std::integral_constant<int, 4>{}, topk_tag, draw_tag, i);
        else finish(std::integral_constant<int, 8>{}, topk_tag, draw_tag, i);
    };
    // The block's tail, which nothing overlaps: a row's top-k by one wavefront, its draw by another where there are twice as many.
    if constexpr (2 * R <= NW) {
        if (wave < rows_here) finish_row(std::true_type{}, std::false_type{}, wave);
        else if (part_smp && wave >= R && wave < R + rows_here) finish_row(std::false_type{}, std::true_type{}, wave - R);
    } else {
        for (int i = wave; i < rows_here; i += NW) finish_row(std::true_type{}, std::true_type{}, i);
    }
}

// ---------------------------------------------------------------------------
// launchers

template <int R>
static hipError_t launch_down(const uint16_t *h, const uint16_t *A, float *tpart,
                              int rows_here, int d, int r, const DownPlan &fp, const int *mat_of_row, hipStream_t st)
{
    RowMats mats{};
    bool one_matrix = true;
    for (int i = 0; i < rows_here && i < 8; ++i) {
        mats.m[i] = mat_of_row ? mat_of_row[i] : 0;
        one_matrix = one_matrix && mats.m[i] == mats.m[0];
    }
    if (one_matrix)        // every row uses the same matrix: the weights are loaded once for all rows
        down_items_kernel<R, false><<<fp.n_items, kDownThreads, 0, st>>>(h, A + (size_t)mats.m[0] * d * r, tpart, rows_here, d, r,
                                                                         fp.n_cb, fp.slice, mats);
    else
        down_items_kernel<R, true><<<fp.n_items, kDownThreads, 0, st>>>(h, A, tpart, rows_here, d, r, fp.n_cb, fp.slice, mats);
    return hipGetLastError();
}

hipError_t launch_down_projection(const uint16_t *h, const uint16_t *A, float *tpart,
                                  int rows_here, int d, int r, const DownPlan &fp, const int *mat_of_row, hipStream_t st)
{
    if (rows_here <= 1) return launch_down<1>(h, A, tpart, rows_here, d, r, fp, mat_of_row, st);
    if (rows_here <= 2) return launch_down<2>(h, A, tpart, rows_here, d, r, fp, mat_of_row, st);
    if (rows_here <= 4) return launch_down<4>(h, A, tpart, rows_here, d, r, fp, mat_of_row, st);
    return launch_down<8>(h, A, tpart, rows_here, d, r, fp, mat_of_row, st);
}

static hipError_t launch_widen_rows(const uint16_t *h, float *x, int n, hipStream_t st)
{
    widen_rows_kernel<<<(n + 255) / 256, 256, 0, st>>>(h, x, n);
    return hipGetLastError();
}

// What a launch of stream_topk_kernel is given (the instances differ in types only).
template <typename WT>
struct StreamCall {
    const void *x; int nds;
    const WT *M;
    float2 *ms; float *pv; int *pi;
    int rows_here, row0, K, V;
    ChunkGeom g;
    int k;
    float4 *smp; uint32_t seed_lo, seed_hi;
    const uint16_t *A = nullptr;
};

constexpr int stream_x_bytes(int src) { return src == kGlobal ? 0 : src == kHalfRows ? 2 : 4; }     // of an element of x in shared memory

template <int R, int NW, typename WT, int SRC>
static hipError_t launch_stream(const StreamCall<WT> &c, hipStream_t st)
{
    const int per_xcd = (c.g.chunks + 7) / 8, k_parts = SRC == kGlobal ? 1 : c.g.k_parts;
    const size_t dyn = stream_lds_bytes(R, NW, c.g, c.K, stream_x_bytes(SRC));
    if (dyn > 32 * 1024) {
        static LdsLimit lds_limit;
        const hipError_t e = lds_limit.raise(reinterpret_cast<const void *>(stream_topk_kernel<R, NW, WT, SRC>), (int)dyn);
        if (e != hipSuccess) return e;
    }
    stream_topk_kernel<R, NW, WT, SRC><<<8 * per_xcd, NW * 64, dyn, st>>>(c.x, c.nds, c.A, c.M, c.ms, c.pv, c.pi, c.rows_here, c.row0, c.K, c.V, c.g.chunks,
                                                                          c.g.lanes, k_parts, stream_parts(NW, k_parts, c.K), c.k, c.smp, c.seed_lo, c.seed_hi);
    return hipGetLastError();
}

template <typename WT, int SRC>
static hipError_t launch_stream_rows(const StreamCall<WT> &c, hipStream_t st)
{
    // One row: the block size the chunk geometry asks for.  More rows: as many wavefronts as the shared memory of
    // the partial sums (NW * R * 2 KB) allows; they split the contraction, and every one of them keeps loads in flight.
    const auto fits = [&](int R, int NW) { return stream_lds_bytes(R, NW, c.g, c.K, stream_x_bytes(SRC)) <= kStreamLdsLimit; };
    if (c.rows_here <= 1) {
        if constexpr (SRC != kOwn)                      // (its rule leaves blocks of 1024 threads out: they lack the registers)
            if (c.g.nw1 == 16 && fits(1, 16)) return launch_stream<1, 16, WT, SRC>(c, st);
        if (c.g.nw1 >= 8 && fits(1, 8)) return launch_stream<1, 8, WT, SRC>(c, st);
        return launch_stream<1, 4, WT, SRC>(c, st);
    }
    if constexpr (SRC == kOwn) return hipErrorInvalidValue;      // (a single row's)
    else {
    if (c.rows_here <= 2)
        return fits(2, 16) ? launch_stream<2, 16, WT, SRC>(c, st) : fits(2, 8) ? launch_stream<2, 8, WT, SRC>(c, st) : launch_stream<2, 4, WT, SRC>(c, st);
    if (c.rows_here <= 4) return fits(4, 8) ? launch_stream<4, 8, WT, SRC>(c, st) : launch_stream<4, 4, WT, SRC>(c, st);
    return fits(8, 4) ? launch_stream<8, 4, WT, SRC>(c, st) : launch_stream<8, 2, WT, SRC>(c, st);
    }
}

template <typename WT>
static hipError_t launch_stream_src(StreamCall<WT> c, float *wide, hipStream_t st)
{
    if constexpr (sizeof(WT) == 2)                      // (the low-rank head's weights are bf16)
        if (c.nds > 0) return launch_stream_rows<WT, kSlices>(c, st);
    // the smallest block's need decides: rows too long for it are read from memory as fp32
    if (stream_rows_fit(c.rows_here, c.g, c.K)) return launch_stream_rows<WT, kHalfRows>(c, st);
    const hipError_t e = launch_widen_rows(static_cast<const uint16_t *>(c.x), wide, c.rows_here * c.K, st);
    if (e != hipSuccess) return e;
    c.x = wide;
    return launch_stream_rows<WT, kGlobal>(c, st);
}

hipError_t launch_stream_topk(const void *x, int nds, float *wide, const void *M, bool m_is_f32, float2 *ms, float *pv, int *pi,
                              int rows_here, int row0, int K, int V, const ChunkGeom &g, int k,
                              float4 *smp, uint32_t seed_lo, uint32_t seed_hi, hipStream_t st)
{
    if (m_is_f32)
        return launch_stream_src<float>({x, nds, static_cast<const float *>(M), ms, pv, pi, rows_here, row0, K, V, g, k, smp, seed_lo, seed_hi}, wide, st);
    return launch_stream_src<uint16_t>({x, nds, static_cast<const uint16_t *>(M), ms, pv, pi, rows_here, row0, K, V, g, k, smp, seed_lo, seed_hi}, wide, st);
}

hipError_t launch_stream_topk_own_input(const uint16_t *h, const uint16_t *A, int d, const uint16_t *M, float2 *ms, float *pv, int *pi,
                                        int K, int V, const ChunkGeom &g, int k, float4 *smp, uint32_t seed_lo, uint32_t seed_hi, hipStream_t st)
{
    return launch_stream_rows<uint16_t, kOwn>({h, d, M, ms, pv, pi, 1, 0, K, V, g, k, smp, seed_lo, seed_hi, A}, st);
}

}  // namespace slimspec
