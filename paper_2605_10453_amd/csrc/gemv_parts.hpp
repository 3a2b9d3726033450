// Device-side pieces shared by the streaming ("lane owns columns") kernels: raw weight loads and
// the per-chunk epilogue (running max, sum of exp, top-k of one chunk of 64 to 512 columns).
#pragma once
#include "device_utils.hpp"
#include "plan.hpp"
#include <type_traits>

namespace slimspec {

// 8 adjacent columns of one matrix row: kept as loaded (raw) while in flight, widened
// to fp32 only when consumed, so that many loads can be outstanding per lane.
struct Raw8Bf16 { uint4 w; };
struct Raw8F32 { float4 a, b; };
__device__ __forceinline__ Raw8Bf16 load_raw8(const uint16_t *p) { return {*reinterpret_cast<const uint4 *>(p)}; }
__device__ __forceinline__ Raw8F32 load_raw8(const float *p) {
    return {*reinterpret_cast<const float4 *>(p), *reinterpret_cast<const float4 *>(p + 4)};
}
__device__ __forceinline__ void widen8(const Raw8Bf16 &q, float (&f)[8]) {
    f[0] = bf16_lo(q.w.x); f[1] = bf16_hi(q.w.x); f[2] = bf16_lo(q.w.y); f[3] = bf16_hi(q.w.y);
    f[4] = bf16_lo(q.w.z); f[5] = bf16_hi(q.w.z); f[6] = bf16_lo(q.w.w); f[7] = bf16_hi(q.w.w);
}
__device__ __forceinline__ void widen8(const Raw8F32 &q, float (&f)[8]) {
    f[0] = q.a.x; f[1] = q.a.y; f[2] = q.a.z; f[3] = q.a.w; f[4] = q.b.x; f[5] = q.b.y; f[6] = q.b.z; f[7] = q.b.w;
}

// ---------------------------------------------------------------------------
// Down-projection t = h A shared out in items of (64 columns of A) x (a slice of d).
constexpr int kItemCols = 64;           // columns of A per item: one 128-byte line per row of A

// Which matrix of a stack of down-projection matrices each of up to 8 rows uses (one matrix per drafted position).
struct RowMats { int m[8]; };

// One down-projection item: columns [64 cb, 64 cb + 64) x rows [ds * slice, ds * slice + slice) of A.
// Thread = (row slot tid / 8, 16-byte piece tid % 8).  tpart is [nds][R][r].
// POS: A is a stack of [d, r] matrices and row i uses matrix mats.m[i] (every row then loads its own weights).
template <int R, int NT, bool POS>
__device__ __forceinline__ void down_item(float (*redd)[R][kItemCols], const uint16_t *__restrict__ h,
                                          const uint16_t *__restrict__ A, float *__restrict__ tpart,
                                          int item, int n_cb, int slice, int rows_here, int d, int r, int tid,
                                          const RowMats &mats)
{
    constexpr int NW = NT / 64;
    const int cb = item % n_cb, ds = item / n_cb;
    const int piece = tid & 7, slot = tid >> 3;
    const int col = cb * kItemCols + piece * 8;
    const int c_beg = ds * slice, c_end = min(d, c_beg + slice);
    float acc[R][8];
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[i][e] = 0.f;
    if (col < r) {
        for (int c = c_beg + slot; c < c_end; c += NT / 8) {
            if constexpr (!POS) {
                const uint4 w = *reinterpret_cast<const uint4 *>(A + (size_t)c * r + col);
                const float f[8] = {bf16_lo(w.x), bf16_hi(w.x), bf16_lo(w.y), bf16_hi(w.y),
                                    bf16_lo(w.z), bf16_hi(w.z), bf16_lo(w.w), bf16_hi(w.w)};
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const float hv = (i < rows_here) ? bf16_to_float(h[(size_t)i * d + c]) : 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[i][e] = fmaf(hv, f[e], acc[i][e]);
                }
            } else {
                uint4 w[R];
#pragma unroll
                for (int i = 0; i < R; ++i)
                    w[i] = *reinterpret_cast<const uint4 *>(A + (size_t)mats.m[i & 7] * d * r + (size_t)c * r + col);
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const float f[8] = {bf16_lo(w[i].x), bf16_hi(w[i].x), bf16_lo(w[i].y), bf16_hi(w[i].y),
                                        bf16_lo(w[i].z), bf16_hi(w[i].z), bf16_lo(w[i].w), bf16_hi(w[i].w)};
                    const float hv = (i < rows_here) ? bf16_to_float(h[(size_t)i * d + c]) : 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[i][e] = fmaf(hv, f[e], acc[i][e]);
                }
            }
        }
    }
    // lanes with equal (lane % 8) hold the same columns: butterfly over lane bits 3, 4, 5
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float v = acc[i][e];
            v += dpp_f32<0x128>(v);                             // row_ror:8  = lane ^ 8 inside a row of 16
            uint32_t a, b;
            swap_pair<16>(__float_as_uint(v), a, b);
            v = __uint_as_float(a) + __uint_as_float(b);
            swap_pair<32>(__float_as_uint(v), a, b);
            v = __uint_as_float(a) + __uint_as_float(b);
            if (lane < 8) redd[wave][i][lane * 8 + e] = v;
        }
    __syncthreads();
    for (int q = tid; q < R * kItemCols; q += NT) {
        const int i = q / kItemCols, c = q % kItemCols;
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += redd[w][i][c];        // fixed order
        if (cb * kItemCols + c < r) tpart[((size_t)ds * R + i) * r + cb * kItemCols + c] = s;
    }
    __syncthreads();
}


// ---------------------------------------------------------------------------
// The k largest of a row's logits that one wavefront holds (up to E per lane, as order bits: 0 where the lane holds no
// column), ranked by (logit desc, id asc) into out_val / out_id.  This is the tail of every block, after its last
// weight row has arrived, and its instruction count is what a call of dozens of rows waits for.  All 64 lanes call.
//   (1) T: the k-th largest of the 64 lane maxima, from a sort across the lanes.  An element below T is preceded by k
//       lane maxima, so it cannot be among the k first.  (Bit by bit with ballots instead, T cost more than the rest.)
//   (2) Where k is close to 64, T admits hundreds of elements and ranking them would take longer than everything else
//       (k = 64: 53 us per launch against 27): T is raised by bisection until at most kCandSlack beyond k are left.
//   (3) The elements >= T are compacted into `cand` (cap keys) through ballots and lane prefix counts and ranked by
//       counting.  More than cap elements at the bound means that many equal logits: the largest key is then taken k
//       times.
// n_e: elements per lane in use (at most E, the same in all lanes); id(e): the id of this lane's element e.
constexpr int kCandSlack = 24;
template <int E, class Id>
__device__ __forceinline__ void wave_topk(const uint32_t (&ob)[E], int n_e, Id id, int lane, int k, uint64_t *cand, int cap,
                                          float *__restrict__ out_val, int *__restrict__ out_id)
{
    uint32_t lane_bits = ob[0];
#pragma unroll
    for (int e = 1; e < E; ++e) lane_bits = max(lane_bits, ob[e]);
    const uint32_t sorted = wave_sort_desc(lane_bits, lane);
    uint32_t T = max(1u, (uint32_t)__builtin_amdgcn_readlane((int)sorted, k - 1));       // fewer than k lanes in use: everything
    const auto compact = [&]() {
        int n = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (e >= n_e) break;
            const bool take = ob[e] >= T;
            const uint64_t mask = __ballot(take);
            const int at = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (take && at < cap) cand[at] = u64_from(ob[e], ~id(e));
            n += __popcll(mask);
        }
        return n;
    };
    int n = compact();
    if (n > 64 && n > k + kCandSlack) {
        uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)sorted) + 1u;      // no element's bits reach it
        while (n > k + kCandSlack && hi - T > 1u) {
            const uint32_t mid = T + (hi - T) / 2;
            int c = 0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if (e >= n_e) break;
                c += __popcll(__ballot(ob[e] >= mid));
            }
            if (c >= k) { T = mid; n = c; } else hi = mid;
        }
        lds_wave_sync();
        n = compact();
    }
    lds_wave_sync();
    if (n <= cap) {
        for (int c0 = 0; c0 < n; c0 += 64) {
            const int c = c0 + lane;
            const uint64_t mine = (c < n) ? cand[c] : kNoKey;
            int rk = 0;
#pragma unroll 8
            for (int q = 0; q < n; ++q) rk += (cand[q] > mine) ? 1 : 0;
            if (c < n && rk < k) {
                out_val[rk] = key_value(mine);
                out_id[rk] = (int)key_tiebreak(mine);
            }
        }
    } else {
        uint64_t last = ~0ull;
        for (int rk = 0; rk < k; ++rk) {
            uint64_t best = kNoKey;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const uint64_t key = u64_from(ob[e], ~id(e));
                if (ob[e] != 0u && key < last) best = u64_max(best, key);
            }
            last = wave_max_key(best);
            if (lane == 0) { out_val[rk] = key_value(last); out_id[rk] = (int)key_tiebreak(last); }
        }
    }
    if (lane >= n && lane < k) {                                 // fewer than k columns in this chunk
        out_val[lane] = kNegInf;
        out_id[lane] = kNoId;
    }
    lds_wave_sync();                                             // the buffers are reused by this wavefront's next row
}

// One row of a chunk of cw columns (at most 512) from chunk_col on: fixed-order sum of its n partial sums (sums[p * stride + c] for
// column c), then (max, sum of exp, top-k) of the logits, written as the partial of (row, chunk).  One wavefront; all 64
// lanes must call.  sel: cw keys of shared memory.
//
// Top-k: wave_topk.  Lane = columns 2 lane, 2 lane + 1 of every 128; E: elements per lane, 2 for every 128 columns begun (known when
// compiled, or every step branches).
// TOPK, DRAW: which of the two parts this call makes (a sampling call gives them to two wavefronts where the block has one to spare).
// part_smp (may be null): the chunk's best z_v + g_v with standard Gumbel noise g (Gumbel-max sampling), as
// (z + g, id, z, -) of the winner; gk: the noise key of this row.
template <int E, bool TOPK, bool DRAW>
__device__ __forceinline__ void chunk_row_epilogue(const float *sums, int n, int stride, int cw, int chunk_col, int V, int lane, int k,
                                                   uint64_t *sel, size_t slot,
                                                   float2 *__restrict__ part_ms, float *__restrict__ part_val,
                                                   int *__restrict__ part_id,
                                                   float4 *__restrict__ part_smp, const GumbelKey &gk)
{
    const auto act = [&](int e) { const int c = 128 * (e >> 1) + 2 * lane; return c < cw && chunk_col + c < V; };      // V and cw are even: both columns or none
    const auto id = [&](int e) { return (uint32_t)(chunk_col + 128 * (e >> 1) + 2 * lane + (e & 1)); };
    float z[E];
#pragma unroll
    for (int e = 0; e < E; e += 2) {
        float2 s = make_float2(kNegInf, kNegInf);
        if (act(e)) {
            const float *src = sums + 64 * e + 2 * lane;
            s = make_float2(0.f, 0.f);
            int p = 0;                          // fixed order: the first rows of the contraction first
            for (; p + 8 <= n; p += 8) {
                float2 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float2 *>(src + (p + u) * stride);
#pragma unroll
                for (int u = 0; u < 8; ++u) { s.x += v[u].x; s.y += v[u].y; }
            }
            for (; p < n; ++p) {
                const float2 v = *reinterpret_cast<const float2 *>(src + p * stride);
                s.x += v.x; s.y += v.y;
            }
        }
        z[e] = s.x; z[e + 1] = s.y;
    }

    if (DRAW && part_smp) {
        // keys are unique (one per id), so exactly one lane holds the wavefront's largest
        uint64_t best = kNoKey;
        float zb = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (act(e)) {
                const uint64_t key = make_key(z[e] + gumbel_base2(gk, id(e)) * kLn2, id(e));
                if (key > best) { best = key; zb = z[e]; }
            }
        const uint64_t top = wave_max_key(best);
        if (best != kNoKey && best == top)
            part_smp[slot] = make_float4(key_value(top), __int_as_float((int)key_tiebreak(top)), zb, 0.f);
    }
    if constexpr (!TOPK) return;
    float lm = z[0];
#pragma unroll
    for (int e = 1; e < E; ++e) lm = fmaxf(lm, z[e]);
    const float m = wave_max(lm);
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < E; e += 2)
        s += fast_exp(z[e] - m) + fast_exp(z[e + 1] - m);     // exp(-inf) = 0 for padding lanes
    s = wave_sum(s);

    if (lane == 0) part_ms[slot] = make_float2(m, s);
    uint32_t ob[E];
#pragma unroll
    for (int e = 0; e < E; ++e) ob[e] = act(e) ? list_bits(z[e]) : 0u;
    wave_topk<E>(ob, E, id, lane, k, sel, cw, part_val + slot * k, part_id + slot * k);
}

// The same for the only row of a block in a wide chunk, by all its wavefronts, for lists of up to 16 ids (plan.hpp: block_row_takes): what one wavefront does
// as a chain of dependent instructions, which nothing overlaps, takes two barriers here.  A lane of the first four wavefronts, one per SIMD, has two adjacent
// columns: with more wavefronts they would wait for each other's instructions.  sums [n][cw], n at most kDirectParts: a wavefront is one lane group there.
// All threads call, behind a barrier; S.groups are zeros beyond the plan's.
//   (1) the partial sums of the columns;
//   (2) T: the smallest of the maxima of k groups of columns (device_utils.hpp), hence k elements reach it;
//   (3) the elements that reach T are ranked by counting, eight by a wavefront at a time.
// By time stamps the tail of d = 4096, r = 512, V = 128256 takes 1.5 us (one wavefront: 2.5), the call 32.0 (32.7).  With every wavefront of the block in
// it the tail took 1.9, and 2 us more where the last chunk has few columns and all of them reached the bound.  (Every instance for a single row has room for S
// in shared memory, 5 KB, also where its chunks are narrow: a CU then has one block.)
constexpr int kBlockRowWaves = 4, kBlockRowMine = 128;      // wavefronts with columns; keys of one's list at most
struct BlockRowLds {
    uint64_t mine[kBlockRowWaves][kBlockRowMine + 8], wave_draw[kBlockRowWaves];
    uint32_t groups[128];                                        // (lanes without a class read beyond the 32)
    int n_mine[kBlockRowWaves];
    float wave_s[kBlockRowWaves], wave_draw_z[kBlockRowWaves], m;
};
struct BlockRowPlan { int lanes; BoundPlan bound; };
__device__ __forceinline__ BlockRowPlan make_block_row_plan(int cw, int chunk_col, int V, int k) {
    BlockRowPlan p;
    p.lanes = min(cw, V - chunk_col) / 2;                        // cw and V are even
    p.bound = make_bound_plan(p.lanes, k, 4);
    return p;
}
static_assert(!block_row_takes(kChunkCols, kBoundMaxK + 1), "lists that bound_of_groups serves");
static_assert(!block_row_takes(8 * 32, 1) && kDirectParts >= 16, "more than half of a wavefront's lanes per chunk, hence one partial sum per wavefront");
template <int NW>
__device__ __forceinline__ void block_row_epilogue(BlockRowLds &S, const BlockRowPlan &plan, const float *sums, int n, int cw, int chunk_col, int tid, int k,
                                                   size_t slot, float2 *__restrict__ part_ms, float *__restrict__ part_val,
                                                   int *__restrict__ part_id, float4 *__restrict__ part_smp, const GumbelKey &gk)
{
    static_assert(NW >= kBlockRowWaves, "the wavefronts with columns");
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const auto add = [&](const float2 *src, int n_src, int stride) {      // fixed order, the first rows of the contraction first
        float2 s = make_float2(0.f, 0.f);
        const auto batch = [&](auto n_tag) {
            constexpr int N = decltype(n_tag)::value;
            float2 v[N];
#pragma unroll
            for (int u = 0; u < N; ++u) v[u] = src[u * stride];
#pragma unroll
            for (int u = 0; u < N; ++u) { s.x += v[u].x; s.y += v[u].y; }
            src += N * stride;
        };
        int p = n_src;
        for (; p >= 16; p -= 16) batch(std::integral_constant<int, 16>{});
        if (p & 8) batch(std::integral_constant<int, 8>{});
        if (p & 4) batch(std::integral_constant<int, 4>{});
        if (p & 2) batch(std::integral_constant<int, 2>{});
        if (p & 1) batch(std::integral_constant<int, 1>{});
        return s;
    };
    const int n2 = cw / 2;
    const bool with_columns = wave * 64 < plan.lanes;            // (at most 256 lanes: the first four wavefronts)
    const bool act = tid < plan.lanes;
    const uint32_t id0 = (uint32_t)(chunk_col + 2 * tid);
    float2 z = make_float2(kNegInf, kNegInf);
    uint32_t b0 = 0u, b1 = 0u;
    const int gl = plan.bound.gl;
    if (with_columns) {
        if (act) {
            z = add(reinterpret_cast<const float2 *>(sums) + tid, n, n2);
            b0 = list_bits(z.x); b1 = list_bits(z.y);
        }
        uint32_t most = max(b0, b1);
        if (gl > 0) most = max(most, dpp_u32<0xB1>(most));
        if (gl > 1) most = max(most, dpp_u32<0x4E>(most));
        if (gl > 2) most = max(most, dpp_u32<0x141>(most));
        if (gl > 3) most = max(most, dpp_u32<0x140>(most));
        if (act && (tid & ((1 << gl) - 1)) == 0) S.groups[tid >> gl] = most;
    }
    __syncthreads();
    int n_mine = 0;
    if (with_columns) {
        uint32_t top;
        const uint32_t T = bound_of_groups(S.groups, plan.bound, k, lane, top);
        const float M = float_from_order_bits(top);              // (where it is no number, the sum of exponentials is none either)
        // (two ballots are fewer instructions here than a prefix sum over the lanes)
        const auto push = [&](bool take, uint32_t bits, uint32_t id) {
            const uint64_t mask = __ballot(take);
            const int at = n_mine + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (take) S.mine[wave][at] = u64_from(bits, ~id);
            n_mine += __popcll(mask);
        };
        push(b0 >= T, b0, id0);
        push(b1 >= T, b1, id0 + 1u);
        const float s = wave_sum(act ? fast_exp(z.x - M) + fast_exp(z.y - M) : 0.f);
        S.wave_s[wave] = s;
        S.m = M;                                                 // (the same in every wavefront)
        if (part_smp) {                                          // the largest z + g
            uint64_t best = kNoKey;
            float zb = z.x;
            if (act) {
                best = make_key(z.x + gumbel_base2(gk, id0) * kLn2, id0);
                const uint64_t k1 = make_key(z.y + gumbel_base2(gk, id0 + 1u) * kLn2, id0 + 1u);
                if (k1 > best) { best = k1; zb = z.y; }
            }
            const uint64_t largest = wave_max_key(best);         // unique keys: one lane holds it
            if (best == largest) { S.wave_draw[wave] = largest; S.wave_draw_z[wave] = zb; }
        }
    }
    if (wave < kBlockRowWaves) {
        if (lane < 8) S.mine[wave][n_mine + lane] = kNoKey;
        S.n_mine[wave] = n_mine;
    }
    __syncthreads();
    constexpr int RW = NW < 8 ? NW : 8;                          // wavefronts that go on: more would only wait for each other's instructions
    if (wave >= RW) return;
    const int n_waves = (plan.lanes + 63) >> 6;
    if (tid == RW * 64 - 1) {
        float s = S.wave_s[0];
        for (int w = 1; w < n_waves; ++w) s += S.wave_s[w];      // fixed order
        part_ms[slot] = make_float2(S.m, s);
        if (part_smp) {
            int best = 0;
            for (int w = 1; w < n_waves; ++w)
                if (S.wave_draw[w] > S.wave_draw[best]) best = w;
            part_smp[slot] = make_float4(key_value(S.wave_draw[best]), __int_as_float((int)key_tiebreak(S.wave_draw[best])), S.wave_draw_z[best], 0.f);
        }
    }
    // A wavefront ranks eight of all the lists' elements at a time.
    int n_w[kBlockRowWaves], n_all = 0, longest = 0;
#pragma unroll
    for (int w = 0; w < kBlockRowWaves; ++w) {
        n_w[w] = __builtin_amdgcn_readfirstlane(S.n_mine[w]);
        n_all += n_w[w];
        longest = max(longest, n_w[w]);
    }
    for (int c0 = 8 * wave; c0 < n_all; c0 += 8 * RW) {
        const int c = c0 + (lane >> 3);
        int at = c, before = 0;                                  // its place in the lists
#pragma unroll
        for (int w = 0; w + 1 < kBlockRowWaves; ++w) {
            before += n_w[w];
            at = c >= before ? c - before + (w + 1) * (kBlockRowMine + 8) : at;
        }
        const uint64_t key = c < n_all ? S.mine[0][at] : kNoKey;
        const int rank = rank_in_lists(S.mine, n_w, longest, key, lane);
        if (c < n_all && (lane & 7) == 0 && rank < k) {
            part_val[slot * k + rank] = key_value(key);
            part_id[slot * k + rank] = (int)key_tiebreak(key);
        }
    }
    if (tid >= n_all && tid < k) {                               // fewer than k columns in this chunk
        part_val[slot * k + tid] = kNegInf;
        part_id[slot * k + tid] = kNoId;
    }
}

}  // namespace slimspec
