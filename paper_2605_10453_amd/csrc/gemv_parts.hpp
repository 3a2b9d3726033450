// Device-side pieces shared by the streaming ("lane owns columns") kernels: raw weight loads and
// the per-chunk epilogue (running max, sum of exp, top-k of one chunk of 64 to 512 columns).
#pragma once
#include "device_utils.hpp"
#include "plan.hpp"

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

}  // namespace slimspec
