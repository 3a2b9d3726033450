// Vocabulary projection with the fused log-sum-exp / top-k epilogue for calls of a few rows (paper section 4.1:
// logits = t B, or h W for the full head, never written to memory): the weight matrix streams from HBM once for up to
// 48 rows, and the products are as exact as fp32 fused multiply-adds.
//
// What bounds it: reading the weight matrix.  The lane-owns-columns kernel (gemv_kernels.hip) spends one fp32
// multiply-add per weight and row, so from two rows on its vector instructions, not the memory, decide (60 us at 4
// rows, 72 us for every 8 rows at d = 4096, r = 512, V = 128256).  Here the matrix cores multiply:
//   * bf16 weights times an fp32 t = hi + mid + lo, three bf16 pieces that hold its 24 significant bits exactly: every
//     product is exact and only the fp32 accumulation rounds, as in a chain of fp32 multiply-adds.  Three times the
//     matrix work is still far below the time the weights need (48 rows: 19 GFLOP beside 131 MB).
//   * A wavefront owns 128 columns and a slice of the contraction.  Its lanes load the weights as they lie in memory
//     (lane = 8 adjacent columns of one row, 256-byte segments, 8 rows each), straight into registers; a lane then
//     holds an 8 x 8 block, which 32 byte permutes turn into 8 operands of v_mfma_f32_16x16x32_bf16 (8 consecutive
//     contraction elements of one column).  Half a vector instruction per weight whatever the number of rows, and no
//     shared memory in the loop.
//   * The wavefronts of a block cover G x 128 adjacent columns in KS slices of the contraction, G chosen so that
//     every block is resident at once (at most 256 chunks): no last, nearly empty round.
// The partials have the layout of the streaming kernel's, and the same merge kernel finishes the call.
//
// The epilogue is a chain of a few hundred instructions per row that nothing overlaps.  With lists of up to 32 ids a wavefront
// takes two rows at a time (the sort, the reductions and the ranking serve both), and what a lane holds of a row is known
// when compiled (GM): without it every step branched.
//
// Measured at d = 4096, r = 512, V = 128256 (kernel alone; 131 MB of weights are 22-26 us at a plain read's rate; one row per
// wavefront and step, in brackets): 23 rows, k = 10 27.8 us (33.0), 40 rows, k = 32 37.6 (42.9), 4 rows, k = 64 29.7 (31.3); 27 rows with
// draws, r = 456, V = 31664 17.5 (22.4).  Calls: 40 rows with k = 32 51.2 to 52.6 us by the machine, 23 rows 41.0 to 41.4.  Error of the
// log-probabilities against 64-bit arithmetic: 7.7e-8 relative, 1.0e-7 with one multiply-add per weight (40 rows, k = 32).
#include "gemv_parts.hpp"
#include "launch.hpp"
#include <type_traits>

namespace slimspec {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));


// Two 16-bit elements (low or high halves of a and b) as one operand dword: a's element first.
template <bool HIGH>
__device__ __forceinline__ uint32_t pair16(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_perm(b, a, HIGH ? 0x07060302u : 0x05040100u);
}

// Sum over each half of 32 lanes, in every lane of it.
__device__ __forceinline__ float half_sum(float v) {
    v += dpp_f32<0xB1>(v);
    v += dpp_f32<0x4E>(v);
    v += dpp_f32<0x141>(v);
    v += dpp_f32<0x140>(v);
    uint32_t a, b;
    swap_pair<16>(__float_as_uint(v), a, b);
    return __uint_as_float(a) + __uint_as_float(b);
}
__device__ __forceinline__ uint64_t half_max_key(uint64_t k) {
    const auto step = [&](uint32_t hi, uint32_t lo) { k = u64_max(k, u64_from(hi, lo)); };
    step(dpp_u32<0xB1>((uint32_t)(k >> 32)), dpp_u32<0xB1>((uint32_t)k));
    step(dpp_u32<0x4E>((uint32_t)(k >> 32)), dpp_u32<0x4E>((uint32_t)k));
    step(dpp_u32<0x141>((uint32_t)(k >> 32)), dpp_u32<0x141>((uint32_t)k));
    step(dpp_u32<0x140>((uint32_t)(k >> 32)), dpp_u32<0x140>((uint32_t)k));
    uint32_t ha, hb, la, lb;
    swap_pair<16>((uint32_t)(k >> 32), ha, hb);
    swap_pair<16>((uint32_t)k, la, lb);
    return u64_max(u64_from(ha, la), u64_from(hb, lb));
}
// bits = 2 bits + (z >= t)
__device__ __forceinline__ void shift_in_ge(uint32_t &bits, float z, float t) {
    asm("v_cmp_ge_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(bits) : "v"(z), "v"(t) : "vcc");
}
__device__ __forceinline__ float max3_number(float a, float b, float c) { float d; asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c)); return d; }

}  // namespace

// X: [NP][8 ceil(K / 64)][16 NT] 16-byte vectors of 8 consecutive contraction elements of one row: the bf16 input
//    itself (NP = 1: full head) or the pieces of t (NP = 3); zero beyond K and beyond the last row.  by_rows (NP = 1): the bf16 input as it
//    lies in memory, [rows, K], whose loads touch twice as many lines, against a launch that regroups it (plan.hpp: rows_read_by_rows).
// M: [K, V] bf16 row-major, V and K multiples of 8
// Block b: columns [128 G b, 128 G (b + 1)); wavefront w: column group w % G, contraction slice w / G (none from KS on).
// Partials of (row, chunk): see stream_topk_kernel.  row0: the index in the call of this launch's first row (noise).
// GM: G at most (what a lane keeps of a row's logits is sized by it: known when compiled, or every step of the epilogue branches)
// SUM (NT 1, NP 3): X is not given; the block adds the nds slices of t, fp32 [nds][rows][K], itself and keeps the pieces in shared memory,
// where a small t takes less time than a launch that does it once (plan.hpp: rows_sum_slices).
// meet_at: where in shared memory, in floats, the slices of the contraction leave their sums; 0: no place for them.
template <int NT, int NP, int GM, bool SUM>
__global__ __launch_bounds__(512) void rows_topk_kernel(
    const uint4 *__restrict__ X, const float *__restrict__ slices, int nds, const uint16_t *__restrict__ M,
    float2 *__restrict__ part_ms, float *__restrict__ part_val, int *__restrict__ part_id, float4 *__restrict__ part_smp,
    int rows, int row0, int K, int V, int chunks, int G, int KS, int k, uint32_t seed_lo, uint32_t seed_hi, int meet_at, int by_rows)
{
    extern __shared__ __align__(16) float z_lds[];               // [16 NT][row_stride]
    constexpr int RP = 16 * NT;
    const int row_stride = rows_lds_stride(G);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cg = wave % G, ks = wave / G;
    const int c16 = lane & 15, kg = lane >> 4;
    const int n_steps = (K + 31) / 32, per = (n_steps + KS - 1) / KS;
    const int s_beg = min(n_steps, ks * per), s_end = min(n_steps, s_beg + per);
    const int chunk_col = blockIdx.x * (128 * G);
    const int x_groups = (K + 63) / 64 * 8;
    const size_t x_piece = (size_t)x_groups * RP;
    uint4 *const x_lds = reinterpret_cast<uint4 *>(reinterpret_cast<unsigned char *>(z_lds) + rows_x_offset(NT, G, (int)(blockDim.x >> 6), k));      // (SUM)

    f32x4 acc[8][NT];                                            // [column in the lane's 8][row tile]
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[j][nt][i] = 0.f;

    {
        // columns beyond V re-read the last group that exists (their logits are masked below)
        const uint16_t *const m_lane = M + min(chunk_col + cg * 128 + 8 * c16, V - 8);
        const uint4 *const x_lane = (SUM ? x_lds : X) + (size_t)kg * RP + c16;
        u32x4 q[2][8], xv[NP][NT];
        // (NP 1) where the lane's row of each tile begins, in elements, and what lies between 8 elements of a row and the next, and between steps
        uint32_t x_row[NT];
        const uint32_t x_kg = by_rows ? 8u : 8u * RP, x_step = 4u * x_kg;
        if constexpr (NP == 1) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) x_row[nt] = by_rows ? (uint32_t)min(16 * nt + c16, rows - 1) * (uint32_t)K : 8u * (uint32_t)(16 * nt + c16);
        }
        const auto load_m = [&](u32x4 (&dst)[8], int s) {
            // K is a multiple of 8: a lane's 8 rows exist or none do (then rows of the step that do are read, and dropped)
            const int k0 = 32 * s + ((32 * s + 8 * kg < K) ? 8 * kg : 0);
            const uint16_t *p = m_lane + (size_t)k0 * V;
#pragma unroll
            for (int u = 0; u < 8; ++u) dst[u] = *reinterpret_cast<const u32x4 *>(p + (size_t)u * V);
        };
        const auto load_x = [&](int s) {
            if constexpr (NP == 1) {
                const uint32_t at = (uint32_t)s * x_step + ((32 * s + 8 * kg < K) ? (uint32_t)kg * x_kg : 0u);
                const uint16_t *h = reinterpret_cast<const uint16_t *>(X) + at;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) xv[0][nt] = *reinterpret_cast<const u32x4 *>(h + x_row[nt]);
            } else {
#pragma unroll
                for (int p = 0; p < NP; ++p)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        xv[p][nt] = *reinterpret_cast<const u32x4 *>(x_lane + p * x_piece + (size_t)(4 * s) * RP + 16 * nt);
            }
        };
        if constexpr (SUM) {
            static_assert(NT == 1 && NP == 3, "a few rows of t");
            constexpr int SB = kRowsMaxSlices;
            const int n_items = rows * (K / 8), per_row = K / 8, nthreads = (int)blockDim.x;
            float4 v[SB][2];
            const auto load_slices = [&](int e) {                // item e: 8 adjacent columns of a row
                const int row = e / per_row, g8 = e - row * per_row;
                const float4 *src = reinterpret_cast<const float4 *>(slices + (size_t)row * K + 8 * g8);
#pragma unroll
                for (int u = 0; u < SB; ++u) {
                    if (u >= nds) break;
                    v[u][0] = src[(size_t)u * rows * (K / 4)];
                    v[u][1] = src[(size_t)u * rows * (K / 4) + 1];
                }
            };
            const auto store_pieces = [&](int e) {
                const int row = e / per_row, g8 = e - row * per_row;
                float t[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int u = 0; u < SB; ++u) {                   // fixed order
                    if (u >= nds) break;
                    t[0] += v[u][0].x; t[1] += v[u][0].y; t[2] += v[u][0].z; t[3] += v[u][0].w;
                    t[4] += v[u][1].x; t[5] += v[u][1].y; t[6] += v[u][1].z; t[7] += v[u][1].w;
                }
                uint4 piece[3];
                cut_pieces(t, piece);
#pragma unroll
                for (int p = 0; p < 3; ++p) x_lds[p * x_piece + (size_t)g8 * RP + row] = piece[p];
            };
            for (int e = tid; e < x_groups * RP; e += nthreads)  // rows beyond the last, elements beyond K
                if ((e & (RP - 1)) >= rows || (e / RP) * 8 >= K) {
#pragma unroll
                    for (int p = 0; p < 3; ++p) x_lds[p * x_piece + e] = make_uint4(0u, 0u, 0u, 0u);
                }
            int e = tid;
            for (; e + nthreads < n_items; e += nthreads) { load_slices(e); store_pieces(e); }
            if (e < n_items) load_slices(e);
            __builtin_amdgcn_sched_barrier(0);
            if (s_beg < s_end) load_m(q[0], s_beg);              // the first weights right behind
            if (s_beg + 1 < s_end) load_m(q[1], s_beg + 1);
            __builtin_amdgcn_sched_barrier(0);
            if (e < n_items) store_pieces(e);
            __syncthreads();
        }
        const auto multiply = [&](u32x4 (&w)[8], int s) {
            if (32 * s + 32 > K) {                               // the last step of a K that is no multiple of 32
                const uint32_t keep = (32 * s + 8 * kg < K) ? 0xffffffffu : 0u;
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[u][e] &= keep;
                if constexpr (NP == 1) {                         // (an infinity there must not meet the cleared weights)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int e = 0; e < 4; ++e) xv[0][nt][e] &= keep;
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                u32x4 a0, a1;                                    // columns 2 e and 2 e + 1 of the lane's 8
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    a0[t] = pair16<false>(w[2 * t][e], w[2 * t + 1][e]);
                    a1[t] = pair16<true>(w[2 * t][e], w[2 * t + 1][e]);
                }
                // The step's products are summed on their own, the smallest pieces first, and then added: the matrix
                // unit's internal roundings then happen at the size of one step's sum, not of the whole.
                f32x4 t0[NT], t1[NT];
                const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int p = NP - 1; p >= 0; --p)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        t0[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a0), __builtin_bit_cast(bf16x8, xv[p][nt]), p == NP - 1 ? zero : t0[nt], 0, 0, 0);
                        t1[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a1), __builtin_bit_cast(bf16x8, xv[p][nt]), p == NP - 1 ? zero : t1[nt], 0, 0, 0);
                    }
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) { acc[2 * e][nt] += t0[nt]; acc[2 * e + 1][nt] += t1[nt]; }
                if (NT == 3) __builtin_amdgcn_sched_barrier(0);   // keeps the next pair's operands out of the registers (256 per lane)
            }
        };
        // Two steps of weights in flight.  Loads return in order, so a step's row operand is requested before the
        // weights of the step after it: waiting for it leaves those in flight.  No step is requested that does not exist: its
        // registers could not be used again before it had arrived, at the end of the block, when nothing hides the trip (0.7 us
        // at 2 to 23 rows).  But with three row tiles the copies of the step that this takes do not fit the registers.
        const auto then = []() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
        if (NT == 3 && s_beg < s_end) {
            load_m(q[0], s_beg); load_x(s_beg); then();
            load_m(q[1], min(s_beg + 1, s_end - 1)); then();
            for (int s = s_beg; s < s_end; s += 2) {
                multiply(q[0], s); then();
                if (s + 1 < s_end) {
                    load_x(s + 1); then();
                    load_m(q[0], min(s + 2, s_end - 1)); then();         // (past the end: the last step once more, unused)
                    multiply(q[1], s + 1); then();
                    load_x(min(s + 2, s_end - 1)); then();
                    load_m(q[1], min(s + 3, s_end - 1)); then();
                }
            }
        } else if (s_beg + 1 == s_end) {
            if (!SUM) load_m(q[0], s_beg);
            load_x(s_beg); then();
            multiply(q[0], s_beg);
        } else if (s_beg < s_end) {
            if (!SUM) load_m(q[0], s_beg);
            load_x(s_beg); then();
            if (!SUM) load_m(q[1], s_beg + 1);
            then();
            int s = s_beg;
            for (; s + 3 < s_end; s += 2) {
                multiply(q[0], s); then();
                load_x(s + 1); then();
                load_m(q[0], s + 2); then();
                multiply(q[1], s + 1); then();
                load_x(s + 2); then();
                load_m(q[1], s + 3); then();
            }
            multiply(q[0], s); then();                           // two or three steps are left
            load_x(s + 1); then();
            if (s + 2 < s_end) {
                load_m(q[0], s + 2); then();
                multiply(q[1], s + 1); then();
                load_x(s + 2); then();
                multiply(q[0], s + 2);
            } else
                multiply(q[1], s + 1);
        }
    }

    // The slices of the contraction meet in shared memory, the last slice first (a fixed order).  Element (m = 4 kg + i, n = c16) of tile j
    // is column 8 m + j of row 16 nt + n.  One slice after the other, each reading what the one before it left, is a chain of KS trips
    // and barriers behind the last weights, most wavefronts idle.  So few rows are added at once, by all threads, where a slice has a place
    // of its own (plan.hpp: rows_meet_at_once), and two slices finish half of the elements each.  One after the other / now, us a call: full
    // head, 4 rows, d = 1024, V = 32000 21.3 / 19.7, 7 rows, d = 4096, V = 20000 43.0 / 42.1; d = 4096, r = 512: 8 rows, V = 32768 23.3 / 22.4,
    // 16 rows 23.4 / 22.6; two slices, V = 66000 to 128256, 120 calls: 33 rows 0.993 of the time, 48 rows 0.991, up to 32 rows level (0.97 to 1.02), with draws the same.
    const auto place = [&](int nt, int i) { return z_lds + (16 * nt + c16) * row_stride + cg * 128 + 8 * (4 * kg + i); };
    const auto put_sums = [&](float *at, int stride) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            if (16 * nt + c16 < rows) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float4 *dst = reinterpret_cast<float4 *>(at + (16 * nt + c16) * stride + cg * 128 + 8 * (4 * kg + i));
                    dst[0] = make_float4(acc[0][nt][i], acc[1][nt][i], acc[2][nt][i], acc[3][nt][i]);
                    dst[1] = make_float4(acc[4][nt][i], acc[5][nt][i], acc[6][nt][i], acc[7][nt][i]);
                }
            }
    };
    if (NT == 1 && meet_at > 0) {                                // (no more than 16 rows)
        const int stride = rows_meet_stride(G), region = rows * stride;
        float *const others = z_lds + meet_at;                   // [KS - 1][rows][stride]; slice 0's are where the logits go
        if (ks < KS) put_sums(ks == 0 ? z_lds : others + (ks - 1) * region, ks == 0 ? row_stride : stride);
        __syncthreads();
        const int items = rows * G, per_row = (65536 + G - 1) / G;       // a half-wavefront takes 128 columns of a row
        for (int e = tid >> 5; e < items; e += (int)(blockDim.x >> 5)) {
            const int row = e * per_row >> 16, col = 128 * (e - row * G) + 4 * (lane & 31);
            const float *src = others + row * stride + col;
            float4 *dst = reinterpret_cast<float4 *>(z_lds + row * row_stride + col);
            float4 p[kRowsMaxKS];
#pragma unroll
            for (int u = 0; u < kRowsMaxKS; ++u) {
                if (u >= KS) break;
                p[u] = u == 0 ? dst[0] : *reinterpret_cast<const float4 *>(src + (u - 1) * region);
            }
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int u = kRowsMaxKS - 1; u >= 0; --u) {
                if (u >= KS) continue;
                if (u == KS - 1) a = p[u];
                else { a.x += p[u].x; a.y += p[u].y; a.z += p[u].z; a.w += p[u].w; }
            }
            dst[0] = a;
        }
        __syncthreads();
    } else if (KS == 2) {
        // either slice finishes half of the elements: the other's half of its own waits where the logits go
        const auto half_of = [&](auto first) {
            constexpr int F = decltype(first)::value;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int i = 2 - F; i < 4 - F; ++i) {
                    float4 *dst = reinterpret_cast<float4 *>(place(nt, i));
                    dst[0] = make_float4(acc[0][nt][i], acc[1][nt][i], acc[2][nt][i], acc[3][nt][i]);
                    dst[1] = make_float4(acc[4][nt][i], acc[5][nt][i], acc[6][nt][i], acc[7][nt][i]);
                }
            __syncthreads();
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int i = F; i < F + 2; ++i) {
                    float4 *dst = reinterpret_cast<float4 *>(place(nt, i));
                    const float4 c = dst[0], d = dst[1];
                    dst[0] = make_float4(acc[0][nt][i] + c.x, acc[1][nt][i] + c.y, acc[2][nt][i] + c.z, acc[3][nt][i] + c.w);
                    dst[1] = make_float4(acc[4][nt][i] + d.x, acc[5][nt][i] + d.y, acc[6][nt][i] + d.z, acc[7][nt][i] + d.w);
                }
        };
        if (ks == 0) half_of(std::integral_constant<int, 0>{});
        else if (ks == 1) half_of(std::integral_constant<int, 2>{});
        else __syncthreads();
        __syncthreads();
    } else {
        for (int kk = KS - 1; kk >= 0; --kk) {
            if (ks == kk) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float4 *dst = reinterpret_cast<float4 *>(place(nt, i));
                        float4 a = make_float4(acc[0][nt][i], acc[1][nt][i], acc[2][nt][i], acc[3][nt][i]);
                        float4 b = make_float4(acc[4][nt][i], acc[5][nt][i], acc[6][nt][i], acc[7][nt][i]);
                        if (kk != KS - 1) {
                            const float4 c = dst[0], d = dst[1];
                            a.x += c.x; a.y += c.y; a.z += c.z; a.w += c.w;
                            b.x += d.x; b.y += d.y; b.z += d.z; b.w += d.w;
                        }
                        dst[0] = a; dst[1] = b;
                    }
            }
            __syncthreads();
        }
    }

    // One row by a whole wavefront: running max, sum of exp and top-k of the chunk.  Lane = columns 2 lane, 2 lane + 1 of every
    // group of 128.
    constexpr int E = 2 * GM;
    const auto finish_row = [&](int row) __attribute__((always_inline)) {
        // (what does not depend on the row would be computed ahead of the loop over the rows, by the calls too that never come
        // here: 0.6 us at the end of every block)
        int lane = tid & 63;
        asm volatile("" : "+v"(lane));
        const auto act = [&](int g) { return (g < GM / 2 + 1 || g < G) && chunk_col + 128 * g + 2 * lane < V; };      // V is even: both columns or none
        const auto id = [&](int e) { return (uint32_t)(chunk_col + 128 * (e >> 1) + 2 * lane + (e & 1)); };
        float *zr = z_lds + row * row_stride;
        const size_t slot = (size_t)row * chunks + blockIdx.x;
        float z[E], m = kNegInf, s = 0.f;
#pragma unroll
        for (int g = 0; g < GM; ++g) {
            float2 v = make_float2(kNegInf, kNegInf);
            if (act(g)) v = *reinterpret_cast<const float2 *>(zr + 128 * g + 2 * lane);
            z[2 * g] = v.x; z[2 * g + 1] = v.y;
        }
        const auto max_and_sum = [&]() {
            m = z[0];
#pragma unroll
            for (int e = 1; e < E; ++e) m = fmaxf(m, z[e]);
            m = wave_max(m);
            s = 0.f;
#pragma unroll
            for (int g = 0; g < GM; ++g)
                s += fast_exp(z[2 * g] - m) + fast_exp(z[2 * g + 1] - m);     // exp(-inf) = 0 beyond V
            s = wave_sum(s);
        };
        max_and_sum();
        if (NP > 1 && !(s < __builtin_huge_valf())) {
            // A logit that is no finite number.  The pieces of t cannot stand for one product with an infinite weight
            // (0 times infinity): sum the chunk's logits of this row again, one multiply-add per weight, from t itself.
            // Eight weights in flight: a row of nothing but such logits comes here in every chunk (one not-a-number row of 4 at
            // d = 4096, r = 512, V = 128256: 611 us a call with one weight in flight, 242 with eight; 38 without such a row).
            // What this needs is made opaque, or the compiler computes the eight strides ahead for every row and spills scalar
            // registers for them: 0.4 us at 16 to 32 rows and 1 us at 48 for calls without such logits.
            const uint16_t *Mq = M;
            const uint4 *Xq = X;
            int Vq = V, Kq = K, rowq = row;
            asm volatile("" : "+s"(Mq), "+s"(Xq), "+s"(Vq), "+s"(Kq), "+s"(rowq));
            if constexpr (SUM) Xq = x_lds;
#pragma unroll 1
            for (int g = 0; g < G; ++g) {
                if (!act(g)) continue;
                const uint16_t *mp = Mq + chunk_col + 128 * g + 2 * lane;
                float z0 = 0.f, z1 = 0.f;
#pragma unroll 1
                for (int j = 0; j < Kq; j += 8) {                // K is a multiple of 8
                    uint32_t w[8];
                    u32x4 xp[NP];
#pragma unroll
                    for (int u = 0; u < 8; ++u) w[u] = *reinterpret_cast<const uint32_t *>(mp + (size_t)(j + u) * Vq);
#pragma unroll
                    for (int p = 0; p < NP; ++p) xp[p] = *reinterpret_cast<const u32x4 *>(Xq + p * ((size_t)((Kq + 63) / 64 * 8) * RP) + (size_t)(j >> 3) * RP + rowq);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        float t = 0.f;                           // the pieces' sum, exact: they do not overlap
#pragma unroll
                        for (int p = 0; p < NP; ++p) {
                            const uint32_t two = xp[p][u >> 1];
                            t += (u & 1) ? bf16_hi(two) : bf16_lo(two);
                        }
                        z0 = fmaf(t, bf16_lo(w[u]), z0);
                        z1 = fmaf(t, bf16_hi(w[u]), z1);
                    }
                }
#pragma unroll
                for (int gg = 0; gg < GM; ++gg)
                    if (gg == g) { z[2 * gg] = z0; z[2 * gg + 1] = z1; }
            }
            max_and_sum();
        }
        if (part_smp) {
            // keys are unique (one per id), so exactly one lane holds the wavefront's largest
            const GumbelKey gk = gumbel_key(seed_lo, seed_hi, (uint32_t)(row0 + row));
            uint64_t best = kNoKey;
            float zb = 0.f;
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (act(e >> 1)) {
                    const uint64_t key = make_key(z[e] + gumbel_base2(gk, id(e)) * kLn2, id(e));
                    if (key > best) { best = key; zb = z[e]; }
                }
            const uint64_t top = wave_max_key(best);
            if (best == top && best != kNoKey)
                part_smp[slot] = make_float4(key_value(top), __int_as_float((int)key_tiebreak(top)), zb, 0.f);
        }
        if (lane == 0) part_ms[slot] = make_float2(m, s);
        uint32_t ob[E];
#pragma unroll
        for (int e = 0; e < E; ++e) ob[e] = act(e >> 1) ? list_bits(z[e]) : 0u;
        // the candidates' keys go where the row's logits were
        lds_wave_sync();
        wave_topk<E>(ob, 2 * G, id, lane, k, reinterpret_cast<uint64_t *>(zr), row_stride / 2, part_val + slot * k, part_id + slot * k);
    };

    const int n_waves = (int)(blockDim.x >> 6);
    // Lists of up to kPairMaxK ids: two rows at a time, one per half-wavefront.  This is bound by its own instruction count, and
    // everything that is done once per row (the sort, the reductions, the ranking) then serves two.  Lane = columns
    // 4 l ... 4 l + 3 of every group of 128.  Rows that hold something else than finite numbers, more candidates than
    // the buffer or fewer than k lanes with columns go through finish_row.
    const int half = lane >> 5, l32 = lane & 31;
    const auto act4 = [&](int g) { return (g < GM / 2 + 1 || g < G) && chunk_col + 128 * g + 4 * l32 < V; };      // all four columns or none
    uint32_t *const cand_bits = reinterpret_cast<uint32_t *>(z_lds + RP * row_stride) + (wave * 2 + half) * (2 * kPairKeys), *const cand_id = cand_bits + kPairCand;
    const auto finish_pair = [&](int row0p) __attribute__((always_inline)) {                    // false: these rows are finish_row's
        const int row = row0p + half;                            // (an odd last row is done twice, and written once)
        const bool exists = row < rows;
        const float *zr = z_lds + min(row, rows - 1) * row_stride + 4 * l32;
        const size_t slot = (size_t)min(row, rows - 1) * chunks + blockIdx.x;
        float z[4 * GM], sub[2] = {kNegInf, kNegInf};
#pragma unroll
        for (int g = 0; g < GM; ++g)
            {
                float4 v = make_float4(kNegInf, kNegInf, kNegInf, kNegInf);
                if (act4(g)) v = *reinterpret_cast<const float4 *>(zr + 128 * g);      // all four columns or none
                z[4 * g] = v.x; z[4 * g + 1] = v.y; z[4 * g + 2] = v.z; z[4 * g + 3] = v.w;
                sub[0] = max3_number(sub[0], v.x, v.y);
                sub[1] = max3_number(sub[1], v.z, v.w);
            }
        // T: the k-th largest of the row's 32 lane maxima, or of the 64 maxima of half lanes (k > 16): k elements reach it
        uint32_t sorted;
        if (k <= 16) sorted = half_sort_desc(float_order_bits(fmaxf(sub[0], sub[1])), lane);
        else {
            const uint32_t a = half_sort_desc(float_order_bits(sub[0]), lane), b = half_sort_desc(float_order_bits(sub[1]), lane);
            const uint32_t rev = lane_xor16(dpp_u32<0x140>(b), lane);
            sorted = half_merge_desc(a > rev ? a : rev, lane);   // the 32 largest of both
        }
        const auto of_half = [&](int at) {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)sorted, at), hi = (uint32_t)__builtin_amdgcn_readlane((int)sorted, 32 + at);
            return float_from_order_bits(half ? hi : lo);
        };
        const float m = of_half(0), T = of_half(k - 1);
        float s = 0.f;
#pragma unroll
        for (int g = 0; g < GM; ++g)
            s += (fast_exp(z[4 * g] - m) + fast_exp(z[4 * g + 1] - m)) + (fast_exp(z[4 * g + 2] - m) + fast_exp(z[4 * g + 3] - m));      // exp(-inf) = 0 beyond V
        s = half_sum(s);
        uint32_t bits = 0u;                                      // the elements that reach T, the first one in the highest place
#pragma unroll
        for (int e = 0; e < 4 * GM; ++e) shift_in_ge(bits, z[e], T);
        const uint32_t mine = (uint32_t)__popc(bits), upto = half_prefix_sum(mine);
        const int n0 = __builtin_amdgcn_readlane((int)upto, 31), n1 = __builtin_amdgcn_readlane((int)upto, 63), n_max = max(n0, n1);
        if (n_max > kPairCand || __ballot(!(s < __builtin_huge_valf()) || T == kNegInf) != 0ull) return false;
        const auto id_at = [&](int e) { return (uint32_t)(chunk_col + 128 * (e >> 2) + 4 * l32 + (e & 3)); };
        if (part_smp) {
            const GumbelKey gk = gumbel_key(seed_lo, seed_hi, (uint32_t)(row0 + row));
            uint64_t best = kNoKey;
            float zb = 0.f;
#pragma unroll
            for (int e = 0; e < 4 * GM; ++e)
                if (act4(e >> 2)) {
                    const uint64_t key = make_key(z[e] + gumbel_base2(gk, id_at(e)) * kLn2, id_at(e));
                    if (key > best) { best = key; zb = z[e]; }
                }
            const uint64_t top = half_max_key(best);             // keys are unique: one lane of the half holds it
            if (exists && best == top && best != kNoKey)
                part_smp[slot] = make_float4(key_value(top), __int_as_float((int)key_tiebreak(top)), zb, 0.f);
        }
        if (exists && l32 == 0) part_ms[slot] = make_float2(m, s);
        // The candidates, compacted, in the row's part of the buffer: first their order bits, then their ids.
        uint32_t at = upto - mine;
        const int n = half ? n1 : n0;
        if (l32 >= n) cand_bits[l32] = 0u;                       // what follows the last is cleared for the ranking
        if (32 + l32 >= n) cand_bits[32 + l32] = 0u;
        while (__ballot(bits != 0u) != 0ull) {
            if (bits != 0u) {
                const int top_bit = 31 - __clz((int)bits), e = 4 * GM - 1 - top_bit;
                cand_bits[at] = float_order_bits(zr[128 * (e >> 2) + (e & 3)]);
                cand_id[at++] = id_at(e);
                bits ^= 1u << top_bit;
            }
        }
        lds_wave_sync();
        // Ranked by their logits alone; equal ones (the same rank twice) are told apart by their ids afterwards.
        const uint32_t b0 = cand_bits[l32], b1 = cand_bits[32 + l32], i0 = cand_id[l32], i1 = cand_id[32 + l32];
        int r0 = 0, r1 = 0;
        const uint4 *four = reinterpret_cast<const uint4 *>(cand_bits);
        if (n_max <= 32) {
#pragma unroll 2
            for (int q = 0; q < n_max; q += 4) {
                const uint4 c = four[q >> 2];
                r0 += (c.x > b0 ? 1 : 0) + (c.y > b0 ? 1 : 0) + (c.z > b0 ? 1 : 0) + (c.w > b0 ? 1 : 0);
            }
        } else {
#pragma unroll 2
            for (int q = 0; q < n_max; q += 4) {
                const uint4 c = four[q >> 2];
                r0 += (c.x > b0 ? 1 : 0) + (c.y > b0 ? 1 : 0) + (c.z > b0 ? 1 : 0) + (c.w > b0 ? 1 : 0);
                r1 += (c.x > b1 ? 1 : 0) + (c.y > b1 ? 1 : 0) + (c.z > b1 ? 1 : 0) + (c.w > b1 ? 1 : 0);
            }
        }
        lds_wave_sync();
        const bool have0 = l32 < n, have1 = 32 + l32 < n;
        if (have0) cand_bits[r0] = (uint32_t)l32;
        if (have1) cand_bits[r1] = (uint32_t)(32 + l32);
        lds_wave_sync();
        if (__ballot((have0 && cand_bits[r0] != (uint32_t)l32) || (have1 && cand_bits[r1] != (uint32_t)(32 + l32))) != 0ull) {
            lds_wave_sync();
            if (have0) cand_bits[l32] = b0;
            if (have1) cand_bits[32 + l32] = b1;
            lds_wave_sync();
            for (int q = 0; q < n_max; ++q) {                    // (beyond a row's n: cleared bits, or a stale rank below any finite logit's)
                const uint32_t c = q < n ? cand_bits[q] : 0u, ci = cand_id[q];
                r0 += c == b0 && ci < i0 ? 1 : 0;
                r1 += c == b1 && ci < i1 ? 1 : 0;
            }
        }
        const auto put = [&](uint32_t bits_of, uint32_t id_of, int rank) {
            part_val[slot * k + rank] = float_from_order_bits(bits_of);
            part_id[slot * k + rank] = (int)id_of;
        };
        if (exists && have0 && r0 < k) put(b0, i0, r0);
        if (n_max > 32 && exists && have1 && r1 < k) put(b1, i1, r1);
        lds_wave_sync();                                         // the buffer is this wavefront's next rows'
        return true;
    };
    // (Up to a row per wavefront and long lists, one row each: 7 rows, k = 27 7.1 us against 7.4.)
    const int at_once = k <= 16 || (k <= kPairMaxK && rows > n_waves) ? 2 : 1;
    for (int row = at_once * wave; row < rows; row += at_once * n_waves) {
        const int n_left = (at_once == 2 && finish_pair(row)) ? 0 : min(at_once, rows - row);
#pragma unroll 1
        for (int q = 0; q < n_left; ++q) finish_row(row + q);
    }
}

template <int NT, int NP, int GM, bool SUM>
static hipError_t launch_rows(const RowsInput &x, const uint16_t *M, float2 *ms, float *pv, int *pi, float4 *smp, int rows, int row0,
                              int K, int V, const RowsGeom &g, int k, uint32_t seed_lo, uint32_t seed_hi, hipStream_t st)
{
    const RowsLds lds = rows_lds(rows, K, g, k, SUM);
    static LdsLimit lds_limit;
    hipError_t e = lds_limit.raise(reinterpret_cast<const void *>(rows_topk_kernel<NT, NP, GM, SUM>), (int)lds.bytes);
    if (e != hipSuccess) return e;
    rows_topk_kernel<NT, NP, GM, SUM><<<g.chunks, 64 * g.waves, lds.bytes, st>>>(static_cast<const uint4 *>(x.X), x.slices, x.nds, M, ms, pv, pi, smp,
                                                                           rows, row0, K, V, g.chunks, g.G, g.KS, k, seed_lo, seed_hi, lds.meet_at, x.by_rows ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_rows_topk(const RowsInput &x, const uint16_t *M, float2 *ms, float *pv, int *pi, float4 *smp,
                            int rows, int row0, int K, int V, const RowsGeom &g, int k, uint32_t seed_lo, uint32_t seed_hi, hipStream_t st)
{
    static_assert(kRowsMaxColGroups == 6, "the instances cover G = 1, 2, up to 4 and up to 6");
#define SLIMSPEC_ROWS_G(NT, NP, GM, SUM) launch_rows<NT, NP, GM, SUM>(x, M, ms, pv, pi, smp, rows, row0, K, V, g, k, seed_lo, seed_hi, st)
#define SLIMSPEC_ROWS(NT, NP, SUM) (g.G == 1 ? SLIMSPEC_ROWS_G(NT, NP, 1, SUM) : g.G == 2 ? SLIMSPEC_ROWS_G(NT, NP, 2, SUM) \
                                             : g.G <= 4 ? SLIMSPEC_ROWS_G(NT, NP, 4, SUM) : SLIMSPEC_ROWS_G(NT, NP, 6, SUM))
    // The kernels lie in memory in this order of first use.  With those that add slices first, the ones for three pieces took longer with the same
    // instructions (7 rows, d = 6392, r = 1040, V = 11896 27.9 / 27.5 us a call, 16 rows, d = 4096, r = 1024, V = 32000 30.0 / 29.4, 4 rows of the router
    // 52.4 / 52.1), and what this order costs is less (5 rows, r = 256, V = 74504 22.6 / 22.7, 23 rows 42.3 / 42.6); with them last 22.6 / 23.1 there.
    if (x.pieces == 3 && !x.slices) return rows <= 16 ? SLIMSPEC_ROWS(1, 3, false) : rows <= 32 ? SLIMSPEC_ROWS(2, 3, false) : SLIMSPEC_ROWS(3, 3, false);
    if (x.slices) return SLIMSPEC_ROWS(1, 3, true);
    return rows <= 16 ? SLIMSPEC_ROWS(1, 1, false) : rows <= 32 ? SLIMSPEC_ROWS(2, 1, false) : SLIMSPEC_ROWS(3, 1, false);
#undef SLIMSPEC_ROWS
#undef SLIMSPEC_ROWS_G
}

}  // namespace slimspec
