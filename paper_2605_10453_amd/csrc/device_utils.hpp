// Small device helpers shared by the gfx950 kernels: bf16 unpacking, the
// (logit desc, id asc) order as a 64-bit key, and wavefront-wide (64-lane)
// reductions built on DPP lane permutes (no LDS traffic, no bpermute latency).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "plan.hpp"

namespace slimspec {

constexpr int kWave = 64;
constexpr float kNegInf = -__builtin_huge_valf();
constexpr int kNoId = 0x7fffffff;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Two bf16 values packed in one 32-bit word (low half = even element).
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float bf16_to_float(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// exp(x) and ln(x) through the hardware base-2 units.
__device__ __forceinline__ float fast_exp(float x) { return __builtin_amdgcn_exp2f(x * kLog2e); }
__device__ __forceinline__ float fast_log(float x) { return __builtin_amdgcn_logf(x) * kLn2; }

// The 16-bit row operand of the matrix-core head kernel: t log2(e) rounded to bf16 (nearest even) or to f16.  One
// definition for the kernel that writes the operand and for the merge, which recomputes from it the logit the head
// kernel saw for a column without a recorded value.
__device__ __forceinline__ uint32_t operand_bf16_bits(float t) {
    const uint32_t u = __float_as_uint(t * kLog2e);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ _Float16 operand_f16(float t) { return (_Float16)(t * kLog2e); }
// ... as two bf16 pieces: the rounded value and what is left of it, rounded (the difference is exact)
__device__ __forceinline__ uint32_t operand_rest_bf16_bits(float t) {
    const uint32_t u = __float_as_uint(t * kLog2e - __uint_as_float(operand_bf16_bits(t) << 16));
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
// ... and the value of t it stands for (how: plan.hpp, kOperandBf16 ...)
__device__ __forceinline__ float operand_value(float t, int how) {
    if (how == kOperandF16) return (float)operand_f16(t) * kLn2;
    const float hi = __uint_as_float(operand_bf16_bits(t) << 16);
    return (how == kOperandTwoBf16 ? hi + __uint_as_float(operand_rest_bf16_bits(t) << 16) : hi) * kLn2;
}

// Eight floats as three bf16 pieces each, cut off the top of the significand, 8 bits each: their sum is the float exactly.
// Infinity and not-a-number stay whole in the first piece (the low bits of a not-a-number may be all it has).
__device__ __forceinline__ void cut_pieces(const float (&v)[8], uint4 (&piece)[3]) {
    uint32_t b[3][8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const uint32_t u = __float_as_uint(v[c]);
        const bool number = (u & 0x7f800000u) != 0x7f800000u;
        const uint32_t top = u & 0xffff0000u;
        const float rest = v[c] - __uint_as_float(top);
        const uint32_t mid = __float_as_uint(rest) & 0xffff0000u;
        const uint32_t low = __float_as_uint(rest - __uint_as_float(mid));
        b[0][c] = number ? top : top | ((u & 0x007fffffu) ? 0x00400000u : 0u);
        b[1][c] = number ? mid : 0u;
        b[2][c] = number ? low : 0u;
    }
#pragma unroll
    for (int p = 0; p < 3; ++p)
        piece[p] = make_uint4((b[p][0] >> 16) | (b[p][1] & 0xffff0000u), (b[p][2] >> 16) | (b[p][3] & 0xffff0000u),
                              (b[p][4] >> 16) | (b[p][5] & 0xffff0000u), (b[p][6] >> 16) | (b[p][7] & 0xffff0000u));
}

// Order of the outputs: larger logit first, equal logits: smaller id first.
__device__ __forceinline__ bool ranks_before(float va, int ia, float vb, int ib) {
    return (va > vb) || (va == vb && ia < ib);
}

// ---------------------------------------------------------------------------
// 64-bit sort key: high word = logit mapped to an unsigned integer with the same
// order (-0 is first turned into +0 so that equal logits give equal words), low
// word = ~tiebreak, so that a larger key ranks first and, among equal logits,
// the smaller tiebreak (vocabulary id or list position) ranks first.
__device__ __forceinline__ uint32_t float_order_bits(float v) {
    uint32_t u = __float_as_uint(v + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
// ... of a logit that may enter a list, where 0 means no entry: the not-a-number with all bits set, whose order bits that are, takes 1.
__device__ __forceinline__ uint32_t list_bits(float v) { return max(1u, float_order_bits(v)); }
__device__ __forceinline__ float float_from_order_bits(uint32_t o) {
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}
__device__ __forceinline__ uint64_t make_key(float v, uint32_t tiebreak) {
    return ((uint64_t)float_order_bits(v) << 32) | (uint32_t)~tiebreak;
}
__device__ __forceinline__ float key_value(uint64_t k) { return float_from_order_bits((uint32_t)(k >> 32)); }
__device__ __forceinline__ uint32_t key_tiebreak(uint64_t k) { return ~(uint32_t)k; }
constexpr uint64_t kNoKey = 0;      // ranks after every real key (a real key has a non-zero high word)

// ---------------------------------------------------------------------------
// Lane permutes.  DPP controls: quad_perm [1,0,3,2] = 0xB1 (lane ^ 1), quad_perm
// [2,3,0,1] = 0x4E (lane ^ 2), row_half_mirror = 0x141 (7 - lane within 8),
// row_mirror = 0x140 (15 - lane within 16).  After the first two steps all lanes
// of a quad agree, after the mirrors all lanes of a row of 16 agree; the two
// gfx950 permlane swaps then exchange rows of 16 and halves of 32.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) { return __uint_as_float(dpp_u32<CTRL>(__float_as_uint(x))); }

// value held by the lane 16 (STEP == 16) or 32 (STEP == 32) positions away, xor-wise
template <int STEP>
__device__ __forceinline__ void swap_pair(uint32_t x, uint32_t &a, uint32_t &b) {
    if constexpr (STEP == 16) {
        auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        a = r[0]; b = r[1];
    } else {
        auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        a = r[0]; b = r[1];
    }
}

#define SLIMSPEC_WAVE_REDUCE_F32(NAME, OP)                                            \
    __device__ __forceinline__ float NAME(float v) {                                  \
        v = OP(v, dpp_f32<0xB1>(v));                                                  \
        v = OP(v, dpp_f32<0x4E>(v));                                                  \
        v = OP(v, dpp_f32<0x141>(v));                                                 \
        v = OP(v, dpp_f32<0x140>(v));                                                 \
        uint32_t a, b;                                                                \
        swap_pair<16>(__float_as_uint(v), a, b);                                      \
        v = OP(__uint_as_float(a), __uint_as_float(b));                               \
        swap_pair<32>(__float_as_uint(v), a, b);                                      \
        v = OP(__uint_as_float(a), __uint_as_float(b));                               \
        return v;                                                                     \
    }
__device__ __forceinline__ float op_max(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ float op_add(float a, float b) { return a + b; }
// Every lane ends with the same bits: each step combines two values that all
// lanes of the group already share, and max / + are commutative bit for bit.
SLIMSPEC_WAVE_REDUCE_F32(wave_max, op_max)
SLIMSPEC_WAVE_REDUCE_F32(wave_sum, op_add)
#undef SLIMSPEC_WAVE_REDUCE_F32

__device__ __forceinline__ uint64_t u64_from(uint32_t hi, uint32_t lo) { return ((uint64_t)hi << 32) | lo; }
__device__ __forceinline__ uint64_t u64_max(uint64_t a, uint64_t b) { return a > b ? a : b; }

// Largest 64-bit key of the wavefront, in every lane.
__device__ __forceinline__ uint64_t wave_max_key(uint64_t k) {
    uint32_t hi = (uint32_t)(k >> 32), lo = (uint32_t)k;
#define SLIMSPEC_STEP(CTRL)                                                           \
    {                                                                                 \
        uint64_t o = u64_from(dpp_u32<CTRL>(hi), dpp_u32<CTRL>(lo));                  \
        k = u64_max(k, o); hi = (uint32_t)(k >> 32); lo = (uint32_t)k;                \
    }
    SLIMSPEC_STEP(0xB1) SLIMSPEC_STEP(0x4E) SLIMSPEC_STEP(0x141) SLIMSPEC_STEP(0x140)
#undef SLIMSPEC_STEP
    uint32_t ha, hb, la, lb;
    swap_pair<16>(hi, ha, hb); swap_pair<16>(lo, la, lb);
    k = u64_max(u64_from(ha, la), u64_from(hb, lb)); hi = (uint32_t)(k >> 32); lo = (uint32_t)k;
    swap_pair<32>(hi, ha, hb); swap_pair<32>(lo, la, lb);
    return u64_max(u64_from(ha, la), u64_from(hb, lb));
}

// Sum of v over every aligned group of P adjacent lanes (P a power of two, at most 64; the same in all lanes of the
// group).  All lanes of the wavefront must be active at the call.
__device__ __forceinline__ int lanes_sum(int v, int P) {
    if (P > 1) v += (int)dpp_u32<0xB1>((uint32_t)v);
    if (P > 2) v += (int)dpp_u32<0x4E>((uint32_t)v);
    if (P > 4) v += (int)dpp_u32<0x141>((uint32_t)v);
    if (P > 8) v += (int)dpp_u32<0x140>((uint32_t)v);
    uint32_t a, b;
    if (P > 16) { swap_pair<16>((uint32_t)v, a, b); v = (int)(a + b); }
    if (P > 32) { swap_pair<32>((uint32_t)v, a, b); v = (int)(a + b); }
    return v;
}
// Lanes that share the scan for one of n items when nthreads threads work on them: the largest power of two P with
// n P <= nthreads (1 when there are more items than threads); returns log2 P.
__device__ __forceinline__ int lanes_per_item_log2(int n, int nthreads) {
    int p = 0;
    while (p < 6 && (2 * n << p) <= nthreads) ++p;
    return p;
}
// Bitonic sorts across lanes, descending.  An exchange pairs lane i with i ^ 1, 2, 8, 16 directly, with the mirror image in its
// block of 4, 8, 16, 32 or 64, and with i ^ 4 as mirror in 8 after mirror in 4: two DPP min / max and a select each.
__device__ __forceinline__ void sort_keep(uint32_t &v, uint32_t p, int lane, int upper_bit) {
    const uint32_t hi = v > p ? v : p, lo = v > p ? p : v;       // the lane below the partner keeps the larger value
    v = (lane & upper_bit) ? lo : hi;
}
// the value of the lane 16 away (XOR), of x
__device__ __forceinline__ uint32_t lane_xor16(uint32_t x, int lane) {
    uint32_t a, b;
    swap_pair<16>(x, a, b);
    return (lane & 16) ? a : b;
}
#define SLIMSPEC_X1 sort_keep(v, dpp_u32<0xB1>(v), lane, 1);
#define SLIMSPEC_X2 sort_keep(v, dpp_u32<0x4E>(v), lane, 2);
#define SLIMSPEC_X4 sort_keep(v, dpp_u32<0x141>(dpp_u32<0x1B>(v)), lane, 4);
#define SLIMSPEC_X8 sort_keep(v, dpp_u32<0x128>(v), lane, 8);
// each half of 32 lanes by itself (lane i of a half: the i-th largest): 15 exchanges
__device__ __forceinline__ uint32_t half_sort_desc(uint32_t v, int lane) {
    SLIMSPEC_X1
    sort_keep(v, dpp_u32<0x1B>(v), lane, 2); SLIMSPEC_X1
    sort_keep(v, dpp_u32<0x141>(v), lane, 4); SLIMSPEC_X2 SLIMSPEC_X1
    sort_keep(v, dpp_u32<0x140>(v), lane, 8); SLIMSPEC_X4 SLIMSPEC_X2 SLIMSPEC_X1
    sort_keep(v, lane_xor16(dpp_u32<0x140>(v), lane), lane, 16);             // mirror in 32: the upper row of 16 meets the lower one reversed
    SLIMSPEC_X8 SLIMSPEC_X4 SLIMSPEC_X2 SLIMSPEC_X1
    return v;
}
// each half's 32 values, where they are a bitonic sequence
__device__ __forceinline__ uint32_t half_merge_desc(uint32_t v, int lane) {
    sort_keep(v, lane_xor16(v, lane), lane, 16);
    SLIMSPEC_X8 SLIMSPEC_X4 SLIMSPEC_X2 SLIMSPEC_X1
    return v;
}
// all 64 lanes (lane i: the i-th largest): 21 exchanges
__device__ __forceinline__ uint32_t wave_sort_desc(uint32_t v, int lane) {
    v = half_sort_desc(v, lane);
    uint32_t a, b;
    swap_pair<32>(lane_xor16(dpp_u32<0x140>(v), lane), a, b);                // mirror in 64
    sort_keep(v, (lane & 32) ? a : b, lane, 32);
    return half_merge_desc(v, lane);
}
#undef SLIMSPEC_X1
#undef SLIMSPEC_X2
#undef SLIMSPEC_X4
#undef SLIMSPEC_X8

// ---------------------------------------------------------------------------
// Standard Gumbel noise as a pure function of (seed, row, vocabulary id), for one draw per row from softmax(z) by
// the Gumbel-max rule argmax_v (z_v + g_v) (sampling at temperature 1, section 5.3):
//     x = id * 0x9E3779B1 + row * 0x85EBCA77 + seed_lo;  x = mix(x);  x += seed_hi * 0xC2B2AE3D;  x = mix(x)
//     mix(x): x ^= x >> 16; x *= 0x21F0AAAD; x ^= x >> 15; x *= 0x735A2D97; x ^= x >> 15
//     n = x >> 9,  u = (2 n + 1) / 2^24,  E = -ln(1 - u) ~ Exp(1),  g = -ln E
// The draws that decide a sample are the large ones, i.e. small E = small u: there E comes from the series of
// -ln(1 - u) (the hardware logarithm of a number next to 1 would lose them); elsewhere 1 - u is exact in fp32.
constexpr uint32_t kGumbelIdStep = 0x9E3779B1u, kGumbelRowStep = 0x85EBCA77u;
struct GumbelKey { uint32_t row_term, hi_term; };      // row * 0x85EBCA77 + seed_lo,  seed_hi * 0xC2B2AE3D
__device__ __forceinline__ GumbelKey gumbel_key(uint32_t seed_lo, uint32_t seed_hi, uint32_t row) {
    return {row * kGumbelRowStep + seed_lo, seed_hi * 0xC2B2AE3Du};
}
__device__ __forceinline__ uint32_t mix32(uint32_t x) {
    x ^= x >> 16; x *= 0x21F0AAADu; x ^= x >> 15; x *= 0x735A2D97u; x ^= x >> 15;
    return x;
}
__device__ __forceinline__ uint32_t gumbel_bits(uint32_t id_row_term, uint32_t hi_term) { return mix32(mix32(id_row_term) + hi_term); }
// g / ln 2 (the noise in base-2 units: add it to a logit times log2 e)
__device__ __forceinline__ float gumbel_base2(const GumbelKey &key, uint32_t id) {
    const uint32_t x = gumbel_bits(id * kGumbelIdStep + key.row_term, key.hi_term);
    const uint32_t m = 2u * (x >> 9) + 1u;                          // u = m / 2^24, m odd, < 2^24
    const float u = (float)m * 5.9604644775390625e-8f;              // exact
    const float series = u * (1.f + u * (0.5f + u * (0.33333334f + u * (0.25f + u * 0.2f))));
    const float direct = -__builtin_amdgcn_logf((float)(16777216u - m) * 5.9604644775390625e-8f) * kLn2;   // 1 - u is exact
    const float E = (m < (1u << 18)) ? series : direct;
    return -__builtin_amdgcn_logf(E);
}
// An upper bound of it for four instructions behind the hash instead of twenty: kGumbelBoundBase - kGumbelBoundScale * gumbel_bound_bits().
// With n' = x >> 9 << 9 as a float, n' / 2^32 < u < E, and a float's bits are its base-2 logarithm with the mantissa as a straight
// line, which lies below it.  For u < 1/32, i.e. noise that can decide a draw, the bound is at most 0.103 + log2(1 + 1 / (2 n)) too large:
// 0.69 for n = 1, 0.2 for n = 6.  n = 0 (one id in 2^23) has no such logarithm: its bound is 159, 135 too large, and the id's group
// takes the first place of its list whatever its logit is (the merge has the noise itself; the list is a place shorter).
constexpr float kGumbelBoundBase = 159.f;               // 32 for the scale of x, 127 for the exponent's bias
constexpr float kGumbelBoundScale = 1.1920928955078125e-7f;      // 2^-23
__device__ __forceinline__ float gumbel_bound_bits(uint32_t x) { return (float)(int)__float_as_uint((float)(x & 0xfffffe00u)); }

// What follows serves tails that are chains of instructions.  Cycles per step of such a chain, one wavefront on a CU: a vector instruction 8, one with a DPP operand
// 12, a permlane swap with its move and maximum 28, a comparison and a branch on its ballot 64, an LDS read 69, an LDS write and a read behind barriers 133
// (four wavefronts) to 158 (eight), an LDS addition by one lane whose result all wait for 174.
//
// A bound that at least k elements reach, k <= 16: `lanes` adjacent lanes hold elements, and the largest order bits of each group of 2^gl of them (at most
// 2^most, no more than 32 groups) are known.  Class i of k is made of the groups i, i + k, ... (`deep` of them, at most 8); the smallest maximum of the classes
// is the bound.  (d = 4096, V = 128256, k = 10: 28 entries of the lists reach it; a sort would leave 12.)
constexpr int kBoundMaxK = 16, kBoundGroups = 32;
struct BoundPlan { int gl, n_groups, deep; bool all; };
__device__ __forceinline__ BoundPlan make_bound_plan(int lanes, int k, int most) {
    BoundPlan p;
    // the largest gl that leaves 2 k groups: ceil(lanes / 2^gl) >= 2 k
    p.gl = __clz(2 * k - 1) - __clz(max(1, lanes - 1));
    if (p.gl > 0 && ((2 * k - 1) << p.gl) > lanes - 1) --p.gl;
    p.gl = min(max(p.gl, 0), most);
    p.gl = max(p.gl, lanes <= kBoundGroups ? 0 : 27 - __clz(lanes - 1));      // no more than 32 groups, and 17 at least
    p.n_groups = (lanes + (1 << p.gl) - 1) >> p.gl;
    p.deep = 1;
    while (p.deep < 8 && (p.deep + 1) * k <= p.n_groups) ++p.deep;
    p.all = p.n_groups < k;                                      // too few for a bound: every element reaches 1
    asm volatile("" : "+s"(p.gl), "+s"(p.n_groups), "+s"(p.deep));      // (worked out here, ahead of the elements, which wait for memory)
    return p;
}
// ... lane's class (beyond the last: all bits)
__device__ __forceinline__ uint32_t class_max(const uint32_t *groups, const BoundPlan &p, int k, int i) {
    uint32_t t = i < k ? groups[i] : ~0u;
#pragma unroll
    for (int j = 1; j < 8; ++j) {
        if (j >= p.deep) break;                                  // (the same for all, and known before)
        t = max(t, groups[i + j * k]);                           // (lanes without a class: nothing beyond all bits)
    }
    return t;
}
// The bound; groups[kBoundGroups] with zeros beyond the last, and room for 128; top: the largest order bits of all.  The same in all lanes.
__device__ __forceinline__ uint32_t bound_of_groups(const uint32_t *groups, const BoundPlan &p, int k, int lane, uint32_t &top) {
    const int i = lane & 15;
    top = max(groups[i], groups[16 + i]);
    uint32_t t = class_max(groups, p, k, i);
    const auto both = [&](uint32_t a, uint32_t b) { t = min(t, a); top = max(top, b); };
    both(dpp_u32<0xB1>(t), dpp_u32<0xB1>(top));
    both(dpp_u32<0x4E>(t), dpp_u32<0x4E>(top));
    both(dpp_u32<0x141>(t), dpp_u32<0x141>(top));
    both(dpp_u32<0x140>(t), dpp_u32<0x140>(top));
    return p.all ? 1u : max(1u, t);
}
// Sum of v over the lanes of this half up to and including this one.
__device__ __forceinline__ uint32_t half_prefix_sum(uint32_t v) {
    v += dpp_u32<0x111>(v);                                      // row_shr:1, 2, 4, 8 (zero from outside the row of 16)
    v += dpp_u32<0x112>(v);
    v += dpp_u32<0x114>(v);
    v += dpp_u32<0x118>(v);
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);      // row_bcast:15 into the upper row of a half
}
// ... over all lanes
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t v) {
    v = half_prefix_sum(v);
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);      // row_bcast:31 into the upper half
}
// How many of the W lists' keys are larger than `key`; longest: the longest list's length, the same in all lanes.  Eight adjacent lanes share the scan
// and all get the sum.  Eight slots behind every list's last key are zeros.
template <int W, int CAP>
__device__ __forceinline__ int rank_in_lists(const uint64_t (*lists)[CAP], const int (&n)[W], int longest, uint64_t key, int lane) {
    int rank = 0;
    for (int q0 = 0; q0 < longest; q0 += 8) {
        uint64_t other[W];
#pragma unroll
        for (int w = 0; w < W; ++w) other[w] = lists[w][min(q0, n[w]) + (lane & 7)];
#pragma unroll
        for (int w = 0; w < W; ++w) rank += other[w] > key ? 1 : 0;
    }
    return lanes_sum(rank, 8);
}

// Orders the shared-memory accesses of one wavefront: writes before it are visible to
// the reads of the other lanes after it (the LDS serves a wavefront's requests in
// order; this keeps the compiler from reordering across the point).
__device__ __forceinline__ void lds_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace slimspec
