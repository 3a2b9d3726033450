// Per-lane stream bookkeeping of the matrix-core head kernel: every lane keeps, for each
// row it owns, a running max / sum of exp and the L largest "group maxima" of its share of the
// vocabulary (a group = the 16 logits of one row that one 32x32 MFMA tile gives a lane).
#pragma once
#include "device_utils.hpp"

namespace slimspec {

// plain VALU min / max / median without the canonicalising pre-ops the compiler adds for fmaxf
__device__ __forceinline__ float vmax(float a, float b) { float d; asm("v_max_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b)); return d; }
__device__ __forceinline__ float vmin(float a, float b) { float d; asm("v_min_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b)); return d; }
__device__ __forceinline__ float vmed3(float a, float b, float c) { float d; asm("v_med3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c)); return d; }

// ---------------------------------------------------------------------------
// Per-lane stream of one row.
template <int L>
struct Stream {
    float mc, s, U;          // running max (times log2 e), sum of exp relative to it, best dropped group maximum
    float x[L], y[L];        // group maxima (low 4 bits = position in the group) and second largest values
    int tag[L];              // group name: vocabulary tile * 8 + MFMA tile
};

constexpr float kNegBig = -3.0e38f;     // stands for "no value" (finite, so that tagging its low bits stays a number)

template <int L>
__device__ __forceinline__ void stream_init(Stream<L> &st) {
    st.mc = kNegBig; st.s = 0.f; st.U = kNegBig;
#pragma unroll
    for (int l = 0; l < L; ++l) { st.x[l] = kNegBig; st.y[l] = kNegBig; st.tag[l] = 0; }
}

__device__ __forceinline__ float vmax3(float a, float b, float c) { float d; asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c)); return d; }

// Largest and second largest of 16 values in 20 instructions: five triples (max3 / med3), then
// "top two of three pairs" = (max3 of the maxima, max(med3 of the maxima, the seconds)).
__device__ __forceinline__ void top2_of_16(const float (&p)[16], float &hi, float &lo) {
    float h[5], l[5];
#pragma unroll
    for (int t = 0; t < 5; ++t) { h[t] = vmax3(p[3 * t], p[3 * t + 1], p[3 * t + 2]); l[t] = vmed3(p[3 * t], p[3 * t + 1], p[3 * t + 2]); }
    const float ha = vmax3(h[0], h[1], h[2]);
    const float la = vmax(vmax3(vmed3(h[0], h[1], h[2]), l[0], l[1]), l[2]);
    const float hb = vmax3(h[3], h[4], p[15]);
    const float lb = vmax3(vmed3(h[3], h[4], p[15]), l[3], l[4]);
    hi = vmax(ha, hb);
    lo = vmed3(ha, hb, vmax(la, lb));
}

// Fold one group into the stream when the 16 values are base-2 logits RELATIVE to `ref` (the accumulators
// were started at -ref): the sum of 2^v needs no subtraction; the group's top two go back to absolute
// values for the list.  The caller rescales st.s and moves st.mc once per tile (see tile_max).
// NAT: the values are natural-log logits (the operand was not pre-multiplied by log2 e): one multiply more.
template <int L, bool NAT>
__device__ __forceinline__ void stream_group_rel(Stream<L> &st, const float (&v)[16], float ref, float &tile_max, int tag)
{
    float p[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) p[i] = __uint_as_float((__float_as_uint(v[i]) & 0xfffffff0u) | (uint32_t)i);
    float gr, g2r;
    top2_of_16(p, gr, g2r);
    __builtin_amdgcn_sched_barrier(0);          // the tagged copies are dead before the exponentials start
    float sum = st.s;
#pragma unroll
    for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f(NAT ? v[i] * kLog2e : v[i]);
    st.s = sum;
    float gm = __uint_as_float((__float_as_uint(gr + ref) & 0xfffffff0u) | (__float_as_uint(gr) & 15u));
    float g2 = g2r + ref;
    tile_max = vmax(tile_max, gm);
    int tg = tag;
#pragma unroll
    for (int l = 0; l < L; ++l) {
        const bool c = gm > st.x[l];
        const float nx = c ? gm : st.x[l], ny = c ? g2 : st.y[l];
        const int nt = c ? tg : st.tag[l];
        gm = c ? st.x[l] : gm; g2 = c ? st.y[l] : g2; tg = c ? st.tag[l] : tg;
        st.x[l] = nx; st.y[l] = ny; st.tag[l] = nt;
    }
    st.U = vmax(st.U, gm);
}

// Fold stream b into stream a (both cover different logits of the same row): log-sum-exp in base 2, the L
// largest group maxima of the union, U = the largest maximum that is not listed.
template <int L>
__device__ __forceinline__ void stream_combine(Stream<L> &a, const Stream<L> &b)
{
    const float m = fmaxf(a.mc, b.mc);
    a.s = a.s * __builtin_amdgcn_exp2f(a.mc - m) + b.s * __builtin_amdgcn_exp2f(b.mc - m);
    a.mc = m;
    a.U = fmaxf(a.U, b.U);
#pragma unroll
    for (int e = 0; e < L; ++e) {
        float gm = b.x[e], g2 = b.y[e];
        int tg = b.tag[e];
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const bool c = gm > a.x[l];
            const float nx = c ? gm : a.x[l], ny = c ? g2 : a.y[l];
            const int nt = c ? tg : a.tag[l];
            gm = c ? a.x[l] : gm; g2 = c ? a.y[l] : g2; tg = c ? a.tag[l] : tg;
            a.x[l] = nx; a.y[l] = ny; a.tag[l] = nt;
        }
        a.U = fmaxf(a.U, gm);
    }
}

// ---------------------------------------------------------------------------
// Gumbel-max sampling next to a stream.  The lane keeps upper bounds of z_v + g_v only (gumbel_bound_bits), in the shape of the top-k
// lists: the two groups of 16 with the largest bounds (x: the bound, its low 4 bits = position in the group; y: the group's second
// largest; tag: the group's name) and x of the best group that fell off.  The merge makes the draw of them: few elements of a row come
// within 0.1 of the winner, and each of them is evaluated exactly there.  What bounds the kernel here is vector instructions: the
// hash's 18 per element stay, but behind them there were 20 for the noise and 9 for the two best with their ids, and are 4 for the
// bound and 3 for the group's best two.
struct SampleTrack { float x[2], y[2], w3; int tag[2]; };
__device__ __forceinline__ void sample_init(SampleTrack &s) {
    s.w3 = kNegBig;
#pragma unroll
    for (int l = 0; l < 2; ++l) { s.x[l] = kNegBig; s.y[l] = kNegBig; s.tag[l] = 0; }
}
// a group's (x, y, tag) into the sorted pair
__device__ __forceinline__ void sample_insert(SampleTrack &s, float x, float y, int tag) {
#pragma unroll
    for (int l = 0; l < 2; ++l) {
        const bool c = x > s.x[l];
        const float nx = c ? x : s.x[l], ny = c ? y : s.y[l];
        const int nt = c ? tag : s.tag[l];
        x = c ? s.x[l] : x; y = c ? s.y[l] : y; tag = c ? s.tag[l] : tag;
        s.x[l] = nx; s.y[l] = ny; s.tag[l] = nt;
    }
    s.w3 = vmax(s.w3, x);
}

// The 16 values of one group (relative to `ref`, as in stream_group_rel); id_row_term: the noise's counter (id times kGumbelIdStep +
// the row's term) of element 0, element i's id is that of element 0 + 8 (i / 4) + i % 4.
template <bool NAT>
__device__ __forceinline__ void sample_group(SampleTrack &s, const float (&v)[16], float ref, uint32_t id_row_term, uint32_t hi_term, int tag)
{
    constexpr float scale = NAT ? -kGumbelBoundScale * kLn2 : -kGumbelBoundScale, base = NAT ? kGumbelBoundBase * kLn2 : kGumbelBoundBase;
    const auto bound = [&](int i) {
        const uint32_t x = gumbel_bits(id_row_term + (uint32_t)(8 * (i >> 2) + (i & 3)) * kGumbelIdStep, hi_term);
        const float w = fmaf(gumbel_bound_bits(x), scale, v[i]);
        return __uint_as_float((__float_as_uint(w) & 0xfffffff0u) | (uint32_t)i);
    };
    float p[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) p[i] = bound(i);
    float gr, g2;
    top2_of_16(p, gr, g2);
    const float at = ref + base;
    sample_insert(s, __uint_as_float((__float_as_uint(gr + at) & 0xfffffff0u) | (__float_as_uint(gr) & 15u)), g2 + at, tag);
}

// fold track b into a (both saw different logits of the same row)
__device__ __forceinline__ void sample_combine(SampleTrack &a, const SampleTrack &b)
{
    sample_insert(a, b.x[0], b.y[0], b.tag[0]);
    sample_insert(a, b.x[1], b.y[1], b.tag[1]);
    a.w3 = vmax(a.w3, b.w3);
}

// a record's part for the draw: 8 floats behind the stream's
__device__ __forceinline__ void sample_store(float *w, const SampleTrack &s) {
#pragma unroll
    for (int l = 0; l < 2; ++l) { w[3 * l] = s.x[l]; w[3 * l + 1] = s.y[l]; w[3 * l + 2] = __int_as_float(s.tag[l]); }
    w[6] = s.w3;
}
__device__ __forceinline__ void sample_load(SampleTrack &s, const float *w) {
#pragma unroll
    for (int l = 0; l < 2; ++l) { s.x[l] = w[3 * l]; s.y[l] = w[3 * l + 1]; s.tag[l] = __float_as_int(w[3 * l + 2]); }
    s.w3 = w[6];
}

// Work of block g: row block rb and the vocabulary tiles col, col + gw, col + 2 gw, ...
// Blocks are dealt round-robin to the 8 XCDs, so blocks g and g + 8 share an L2: they get the same
// vocabulary tiles and different row blocks, and so read each tile of M from HBM once.
struct HeadGrid { int n_rb, gw, n_vt, spb; };      // spb: records a block leaves per row (4, 2 or 1)

}  // namespace slimspec
