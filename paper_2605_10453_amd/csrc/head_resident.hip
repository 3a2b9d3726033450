// Vocabulary projection with the fused log-sum-exp / top-k epilogue for many rows and a contraction of up to 512
// elements (paper section 4.1: logits = t B, never written to memory), the row operand resident in registers.
//
// What bounds it: the matrix cores and, next to them, what feeds them.  head_tile_kernel reads both operands of every
// MFMA from LDS (0.75 KB each), loads the rows again with every stage, and runs its epilogue (a fifth of its time)
// while the matrix cores wait.  Here
//   * a wavefront owns 32 rows for the whole kernel and keeps their operand in registers: 32 rows x 512 elements are 128
//     of the 256 registers per lane that two wavefronts per SIMD have each.  Only the weights pass through LDS;
//   * the tiles are 64 columns wide, so the accumulators (32 registers) exist twice: while one tile accumulates, the
//     epilogue of the tile before runs in the vector-instruction slots that MFMAs leave free.
// (One wavefront per SIMD with 64 rows and 512 registers reads each fragment for two MFMAs, but a wavefront issues one
// instruction in four cycles, and the epilogue's and the loads' no longer fit between the MFMAs: 73 us at 512 rows.)
// A block is eight wavefronts, 256 rows, one block per CU; it walks the 64-column tiles col, col + gw, col + 2 gw, ...
// Blocks that share tiles (different row blocks) sit on the same XCD.
//
// Measured at 512 rows, V = 128256 (kernel; head_tile_kernel in brackets): r = 512 66.9 us (72-75), r = 256 41.6 us (44-46);
// calls with prepared weights 112 -> 105 us and 78.7 -> 69.7 us, 700 rows 178 -> 165 us, 512 rows at r = 128, V = 32000
// 42.3 -> 37.8 us.  A tile takes 6000 cycles of the 4096 that its MFMAs occupy; what is left over is the wavefronts' issue
// slots (1200 cycles without loads and barriers), the loads into LDS (900) and the barriers (300).  12000 cycles pass
// before the first MFMA: 256 KB of row operand per CU at the 30 bytes per cycle a CU takes in.
//
// Sampling: the draw's bounds are 22 vector instructions per logit, more than all the rest, and run between the MFMAs too: 512 rows, r = 512
// 97 to 112 us by the profiler, 154 in head_tile_kernel with the noise itself; calls 223.3 (there; 182 with bounds) -> 159.6 us, with a row
// whose best groups crowd into one record 223.4 -> 222.3 (prepared 197.3 -> 136.2 and 197.8 -> 188.5); 300 rows, r = 256, prepared 152.2 -> 100.5.
//
// Weights: stages of 128 contraction elements x 64 columns (16 KB) travel global memory -> LDS without passing registers
// (global_load_lds_dwordx4), eight stage buffers.  The 16-byte pieces of a 128-byte stage row are stored XOR-swizzled by
// twice (row mod 4), so that the four rows of a transposing read (ds_read_b64_tr_b16) fall into different banks.
// The compiler does not see these loads: every wavefront issues exactly two per stage, vector memory returns in order,
// and "s_waitcnt vmcnt(N)" means that the stages needed next have landed (see do_tile).  Nothing else in the loop may use
// vector memory: the kernel must not spill (for which it needs the build's -amdgpu-mfma-vgpr-form).
#include "head_stream.hpp"
#include "launch.hpp"
#include <type_traits>

namespace slimspec {

namespace {

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#define LDS_PTR(T, byte_addr) ((__attribute__((address_space(3))) T *)(uintptr_t)(byte_addr))

constexpr int kRTile = kResidentTileCols;                 // columns per tile
constexpr int kRStageK = 128;                             // contraction elements per stage
constexpr uint32_t kRStageBytes = kRStageK * kRTile * 2;  // 16 KB
constexpr int kRNB = 8;                                   // stage buffers
constexpr int kRLoads = 2;                                // loads per wavefront and stage, 8 stage rows each
constexpr int kAhead = 1;                                 // contraction steps that weight fragments are read ahead
constexpr int kSlots = 32;                                // slots of an MFMA tile's epilogue
constexpr int kSampleSlots = 32;                          // ... and of its noise: two for each of its 16 elements

template <int OFF>
__device__ __forceinline__ void dma16(uint32_t buf, uint32_t voff, const void *base) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(buf), "v"(voff), "s"(base), "n"(OFF) : "memory", "scc");
}
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }
__device__ __forceinline__ void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
template <int N> using Int = std::integral_constant<int, N>;

// calls f(Int<B>{}), ..., f(Int<E - 1>{})
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F f) {
    if constexpr (B < E) { f(Int<B>{}); static_for<B + 1, E>(f); }
}

constexpr float kNoMax = -1.0e30f;                        // a reference for a stream that has seen masked columns only

}  // namespace

// X: [8 ceil(K / 64)][rows_pad] 16-byte vectors: t log2(e) in bf16, 8 consecutive contraction elements of one row, zero
//    beyond K and beyond the last row; rows_pad a multiple of 256.  M: [K][V] bf16 row-major, K and V multiples of 8.
// part: [rows][gw * 2] records as head_tile_kernel writes them, one per half-wavefront.
// KS: contraction steps of 16, ceil(K / 128) * 8.  split (16, 32 or 64, at least K; 0: one piece): X holds two pieces of
// every element, [2][split / 8][rows_pad].
// SAMPLE: the records also carry what the Gumbel-max draw needs (head_stream.hpp; the second group's y is folded into the bound of
// all others): 20 floats.
template <int KS, bool SAMPLE>
__global__ __launch_bounds__(512, 2) void head_resident_kernel(
    const uint4 *__restrict__ X, const uint16_t *__restrict__ M, float *__restrict__ part,
    int rows, int rows_pad, int K, int V, int split, ResidentGrid hg, uint32_t seed_lo, uint32_t seed_hi, int row_base)
{
    constexpr int L = kStreamList, REC = SAMPLE ? kStreamRecSample : kStreamRec;
    constexpr int SPT = KS / 8;                           // stages per tile
    constexpr int SYNC = SPT % 2 == 0 ? 2 : 1;            // stages per barrier (two: 70.5 -> 68.6 us at 512 rows)
    extern __shared__ __align__(1024) unsigned char lds_raw[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) unsigned char *)lds_raw);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31, g1 = (lane >> 4) & 1, j16 = lane & 15;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int rb = slot % hg.n_rb, col = (slot / hg.n_rb) * 8 + xcd;
    const int row0 = rb * 256 + wave * 32;
    const int n_tiles = (col < hg.n_t) ? (hg.n_t - col + hg.gw - 1) / hg.gw : 0;
    const int n_stages = n_tiles * SPT;

    Stream<L> st;
    stream_init(st);
    // the draw's bounds: largest group (x, second largest y), second largest group (x), all others; the two groups' names, 2 (tile - col) / gw
    // + MFMA tile, as 16 bits each (V <= kResidentMaxV)
    static_assert(2 * ((kResidentMaxV / kResidentTileCols + 7) / 8) <= 1 << 16, "a group's name fits 16 bits");
    float smp_x = kNegBig, smp_y = kNegBig, smp_x2 = kNegBig, smp_rest = kNegBig;
    uint32_t smp_tags = 0u;

    if (n_tiles > 0) {
        // ---- direct-to-LDS loads.  Load u of this wavefront: stage rows 16 wave + 8 u + lane / 8; stored piece lane % 8
        // holds source piece (lane % 8) ^ 2 (row % 4).  A lane's byte offsets from the stage's corner are kept in
        // registers, so that a stage costs few scalar instructions, which take issue slots from everything else.
        static_assert((uint64_t)kRStageK * 2u * kResidentMaxV <= (uint64_t)1 << 32, "a stage's offsets fit 32 bits");
        const uint32_t rowb = (uint32_t)V * 2u;
        const uint32_t src_piece = (uint32_t)((lane & 7) ^ (((lane >> 3) & 3) << 1)) * 16u;
        uint32_t voff[kRLoads];
        // two pieces of t (K <= 64, one stage) meet the same rows
        const int row_mask = KS == 8 && split ? split - 1 : kRStageK - 1;
        const auto set_offsets = [&](int t, int st_k) {
            // columns beyond V re-read the last 16 bytes that exist, rows beyond K the last 8 (they meet zeros of X);
            // K is a multiple of 8: the 8 rows of a load all exist or none does
            const uint32_t c = min(src_piece, (uint32_t)(V - t * kRTile - 8) * 2u);
#pragma unroll
            for (int u = 0; u < kRLoads; ++u)
                voff[u] = (uint32_t)(min((16 * wave + 8 * u) & row_mask, K - 8 - st_k * kRStageK) + (lane >> 3)) * rowb + c;
        };
        const size_t stage_step = (size_t)kRStageK * rowb;
        const bool ragged_k = (K & (kRStageK - 1)) != 0;
        const unsigned char *src = reinterpret_cast<const unsigned char *>(M) + (size_t)col * (kRTile * 2);
        const unsigned char *tile_src = src;
        int a_t = col, a_st = 0;                          // the stage loaded next: tile, stage of the tile
        uint32_t buf_ahead = lds0 + (uint32_t)wave * 2048u;
        const uint32_t buf_end = buf_ahead + kRNB * kRStageBytes;
        int left = n_stages;                              // stages not yet asked for
        const auto issue_load = [&](auto u_tag) { constexpr int u = decltype(u_tag)::value; dma16<1024 * u>(buf_ahead, voff[u], src); };
        const auto advance_loads = [&]() {
            buf_ahead += kRStageBytes;
            buf_ahead = (buf_ahead == buf_end) ? buf_end - kRNB * kRStageBytes : buf_ahead;
            // past the end the last stage is loaded again (nobody reads it): the count stays uniform
            if (--left > 0) {
                src += stage_step;
                if (++a_st == SPT) {
                    a_st = 0; a_t += hg.gw;
                    tile_src += (size_t)hg.gw * (kRTile * 2);
                    src = tile_src;
                    if (ragged_k || a_t * kRTile + kRTile > V) set_offsets(a_t, 0);
                }
                if (ragged_k && a_st == SPT - 1) set_offsets(a_t, a_st);
            }
        };
        set_offsets(col, 0);
#pragma unroll
        for (int pre = 0; pre < kRNB - 1; ++pre) {
            static_for<0, kRLoads>(issue_load);
            advance_loads();
        }

        // ---- the rows' operand: lane (row l32, contraction elements 16 s + 8 half ...)
        u32x4 xr[KS];
        {
            const int n_groups = KS == 8 && split ? split / 4 : (K + 63) / 64 * 8;      // 8-element groups that X holds
            const uint4 *src = X + (size_t)half * rows_pad + row0 + l32;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                u32x4 v = {0u, 0u, 0u, 0u};
                if (2 * s < n_groups) v = *reinterpret_cast<const u32x4 *>(src + (size_t)(2 * s) * rows_pad);
                xr[s] = v;
            }
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) asm volatile("" : "+a"(xr[s]));      // kept in accumulation registers
        wait_loads<0>();
        __builtin_amdgcn_s_barrier();

        // ---- weight fragments: MFMA tile jj of step ks at (buf + ma0) ^ (jj << 6), + 2048 per step, + 512 for the second half
        const uint32_t ma0 = (uint32_t)((8 * half + (j16 >> 2)) * 128
                                        + (((2 * g1 + ((j16 & 3) >> 1)) ^ ((j16 >> 2) << 1)) * 16) + (j16 & 1) * 8);
        // Read kAhead steps before their MFMAs.
        v4i16 mf[kAhead + 1][2][2];                       // [step mod (kAhead + 1)][jj][half of the fragment]
        const auto read_frag = [&](const uint32_t (&addr)[2], auto ks_tag, auto slot_tag, auto part_tag) {
            constexpr int ks = decltype(ks_tag)::value, slot = decltype(slot_tag)::value, part = decltype(part_tag)::value;
            mf[slot][part >> 1][part & 1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(v4i16, addr[part >> 1] + ks * 2048 + (part & 1) * 512));
        };

        // ---- epilogue of the tile before (head_stream.hpp explains the bookkeeping; here the logits are absolute and the
        // running maximum moves with every group of 16, so that no exponent is ever positive).  A wavefront issues in order
        // and an MFMA occupies the matrix cores for 32 cycles, so no more than 24 cycles of vector instructions (six, or an
        // exponential and two) may stand between two MFMAs: with four MFMAs in a row and 20 instructions after them the
        // same work takes 183 cycles instead of 134.  The epilogue of an MFMA tile is therefore cut into 28 slots of that
        // size, four more are left free for the loads of a stage, and each slot stays behind its MFMA (scheduling barriers,
        // and empty asm statements that keep the compiler from moving sums to where they are read).
        f32x16 acc[2][2];                                 // [tile parity][jj]
        float p[3], h5[5], l5[5], ha = 0.f, hb = 0.f, la = 0.f, gr = 0.f, g2 = 0.f, e0 = 0.f;
        int tg = 0;
        uint32_t hx = 0u, id_row = 0u;                    // (sampling)
        constexpr int SLOTS = kSlots + (SAMPLE ? kSampleSlots : 0);
        const auto epilogue_slot = [&](auto u_tag, f32x16 (&a)[2], int tile, int nth) {
            constexpr int U = decltype(u_tag)::value, jj = U / SLOTS, at = U % SLOTS;
            constexpr int w = at < 20 ? at : at < 24 ? -1 : at < kSlots ? at - 4 : -1;      // 20 .. 23: free
            Stream<L> &q = st;
            const f32x16 &v = a[jj];
#define SLIMSPEC_PIN(x) asm volatile("" : "+v"(x))
            const auto level = [&](int l) {               // one level of the sorted list: (gr, g2, tg) in, what falls out out
                const bool c = gr > q.x[l];
                const float nx = c ? gr : q.x[l], ny = c ? g2 : q.y[l];
                const int nt = c ? tg : q.tag[l];
                gr = c ? q.x[l] : gr; g2 = c ? q.y[l] : g2; tg = c ? q.tag[l] : tg;
                q.x[l] = nx; q.y[l] = ny; q.tag[l] = nt;
                SLIMSPEC_PIN(q.x[l]); SLIMSPEC_PIN(q.y[l]); SLIMSPEC_PIN(q.tag[l]); SLIMSPEC_PIN(gr); SLIMSPEC_PIN(g2); SLIMSPEC_PIN(tg);
            };
            const auto tagged = [&](int i) { return __uint_as_float((__float_as_uint(v[i]) & 0xfffffff0u) | (uint32_t)i); };
            if constexpr (w >= 0 && w < 5) {              // three elements: tags, largest, second largest
                p[0] = tagged(3 * w); p[1] = tagged(3 * w + 1); p[2] = tagged(3 * w + 2);
                h5[w] = vmax3(p[0], p[1], p[2]); l5[w] = vmed3(p[0], p[1], p[2]);
                SLIMSPEC_PIN(h5[w]); SLIMSPEC_PIN(l5[w]);
            } else if constexpr (w == 5) {
                ha = vmax3(h5[0], h5[1], h5[2]);
                la = vmax(vmax3(vmed3(h5[0], h5[1], h5[2]), l5[0], l5[1]), l5[2]);
                p[0] = tagged(15);
                hb = vmax3(h5[3], h5[4], p[0]);
                SLIMSPEC_PIN(ha); SLIMSPEC_PIN(la); SLIMSPEC_PIN(hb); SLIMSPEC_PIN(p[0]);
            } else if constexpr (w == 6) {
                const float lb = vmax3(vmed3(h5[3], h5[4], p[0]), l5[3], l5[4]);
                gr = vmax(ha, hb);
                g2 = vmed3(ha, hb, vmax(la, lb));
                SLIMSPEC_PIN(gr); SLIMSPEC_PIN(g2);
            } else if constexpr (w == 7) {
                const float m = vmax3(q.mc, gr, kNoMax);
                e0 = __builtin_amdgcn_exp2f(q.mc - m);
                q.mc = m;
                SLIMSPEC_PIN(e0); SLIMSPEC_PIN(q.mc);
            } else if constexpr (w >= 8 && w < 24) {      // the exponential of one element, the sum with the one before
                const float e1 = __builtin_amdgcn_exp2f(v[w - 8] - q.mc);
                q.s = w == 8 ? q.s * e0 : q.s + e0;
                e0 = e1;
                SLIMSPEC_PIN(e0); SLIMSPEC_PIN(q.s);
            } else if constexpr (w == 24) {
                q.s += e0;
                tg = tile * 2 + jj;
                SLIMSPEC_PIN(q.s); SLIMSPEC_PIN(tg);
            } else if constexpr (w == 25) level(0);
            else if constexpr (w == 26) level(1);
            else if constexpr (w == 27) { level(2); q.U = vmax(q.U, gr); SLIMSPEC_PIN(q.U); }
            if constexpr (at >= kSlots) {                 // the draw, behind the rest: element i in two slots; gr and g2 are the group's best two here
                constexpr int i = (at - kSlots) >> 1;
                const uint32_t hi_term = seed_hi * 0xC2B2AE3Du;
                if constexpr (((at - kSlots) & 1) == 0) {
                    if constexpr (i == 0) {
                        const uint32_t ln = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));      // (recomputed: a register less)
                        id_row = (uint32_t)(tile * kRTile + 32 * jj) * kGumbelIdStep + (ln >> 5) * (4u * kGumbelIdStep)
                                 + gumbel_key(seed_lo, seed_hi, (uint32_t)(row_base + row0)).row_term + (ln & 31) * kGumbelRowStep;
                        SLIMSPEC_PIN(id_row);
                    }
                    hx = mix32(id_row + (uint32_t)(8 * (i >> 2) + (i & 3)) * kGumbelIdStep) + hi_term;
                    SLIMSPEC_PIN(hx);
                } else {
                    const float b = fmaf(gumbel_bound_bits(mix32(hx)), -kGumbelBoundScale, v[i]);
                    const float p = __uint_as_float((__float_as_uint(b) & 0xfffffff0u) | (uint32_t)i);
                    if constexpr (i == 0) { gr = p; g2 = kNegBig; }
                    else { g2 = vmed3(gr, g2, p); gr = vmax(gr, p); }
                    SLIMSPEC_PIN(gr); SLIMSPEC_PIN(g2);
                }
                if constexpr (at == SLOTS - 1) {
                    float x = __uint_as_float((__float_as_uint(gr + kGumbelBoundBase) & 0xfffffff0u) | (__float_as_uint(gr) & 15u));
                    float y = g2 + kGumbelBoundBase;
                    const bool c1 = x > smp_x, c2 = x > smp_x2;
                    smp_rest = vmax(smp_rest, c1 ? vmax(smp_x2, smp_y) : vmax(y, c2 ? smp_x2 : x));
                    smp_tags = c1 ? smp_tags << 16 | (uint32_t)(2 * nth + jj) : c2 ? (smp_tags & 0xffffu) | (uint32_t)(2 * nth + jj) << 16 : smp_tags;
                    smp_x2 = c1 ? smp_x : c2 ? x : smp_x2;
                    smp_y = c1 ? y : smp_y;
                    smp_x = c1 ? x : smp_x;
                    SLIMSPEC_PIN(smp_rest); SLIMSPEC_PIN(smp_tags); SLIMSPEC_PIN(smp_x2); SLIMSPEC_PIN(smp_y); SLIMSPEC_PIN(smp_x);
                }
            }
#undef SLIMSPEC_PIN
        };
        const auto mask_tail = [&](f32x16 (&a)[2], int tile) {
            if (tile * kRTile + kRTile > V) {             // the vocabulary's last tile
#pragma unroll
                for (int jj = 0; jj < 2; ++jj) {
                    const int cbase = tile * kRTile + 32 * jj + 4 * half;
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (cbase + 8 * (i >> 2) + (i & 3) >= V) a[jj][i] = kNegBig;
                }
            }
        };

        uint32_t buf = lds0;
        // (the lane's addresses in the stage read next, one per MFMA tile, set once per stage)
        uint32_t frag_addr[2];
        const auto set_frag_addr = [&]() {
            frag_addr[0] = buf + ma0; frag_addr[1] = (buf + ma0) ^ 64u;
            asm volatile("" : "+v"(frag_addr[0]), "+v"(frag_addr[1]));
        };
        set_frag_addr();
        static_for<0, kAhead>([&](auto k_tag) { static_for<0, 4>([&](auto part_tag) { read_frag(frag_addr, k_tag, k_tag, part_tag); }); });
        // One tile: its MFMAs, and between them the epilogue of the tile before (EPI)
        const auto do_tile = [&](auto par_tag, auto epi_tag, int nth) {
            const int tile = col + nth * hg.gw;
            constexpr int P = decltype(par_tag)::value;
            constexpr bool EPI = decltype(epi_tag)::value != 0;
            const int prev = tile - hg.gw;
            if constexpr (EPI) mask_tail(acc[1 - P], prev);
            static_for<0, 2 * KS>([&](auto mfma_tag) {
                constexpr int n = decltype(mfma_tag)::value, k = n >> 1, jj = n & 1;
                constexpr int ks = k & 7, now = k % (kAhead + 1);
                f32x16 c = acc[P][jj];
                if constexpr (k == 0) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) c[i] = 0.f;
                }
                acc[P][jj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8, __builtin_shufflevector(mf[now][jj][0], mf[now][jj][1], 0, 1, 2, 3, 4, 5, 6, 7)),
                    __builtin_bit_cast(bf16x8, xr[k]), c, 0, 0, 0);
                constexpr bool stage_end = ks == 8 - kAhead && jj == 0;
                if constexpr (stage_end && ((k >> 3) + 1) % SYNC == 0) {
                    // The next SYNC stages have landed, in every wavefront's share: stage q ends here, up to stage
                    // q + kRNB - 2 is asked for (with either SYNC), q + SYNC is needed.  And every wavefront's reads of
                    // stage q have returned, the fragment of the MFMA after this one included: until the next barrier the
                    // buffers of stages q - 1 (SYNC 1) or q - 1 and q (SYNC 2) are loaded again.
                    wait_loads<(kRNB - 2 - SYNC) * kRLoads>();
                    wait_lds_reads();
                    __builtin_amdgcn_s_barrier();
                }
                if constexpr (stage_end) {
                    buf = (buf + kRStageBytes == lds0 + kRNB * kRStageBytes) ? lds0 : buf + kRStageBytes;
                    set_frag_addr();
                }
                if constexpr (SYNC == 1 ? ks == 8 - kAhead : ((k & 15) == 16 - kAhead || (k & 15) == 5)) {
                    issue_load(Int<jj>{});
                    if constexpr (jj == 1) advance_loads();
                }
                // (after the last stage: a buffer loaded again, unused)
                read_frag(frag_addr, Int<(ks + kAhead) & 7>{}, Int<(k + kAhead) % (kAhead + 1)>{}, Int<2 * jj>{});
                read_frag(frag_addr, Int<(ks + kAhead) & 7>{}, Int<(k + kAhead) % (kAhead + 1)>{}, Int<2 * jj + 1>{});
                if constexpr (EPI) static_for<n * SLOTS / KS, (n + 1) * SLOTS / KS>([&](auto u_tag) { epilogue_slot(u_tag, acc[1 - P], prev, nth - 1); });
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        const auto drain = [&](auto par_tag, int nth) {
            constexpr int P = decltype(par_tag)::value;
            mask_tail(acc[P], col + nth * hg.gw);
            static_for<0, 2 * SLOTS>([&](auto u_tag) { epilogue_slot(u_tag, acc[P], col + nth * hg.gw, nth); });
        };
        do_tile(Int<0>{}, Int<0>{}, 0);
        int i = 1;
        for (; i + 1 < n_tiles; i += 2) {
            do_tile(Int<1>{}, Int<1>{}, i);                          // with it, the epilogue of tile i - 1 is done
            do_tile(Int<0>{}, Int<1>{}, i + 1);
        }
        if (i < n_tiles) {
            do_tile(Int<1>{}, Int<1>{}, i);
            drain(Int<1>{}, i);
        } else
            drain(Int<0>{}, n_tiles - 1);
        wait_loads<0>();                                  // the surplus loads of the last stages
    }

    // ---- records.  Lane by lane they would be 48-byte pieces in rows far apart; through LDS (the stage buffers are free by
    // now) a wavefront writes every row's records of this block as one contiguous run.
    __syncthreads();
    constexpr int ROW_BYTES = 2 * REC * 4, PIECES = ROW_BYTES / 16;
    unsigned char *const rec_lds = lds_raw + wave * (32 * ROW_BYTES);       // [32 rows][half][REC]
    {
        float *o = reinterpret_cast<float *>(rec_lds + l32 * ROW_BYTES) + half * REC;
        o[0] = st.mc; o[1] = st.s; o[2] = st.U;
#pragma unroll
        for (int l = 0; l < L; ++l) { o[3 + 3 * l] = st.x[l]; o[4 + 3 * l] = st.y[l]; o[5 + 3 * l] = __int_as_float(st.tag[l] * 2 + half); }
        if constexpr (SAMPLE) {
            const auto name = [&](uint32_t t) { return ((col + (int)(t >> 1) * hg.gw) * 2 + (int)(t & 1u)) * 2 + half; };
            sample_store(o + kStreamRec, {{smp_x, smp_x2}, {smp_y, kNegBig}, smp_rest, {name(smp_tags & 0xffffu), name(smp_tags >> 16)}});
        }
    }
    lds_wave_sync();
#pragma unroll
    for (int e = lane; e < 32 * PIECES; e += 64) {
        const int r = e / PIECES, row = row0 + r;
        if (row < rows)
            *reinterpret_cast<float4 *>(part + ((size_t)row * hg.gw + col) * (2 * REC) + 4 * (e - r * PIECES)) =
                *reinterpret_cast<const float4 *>(rec_lds + e * 16);
    }
}

template <int KS, bool SAMPLE>
static hipError_t launch_resident(const void *X, int split, const uint16_t *M, float *part, int rows, int rows_pad, int K, int V,
                                  const ResidentGrid &g, const SampleOut &so, int row_base, hipStream_t st)
{
    const int lds = kRNB * (int)kRStageBytes;
    static LdsLimit lds_limit;
    hipError_t e = lds_limit.raise(reinterpret_cast<const void *>(head_resident_kernel<KS, SAMPLE>), lds);
    if (e != hipSuccess) return e;
    head_resident_kernel<KS, SAMPLE><<<g.n_rb * g.gw, 512, lds, st>>>(static_cast<const uint4 *>(X), M, part, rows, rows_pad, K, V, split, g,
                                                                      so.seed_lo, so.seed_hi, row_base);
    return hipGetLastError();
}

hipError_t launch_head_resident(const void *X, Operand operand, const uint16_t *M, float *part, int rows, int rows_pad, int K, int V,
                                const ResidentGrid &g, const SampleOut &so, int row_base, hipStream_t st)
{
    const int split = operand == kOperandTwoBf16 ? two_pieces_stride(K) : 0;
#define SLIMSPEC_RESIDENT(KS) (so.on ? launch_resident<KS, true>(X, split, M, part, rows, rows_pad, K, V, g, so, row_base, st) \
                                     : launch_resident<KS, false>(X, split, M, part, rows, rows_pad, K, V, g, so, row_base, st))
    if (K <= 128) return SLIMSPEC_RESIDENT(8);
    if (K <= 256) return SLIMSPEC_RESIDENT(16);
    if (K <= 384) return SLIMSPEC_RESIDENT(24);
    return SLIMSPEC_RESIDENT(32);
#undef SLIMSPEC_RESIDENT
}

}  // namespace slimspec
