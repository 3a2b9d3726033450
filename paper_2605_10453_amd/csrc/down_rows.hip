// Down-projection t = h A for calls of a few rows (paper section 4.1, the first of the two dense products), written as the three
// bf16 pieces of every element that rows_topk_kernel multiplies with.
//
// What bounds it: latency.  A is a few megabytes and the chip could read it in a microsecond, but a split of the contraction over
// blocks needs a second launch that adds the parts (3.6 to 4.7 us after the 3.6 to 5.2 us of the first).  Here a block owns 16
// columns of t for all rows of a group and its 16 wavefronts split the contraction, so that the parts meet in shared memory:
//   * a step is 32 contraction elements: one 16-byte load per lane of A (32 rows of 32 bytes; four adjacent blocks, which share
//     the lines, sit on one XCD) and one of h per 16 rows, as the MFMA wants it.  A is turned by the transposing LDS read
//     (a wavefront's own kilobyte, no barrier).  kDRBatch steps are in flight per wavefront;
//   * every step is summed on its own and then added, as in the kernels it feeds: the matrix unit's internal roundings then
//     happen at the size of one step's sum.
#include "device_utils.hpp"
#include "launch.hpp"
#include "read_ahead.hpp"

namespace slimspec {

namespace {

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#define LDS_PTR(T, byte_addr) ((__attribute__((address_space(3))) T *)(uintptr_t)(byte_addr))

constexpr int kDRWaves = 16;
constexpr int kDRCols = 16;

}  // namespace

// X: [3][8 ceil(r / 64)][rows_pad] 16-byte vectors of 8 consecutive columns of t; zero beyond r and beyond the last row.
// Block (XCD-aware number b of a 16-column tile, group y): the rows of group y with the group's matrix; NT: 16-row tiles of the
// largest group.  Blocks beyond the tiles read weights ahead.
template <int NT>
__global__ __launch_bounds__(64 * kDRWaves) void down_rows_kernel(
    const uint16_t *__restrict__ h, const uint16_t *__restrict__ A, uint4 *__restrict__ X, int rows_pad, int d, int r, DownGrid g, ReadAhead ahead)
{
    constexpr int kDRBatch = NT == 1 ? 8 : 4;                          // steps in flight per wavefront
    __shared__ __align__(16) float part[kDRWaves][NT][4][64];          // [wavefront][row tile][element][lane]; before that the wavefronts' tiles of A
    __shared__ float t_tile[NT * 16][kDRCols + 1];
    static_assert(sizeof(part[0]) >= 1024, "a wavefront's 32 x 16 tile of A fits where its sums go later");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_tiles = (r + 63) / 64 * 4;
    if ((int)blockIdx.x >= n_tiles) {
        const int first = (n_tiles + 7) & ~7, n_each = (int)gridDim.x - first;         // (of every group, a multiple of 8)
        if ((int)blockIdx.x >= first) read_ahead_block<kDRWaves>(ahead, (int)blockIdx.y * n_each + (int)blockIdx.x - first);
        return;
    }
    const int tile = (n_tiles & 7) == 0 ? (int)(blockIdx.x & 7) * (n_tiles >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    const int grp = blockIdx.y, n0 = tile * kDRCols;
    const int lo = g.g_row0[grp], hi = g.g_row0[grp + 1];
    const int kg = lane >> 4, l16 = lane & 15;

    f32x4 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[nt][i] = 0.f;

    const int n_steps = (d + 31) / 32, per = (n_steps + kDRWaves - 1) / kDRWaves;
    const int s_beg = min(n_steps, wave * per), s_end = (n0 < r) ? min(n_steps, s_beg + per) : s_beg;      // columns of padding load nothing
    if (s_beg < s_end) {
        const uint32_t buf = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) float *)&part[wave][0][0][0]);
        const uint16_t *a_src = A + (size_t)g.g_mat[grp] * d * r + min(n0 + 8 * (lane & 1), r - 8);        // (r is a multiple of 8; a column beyond it is not used)
        u32x4 a[kDRBatch], x[kDRBatch][NT];
        for (int s0 = s_beg; s0 < s_end; s0 += kDRBatch) {
#pragma unroll
            for (int u = 0; u < kDRBatch; ++u) {
                if (s0 + u >= s_end) continue;
                // d is a multiple of 8: of the last step's elements those beyond d are cleared below, in both operands
                const int k0 = 32 * (s0 + u);
                a[u] = *reinterpret_cast<const u32x4 *>(a_src + (size_t)min(k0 + (lane >> 1), d - 1) * r);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    x[u][nt] = *reinterpret_cast<const u32x4 *>(h + (size_t)min(lo + 16 * nt + l16, hi - 1) * d + min(k0 + 8 * kg, d - 8));
            }
#pragma unroll
            for (int u = 0; u < kDRBatch; ++u) {
                if (s0 + u >= s_end) continue;
                const int k0 = 32 * (s0 + u);
                if (k0 + 32 > d) {
                    const uint32_t keep_a = k0 + (lane >> 1) < d ? 0xffffffffu : 0u, keep_x = k0 + 8 * kg < d ? 0xffffffffu : 0u;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        a[u][e] &= keep_a;
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) x[u][nt][e] &= keep_x;
                    }
                }
                lds_wave_sync();                                 // the step before has been read
                *LDS_PTR(u32x4, buf + 16 * lane) = a[u];
                lds_wave_sync();
                const uint32_t at = buf + (uint32_t)(8 * kg + (l16 >> 2)) * 32u + (uint32_t)(l16 & 3) * 8u;
                const v4i16 first = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(v4i16, at));
                const v4i16 second = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(v4i16, at + 128));
                const bf16x8 af = __builtin_bit_cast(bf16x8, __builtin_shufflevector(first, second, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                    acc[nt] += __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, __builtin_bit_cast(bf16x8, x[u][nt]), zero, 0, 0, 0);
                }
            }
        }
        lds_wave_sync();
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) part[wave][nt][i][lane] = acc[nt][i];
    __syncthreads();
    // element (column 4 (lane / 16) + i, row lane % 16) of a tile: the wavefronts' sums in order
    for (int e = tid; e < NT * 256; e += 64 * kDRWaves) {
        const int nt = e >> 8, i = (e >> 6) & 3, ln = e & 63;
        float v[kDRWaves], s = 0.f;
#pragma unroll
        for (int w = 0; w < kDRWaves; ++w) v[w] = part[w][nt][i][ln];
#pragma unroll
        for (int w = 0; w < kDRWaves; ++w) s += v[w];
        t_tile[16 * nt + (ln & 15)][4 * (ln >> 4) + i] = s;
    }
    __syncthreads();
    // thread (row, 8 columns): the pieces.  The last group's
    // block also clears the rows of padding.
    const int row_end = grp + 1 == (int)gridDim.y ? rows_pad : hi;
    const size_t piece_stride = (size_t)((r + 63) / 64 * 8) * rows_pad;
    for (int e = tid; e < 2 * (row_end - lo); e += 64 * kDRWaves) {
        const int row = lo + (e >> 1), col = 8 * (e & 1);
        const bool valid = row < hi && n0 + col < r;
        float v[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = valid ? t_tile[row - lo][col + c] : 0.f;
        uint4 piece[3];
        cut_pieces(v, piece);
#pragma unroll
        for (int p = 0; p < 3; ++p)
            X[p * piece_stride + (size_t)((n0 + col) >> 3) * rows_pad + row] = piece[p];
    }
}

template <int NT>
static hipError_t launch_down_rows_nt(const uint16_t *h, const uint16_t *A, void *X, int rows_pad, int d, int r, const DownGrid &g, const ReadAhead &ahead, hipStream_t st)
{
    const int n_tiles = (r + 63) / 64 * 4, n_each = ahead_blocks_each(ahead, g.n_groups);
    const dim3 grid(n_each ? (n_tiles + 7) / 8 * 8 + n_each : n_tiles, g.n_groups);
    down_rows_kernel<NT><<<grid, 64 * kDRWaves, 0, st>>>(h, A, static_cast<uint4 *>(X), rows_pad, d, r, g, ahead);
    return hipGetLastError();
}

hipError_t launch_down_rows(const uint16_t *h, const uint16_t *A, void *X, int rows_pad, int d, int r, const DownGrid &g, const ReadAhead &ahead, hipStream_t st)
{
    const int most = largest_group(g);
    if (most <= 16) return launch_down_rows_nt<1>(h, A, X, rows_pad, d, r, g, ahead, st);
    if (most <= 32) return launch_down_rows_nt<2>(h, A, X, rows_pad, d, r, g, ahead, st);
    return launch_down_rows_nt<3>(h, A, X, rows_pad, d, r, g, ahead, st);
}

}  // namespace slimspec
