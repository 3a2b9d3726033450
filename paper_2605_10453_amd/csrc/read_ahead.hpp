// Further blocks of a launch that leaves the memory idle: they read the weights that the next kernel asks for first (plan.hpp: rows_read_ahead).
#pragma once
#include "device_utils.hpp"
#include "plan.hpp"

namespace slimspec {

// Block b of those that read ahead, NW wavefronts; b mod 8 is its XCD.  Everything read lies inside M: rows up to K - 1, whole groups
// of 8 columns below V.  (No load is conditional: the compiler waits for a load where the paths around it meet.)
template <int NW>
__device__ __forceinline__ void read_ahead_block(const ReadAhead &a, int b)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    AheadSlot s = ahead_slot(a, b & 7, (b >> 3) * NW + wave);
    int kp = 0;                                             // lane / lanes
    for (int first = a.lanes; first < 64; first += a.lanes) kp += lane >= first ? 1 : 0;
    const int col = s.col0 + 8 * (lane - kp * a.lanes);
    if (!s.on || kp >= a.rows_step || col >= a.V) return;
    const uint32_t off = (uint32_t)kp * (uint32_t)a.V + (uint32_t)col;      // (kp < 4: a unit has at least 16 lanes)
    u32x4 w[kAheadLoads];
#pragma unroll
    for (int n = 0; n < kAheadLoads; ++n) {
        w[n] = *reinterpret_cast<const u32x4 *>(a.M + (size_t)ahead_row(a, s) * a.V + off);
        ahead_next(a, s);
    }
#pragma unroll
    for (int n = 0; n < kAheadLoads; ++n) asm volatile("" :: "v"(w[n]));
}

}  // namespace slimspec
