// What the matrix-product kernels with whole-line stages share: fragments and their MFMA, the barrier of their rings, the order of tiles.
#pragma once

#include "gfx950_prims.h"
#include "tile_schedule.h"

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

constexpr int T_GROUP_M = 8;                    // tile rows per raster group: see tile_coords in gemm_nt_kernel.hip

// Workgroup barrier that no LDS access of the compiler's moves across (the copies' arrival is not visible to it).
__device__ __forceinline__ void ring_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// One k-step of one 32-row block: 16 bytes per lane (16-bit operands) or 32 (E4M3).
template <int IN> struct TileFrag { i32x4 h[IN == 2 ? 2 : 1]; };

template <int IN>
__device__ __forceinline__ f32x16 tile_mfma(const TileFrag<IN>& a, const TileFrag<IN>& b, f32x16 c)
{
    if constexpr (IN == 2) {
        const i32x8 x = __builtin_shufflevector(a.h[0], a.h[1], 0, 1, 2, 3, 4, 5, 6, 7);
        const i32x8 y = __builtin_shufflevector(b.h[0], b.h[1], 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, y, c, 0, 0, 0, 0, 0, 0);   // scales 0: unscaled E4M3
    } else {
        return Elem<IN>::mfma(__builtin_bit_cast(s16x8, a.h[0]), __builtin_bit_cast(s16x8, b.h[0]), c);
    }
}

// The workgroup's tile (tile row, tile column).
__device__ __forceinline__ void raster_tile(int ntm, int ntn, int& tm, int& tn)
{
    const int t = __builtin_amdgcn_readfirstlane(tile_schedule(ntm * ntn, (int)gridDim.x, (int)blockIdx.x, 0));
    const int per_group = T_GROUP_M * ntn;
    const int group = t / per_group, in_group = t - group * per_group;
    const int first = group * T_GROUP_M, rows = min(ntm - first, T_GROUP_M);
    tm = __builtin_amdgcn_readfirstlane(first + in_group % rows);
    tn = __builtin_amdgcn_readfirstlane(in_group / rows);
}

}  // namespace
