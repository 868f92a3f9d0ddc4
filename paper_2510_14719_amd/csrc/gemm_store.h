// Epilogue of the 256 x 256 matrix-product kernels: one wave's block of C, from the accumulators to memory.
#pragma once

#include "gfx950_prims.h"

namespace {

// The block is 128 (m) x 32 NB (n); acc[nb][mb] holds, transposed, its 32 x 32 blocks: a lane has one row m and per register
// quad four consecutive n.  Stored straight from the registers an instruction touches 32 rows with 16 bytes each, and the
// stores of a tile (128 KiB) take longer than 256 bytes per row of K do.  So 32 rows at a time go through `st`, 2 NB KiB of the
// LDS that only this wave uses (no barrier: the LDS accesses of a wave complete in order), and leave as segments of
// 32 NB columns: 16 bytes per lane, 8 where rows of C are only 8-byte aligned, or single elements side by side.
// The 16-byte chunks of a row are stored permuted, so that the writes and the wide reads cover all banks.
// Microseconds before and after, M = N = 8192 on MI355X: fp16, K = 1024: 152 -> 132, K = 8192: 862 -> 839; E4M3, K = 8192:
// 410 -> 374; M = N = 8191 (single elements), K = 512: fp16 225 -> 109.
template <typename E, int NB>
__device__ __forceinline__ void store_wave_block(char* st, const f32x16 (&acc)[NB][4], uint16_t* C, int M, int N, int m0, int n0, int lane)
{
    constexpr int CH = NB * 4, RPB = 16 / CH;                    // 16-byte chunks per staged row, rows per 256 bytes
    const int lr = lane & 31, g = lane >> 5;
    const bool v16 = (N & 7) == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0;
    const bool v8 = (N & 3) == 0 && (reinterpret_cast<uintptr_t>(C) & 7) == 0;
    auto chunk = [&](int row, int c) __attribute__((always_inline)) -> char* {
        return st + row * (CH * 16) + ((c ^ ((row / RPB) & (CH - 1))) * 16);
    };
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
        asm volatile("" ::: "memory");          // (another lane's elements are read: keep the order of the LDS accesses)
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const f32x16& x = acc[c / 4][mb];
            u32x2 w;
            w[0] = E::pack2(x[c % 4 * 4 + 0], x[c % 4 * 4 + 1]);
            w[1] = E::pack2(x[c % 4 * 4 + 2], x[c % 4 * 4 + 3]);
            *reinterpret_cast<u32x2*>(chunk(lr, c) + g * 8) = w;
        }
        asm volatile("" ::: "memory");
        const int m1 = m0 + mb * 32;
        if (v16) {
            const int c = lane % CH, n = n0 + c * 8;
#pragma unroll
            for (int p = 0; p < CH / 2; ++p) {
                const int row = (p * 64 + lane) / CH;
                const u32x4 w = *reinterpret_cast<const u32x4*>(chunk(row, c));
                if (m1 + row < M && n < N) *reinterpret_cast<u32x4*>(C + (size_t)(m1 + row) * N + n) = w;
            }
        } else if (v8) {
            const int h = lane % (2 * CH), n = n0 + h * 4;
#pragma unroll 4
            for (int p = 0; p < CH; ++p) {
                const int row = (p * 64 + lane) / (2 * CH);
                const u32x2 w = *reinterpret_cast<const u32x2*>(chunk(row, h / 2) + (h & 1) * 8);
                if (m1 + row < M && n < N) *reinterpret_cast<u32x2*>(C + (size_t)(m1 + row) * N + n) = w;
            }
        } else {
#pragma unroll 4
            for (int p = 0; p < 4 * CH; ++p) {
                const int e = p * 64 + lane, row = e / (8 * CH), col = e % (8 * CH);
                const uint16_t w = *reinterpret_cast<const uint16_t*>(chunk(row, col / 8) + (col & 7) * 2);
                if (m1 + row < M && n0 + col < N) C[(size_t)(m1 + row) * N + n0 + col] = w;
            }
        }
    }
}

}  // namespace
