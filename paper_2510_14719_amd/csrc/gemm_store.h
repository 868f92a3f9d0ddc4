// Epilogue of the 256 x 256 matrix-product kernels: one wave's block of C, from the accumulators to memory.
#pragma once

#include "gfx950_prims.h"

namespace {

// Eight elements of a row of C, of which the first `left` exist.  Rows of C are aligned to the element only, which the
// memory path of gfx950 allows for stores of any width: unaligned rows cost a second line at most (8191 x 8191 x 512, fp16:
// 90 us, with stores of single elements 107; 8192 x 8192 x 512: 85).  The stores are non-temporal: C is written once and not
// read here, and its dirty lines otherwise push the operands out of the L2 (8192 x 8192, bf16, three sets of buffers in
// turn: K = 256 77 -> 56 us, K = 1024 126 -> 119; 4096 x 4096 x 512 with the consumer of C behind it: 36 -> 33.5).  What it
// costs: a C of 128 MiB that is written again and again by short products no longer stays in the last-level cache (K = 256,
// one C: 51 -> 56; with a consumer 87 -> 97).
typedef u32x4 u32x4_any __attribute__((aligned(2)));
__device__ __forceinline__ void store_chunk(uint16_t* dst, u32x4 w, int left)
{
    if (left >= 8) {
        __builtin_nontemporal_store(w, reinterpret_cast<u32x4_any*>(dst));
    } else {
#pragma unroll
        for (int e = 0; e < 7; ++e)
            if (e < left) dst[e] = (uint16_t)(w[e >> 1] >> ((e & 1) * 16));
    }
}

// The block is 128 (m) x 32 NB (n); acc[nb][mb] holds, transposed, its 32 x 32 blocks: a lane has one row m and per register
// quad four consecutive n.  Stored straight from the registers an instruction touches 32 rows with 16 bytes each, and the
// stores of a tile (128 KiB) take longer than 256 bytes per row of K do.  So 32 rows at a time go through `st`, 2 NB KiB of the
// LDS that only this wave uses (no barrier: the LDS accesses of a wave complete in order), and leave as segments of
// 32 NB columns, 16 bytes per lane.
// The 16-byte chunks of a row are stored permuted, so that the writes and the wide reads cover all banks.
// Microseconds before and after, M = N = 8192 on MI355X: fp16, K = 1024: 152 -> 132, K = 8192: 862 -> 839; E4M3, K = 8192:
// 410 -> 374; M = N = 8191, K = 512: fp16 225 -> 94.
template <int CH>       // 16-byte chunks per staged row
__device__ __forceinline__ char* staged_chunk(char* st, int row, int c)
{
    constexpr int RPB = 16 / CH;                // rows per 256 bytes
    return st + row * (CH * 16) + ((c ^ ((row / RPB) & (CH - 1))) * 16);
}

// The 32 staged rows from row m1 of C on, columns from n0 on.
template <int CH>
__device__ __forceinline__ void store_staged_rows(char* st, uint16_t* C, int M, int N, int m1, int n0, int lane)
{
    asm volatile("" ::: "memory");              // (another lane's elements are read: keep the order of the LDS accesses)
    const int c = lane % CH, n = n0 + c * 8;
#pragma unroll
    for (int p = 0; p < CH / 2; ++p) {
        const int row = (p * 64 + lane) / CH;
        const u32x4 w = *reinterpret_cast<const u32x4*>(staged_chunk<CH>(st, row, c));
        if (m1 + row < M) store_chunk(C + (size_t)(m1 + row) * N + n, w, N - n);
    }
    asm volatile("" ::: "memory");
}

template <typename E, int NB>
__device__ __forceinline__ void store_wave_block(char* st, const f32x16 (&acc)[NB][4], uint16_t* C, int M, int N, int m0, int n0, int lane)
{
    const int lr = lane & 31, g = lane >> 5;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
#pragma unroll
        for (int c = 0; c < NB * 4; ++c) {
            const f32x16& x = acc[c / 4][mb];
            u32x2 w;
            w[0] = E::pack2(x[c % 4 * 4 + 0], x[c % 4 * 4 + 1]);
            w[1] = E::pack2(x[c % 4 * 4 + 2], x[c % 4 * 4 + 3]);
            *reinterpret_cast<u32x2*>(staged_chunk<NB * 4>(st, lr, c) + g * 8) = w;
        }
        store_staged_rows<NB * 4>(st, C, M, N, m0 + mb * 32, n0, lane);
    }
}

// The same for a 128 x 128 block held as 16 x 16 blocks acc[nb][mb] (lane: row lane % 16, four n from 4 (lane / 16) on).
template <typename E>
__device__ __forceinline__ void store_wave_block(char* st, const f32x4 (&acc)[8][8], uint16_t* C, int M, int N, int m0, int n0, int lane)
{
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) {
#pragma unroll
        for (int nb = 0; nb < 8; ++nb) {
            const f32x4& x = acc[nb][mb];
            u32x2 w;
            w[0] = E::pack2(x[0], x[1]);
            w[1] = E::pack2(x[2], x[3]);
            *reinterpret_cast<u32x2*>(staged_chunk<16>(st, (mb & 1) * 16 + (lane & 15), nb * 2 + (lane >> 5)) + ((lane >> 4) & 1) * 8) = w;
        }
        if (mb & 1) store_staged_rows<16>(st, C, M, N, m0 + (mb - 1) * 16, n0, lane);
    }
}

}  // namespace
