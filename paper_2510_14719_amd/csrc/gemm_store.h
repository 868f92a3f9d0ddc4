// Epilogue of the 256 x 256 matrix-product kernels: one wave's block of C, from the accumulators to memory.
#pragma once

#include <type_traits>

#include "gfx950_prims.h"

namespace {

// How C leaves.  Where its rows are whole memory lines it is written through the L2 (store_through), so that its dirty lines do
// not push the operands out of there.  From about a third of the last-level cache on a few such results push each other
// out of that cache: then every other tile goes past the caches, and all of C where it is too large to be found there by its reader.
// Else, and when C is small, ordinary stores: a row segment that ends inside a line is completed by its neighbour's, and only the
// L2 can put the two together.
// Microseconds on MI355X, 16-bit operands, M x N x K, three C in turn, alone and with an elementwise kernel that reads C behind it:
// ordinary / all through / all past the caches / every other tile:
//    1024 x 1024 x 256, 2 MiB       4.1 / 4.1 / 4.2              8.3 / 8.3 / 8.3
//    2048 x 3008 x 512, 12 MiB     12.5 / 11.0 / 11.4           18.2 / 16.8 / 17.7
//    4096 x 4160 x 256, 32 MiB     20.0 / 19.2 / 18.7           32.5 / 31.6 / 32.5
//    8192 x 6144 x 256, 96 MiB       44 / 43 / 41                 88 / 77 / 89
//    8192 x 8192 x 256, 128 MiB      77 / 67 / 57 / 58           118 / 106 / 125 / 116
//    8192 x 8192 x 512, 128 MiB      83 / 85 / 80 / 72           126 / 123 / 138 / 124
//    16384 x 8192 x 256, 256 MiB    123 / 114 / 109              203 / 195 / 225
//    16384 x 16128 x 256, 504 MiB   256 / 251 / 216              458 / 425 / 415
// (the same C again and again, 8192 x 8192 x 256: 53 / 53 / 57 / 56 and 91 / 92 / 99 / 99, x 512: 77 / 72 / 81 / 71 and 114 / 111 / 122 / 116).
// Rows that are not whole lines:
//    1000 x 777 x 512               4.7 / 5.2 / 5.0              8.2 / 8.4 / 8.4
//    4096 x 4090 x 256               17 / 23 / 19                 29 / 35 / 32
//    8191 x 8191 x 256               77 / 95 / 130               118 / 123 / 129
//    16384 x 16383 x 256            284 / 374 / 475              483 / 565 / 612
enum class Stores { ORDINARY, THROUGH, PAST };
constexpr long long LAST_LEVEL_CACHE = 256ll << 20;
// (uniform over the workgroup, which stores one tile)
__device__ __forceinline__ Stores stores_of(const uint16_t* C, int M, int N)
{
    const long long bytes = 2ll * M * N;
    if ((N & 63) != 0 || (reinterpret_cast<uintptr_t>(C) & 127) != 0 || bytes <= SMALL_RESULT) return Stores::ORDINARY;
    if (bytes <= LAST_LEVEL_CACHE / 8 * 3) return Stores::THROUGH;
    return bytes <= LAST_LEVEL_CACHE / 2 && ((blockIdx.x >> 3) & 1) != 0 ? Stores::THROUGH : Stores::PAST;   // (workgroups go to the eight XCDs in turn)
}
// f(the way as a compile-time constant)
template <typename F>
__device__ __forceinline__ void with_stores(Stores how, F f)
{
    if (how == Stores::ORDINARY) f(std::integral_constant<Stores, Stores::ORDINARY>{});
    else if (how == Stores::THROUGH) f(std::integral_constant<Stores, Stores::THROUGH>{});
    else f(std::integral_constant<Stores, Stores::PAST>{});
}

// Eight elements of a row of C, of which the first `left` exist.  Rows of C are aligned to the element only, which the
// memory path of gfx950 allows for stores of any width: unaligned rows cost a second line at most (8191 x 8191 x 512, fp16:
// 90 us, with stores of single elements 107; 8192 x 8192 x 512: 85).
typedef u32x4 u32x4_any __attribute__((aligned(2)));
template <Stores HOW>
__device__ __forceinline__ void store_chunk(uint16_t* dst, u32x4 w, int left)
{
    if constexpr (HOW != Stores::ORDINARY) {    // N is a multiple of 64: a chunk exists wholly or not at all
        if (left <= 0) return;
        if (HOW == Stores::THROUGH) store_through(dst, w);
        else __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(dst));
    } else if (left >= 8) {
        *reinterpret_cast<u32x4_any*>(dst) = w;
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
template <Stores HOW, int CH>
__device__ __forceinline__ void store_staged_rows(char* st, uint16_t* C, int M, int N, int m1, int n0, int lane)
{
    asm volatile("" ::: "memory");              // (another lane's elements are read: keep the order of the LDS accesses)
    const int c = lane % CH, n = n0 + c * 8;
#pragma unroll
    for (int p = 0; p < CH / 2; ++p) {
        const int row = (p * 64 + lane) / CH;
        const u32x4 w = *reinterpret_cast<const u32x4*>(staged_chunk<CH>(st, row, c));
        if (m1 + row < M) store_chunk<HOW>(C + (size_t)(m1 + row) * N + n, w, N - n);
    }
    asm volatile("" ::: "memory");
}

template <typename E, Stores HOW, int NB>
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
        store_staged_rows<HOW, NB * 4>(st, C, M, N, m0 + mb * 32, n0, lane);
    }
}

// The same for a 128 x 128 block held as 16 x 16 blocks acc[nb][mb] (lane: row lane % 16, four n from 4 (lane / 16) on).
template <typename E, Stores HOW>
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
        if (mb & 1) store_staged_rows<HOW, 16>(st, C, M, N, m0 + (mb - 1) * 16, n0, lane);
    }
}

// The block in the way that suits this C.
template <typename E, typename Acc>
__device__ __forceinline__ void store_wave_block_of(char* st, const Acc& acc, uint16_t* C, int M, int N, int m0, int n0, int lane)
{
    with_stores(stores_of(C, M, N), [&](auto how) __attribute__((always_inline)) {
        store_wave_block<E, decltype(how)::value>(st, acc, C, M, N, m0, n0, lane);
    });
}

}  // namespace
