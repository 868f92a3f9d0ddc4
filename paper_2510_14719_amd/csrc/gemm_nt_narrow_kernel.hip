// NT matrix products with the smallest tiles of C for gfx950 (MI355X), 16-bit and E4M3 operands: the same contract as
// gemm_nt_tile_kernel.hip, in the place of its shape 1 where 64 x 64 tiles are few.
//
// 32 x 32 or 16 x 16 of C per workgroup (T), for products with few 64 x 64 tiles.
//
// What bounds those is one CU's share of the operands: copies reach the LDS at 64 bytes per cycle and CU (16 cycles for the 1 KiB of
// an instruction), 256 cycles for a 128-byte step of a 64 x 64 tile, while its MFMAs take 128; measured 64 x 64 x 16384, one CU:
// 370 cycles a step, and a deeper ring changes nothing.  Smaller tiles read more in all but spread it over more CUs: T = 32 takes half of
// that per step and CU, T = 16 a quarter (43 -> 22 -> 12.5 us; more beside narrow_tile).
//
// A stage is always 16 KiB, 256 (T = 32) or 512 bytes of T rows of A and of B, two copies for each of eight waves.  16-bit
// operands: the stage's eight k-steps (32x32x16 or 16x16x32 MFMA) go one to a wave, whose sums are added in the LDS at the end.
// E4M3 products keep one order of summation, so wave 0 takes all four k-steps (256 cycles, as long as the copies) and the others only
// copy.  Ring of four stages with the protocol of the small-tile kernel: fragments one stage ahead, at barrier j
// stage j has been read and stage j + 1 is complete, and the copies of stage j + 4 go out behind it.  (Eight stages, 128 KiB:
// as fast on long rows, 0.5 us more on short ones.)  A last stage that is not whole copies its missing columns from the first 64
// bytes and leaves out the k-steps beyond the end.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "gemm_launch.h"
#include "gemm_store.h"
#include "gemm_tile_prims.h"
#include "launch_once.h"

namespace {

constexpr int NARROW_STAGES = 4;

template <int IN, int OUT, int T>
__global__ __launch_bounds__(512)
void gemm_nt_narrow_kernel(const char* __restrict__ A, const char* __restrict__ B, uint16_t* __restrict__ C,
                           int M, int N, int row_bytes, int ntm, int ntn)
{
    typedef Elem<OUT> E;
    constexpr bool F8 = IN == 2;
    constexpr int NW = 8, PPW = 2, S = NARROW_STAGES;            // waves, copies of 1 KiB per wave and stage, stages
    constexpr int ROW = 8192 / T, STAGE_BYTES = 2 * T * ROW;     // bytes of a row per stage: 256 or 512
    constexpr int CPR = ROW / 16, RPP = 64 / CPR;                // 16-byte columns of it, rows per copy
    constexpr int HALVES = F8 ? 2 : 1, KSW = F8 ? 4 : 1;         // 16-byte reads per fragment, k-steps of a stage that a computing wave takes
    constexpr int KBYTES = F8 || T == 16 ? 64 : 32;              // bytes of a row per k-step
    constexpr int QUADS = T / 8 == 4 ? 4 : 1;                    // runs of four n that a lane holds of the result
    constexpr int PART = QUADS * 1024;                           // bytes of one wave's sums
    constexpr int C_STRIDE = T * 2 + 16;
    static_assert(T == 32 || (T == 16 && !F8), "MFMA shapes");
    static_assert(S == 4 && NW * PART + T * C_STRIDE <= S * STAGE_BYTES, "the epilogue reuses the ring");

    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const unsigned lds_base = (unsigned)(size_t)(LDS_AS void*)smem;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int lr = lane & (T - 1), g = lane / T;
    const bool computes = !F8 || wave == 0;

    int tm, tn;
    raster_tile(ntm, ntn, tm, tn);
    const int m0 = tm * T, n0 = tn * T;
    const int nk = (row_bytes + ROW - 1) / ROW, tail = row_bytes - (nk - 1) * ROW;   // stages, bytes of every row in the last one

    // ---- copies: lane L of piece p fetches row RPP p + L / CPR of the stage (A's T rows, then B's), into slot L % CPR: column (L % CPR) ^ (row % 16)
    const char* src[PPW];
    unsigned voff[PPW], voff_tail[PPW];
#pragma unroll
    for (int i = 0; i < PPW; ++i) {
        const int p = wave * PPW + i;
        const bool is_b = p >= 8;
        const int row = (is_b ? p - 8 : p) * RPP + lane / CPR;
        const int col = (lane % CPR) ^ (row & 15);
        src[i] = is_b ? B : A;
        const unsigned start = (unsigned)(is_b ? min(n0 + row, N - 1) : min(m0 + row, M - 1)) * (unsigned)row_bytes;
        voff[i] = start + col * 16;
        voff_tail[i] = start + (col * 16 < tail ? col : col & 3) * 16;           // (a row's last 64 bytes or more exist; the others are not used)
    }
    auto issue = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PPW; ++i)
            dma16(src[i] + (size_t)s * ROW, s == nk - 1 ? voff_tail[i] : voff[i], lds_base + (s % S) * STAGE_BYTES + (wave * PPW + i) * 1024);
    };

    struct Frags { TileFrag<IN> am[KSW], bn[KSW]; };
    auto read_stage = [&](Frags& f, int s) __attribute__((always_inline)) {
        if (!computes) return;
        const char* st = smem + (s % S) * STAGE_BYTES + lr * ROW;
#pragma unroll
        for (int k = 0; k < KSW; ++k)
#pragma unroll
            for (int h = 0; h < HALVES; ++h) {
                const int col = F8 ? k * 4 + g * 2 + h : wave * (KBYTES / 16) + g;
                const int off = (col ^ (lr & 15)) * 16;
                f.am[k].h[h] = *reinterpret_cast<const i32x4*>(st + off);
                f.bn[k].h[h] = *reinterpret_cast<const i32x4*>(st + T * ROW + off);
            }
    };
    typename std::conditional<T == 32, f32x16, f32x4>::type acc = {};
    // own copies of every stage but the last `out` ones issued are complete
    auto wait_out = [&](int out) __attribute__((always_inline)) {
        if (out == 3) wait_vmcnt<3 * PPW>();
        else if (out == 2) wait_vmcnt<2 * PPW>();
        else if (out == 1) wait_vmcnt<1 * PPW>();
        else wait_vmcnt<0>();
    };
#pragma unroll
    for (int s = 0; s < S; ++s)
        if (s < nk) issue(s);
    wait_out(min(S - 1, nk - 1));
    ring_barrier();
    Frags X, Y;
    read_stage(X, 0);
    // Stage j: at the barrier everyone has read it and its successor is complete.
    auto stage = [&](int j, const Frags& cur, Frags& nxt, auto steady_tag) __attribute__((always_inline)) {
        constexpr bool STEADY = decltype(steady_tag)::value;             // stage j + S exists
        if (STEADY) wait_vmcnt<(S - 2) * PPW>(); else wait_out(min(S - 2, nk - 2 - j));
        __builtin_amdgcn_s_waitcnt(0xC07F);     // lgkmcnt(0)
        ring_barrier();
        if (STEADY || j + 1 < nk) read_stage(nxt, j + 1);
        if (STEADY || j + S < nk) issue(j + S);
        if (computes) {
#pragma unroll
            for (int k = 0; k < KSW; ++k)
                if (STEADY || j < nk - 1 || (F8 ? k : wave) * KBYTES < tail) {
                    if constexpr (T == 32) acc = tile_mfma<IN>(cur.bn[k], cur.am[k], acc);
                    else acc = Elem<IN>::mfma16(__builtin_bit_cast(s16x8, cur.bn[k].h[0]), __builtin_bit_cast(s16x8, cur.am[k].h[0]), acc);
                }
        }
    };
    int j = 0;
    for (; j + 1 + S < nk; j += 2) {
        stage(j, X, Y, std::true_type());
        stage(j + 1, Y, X, std::true_type());
    }
    for (; j + 1 < nk; j += 2) {
        stage(j, X, Y, std::false_type());
        stage(j + 1, Y, X, std::false_type());
    }
    if (j < nk) stage(j, X, Y, std::false_type());

    // ---- the waves' sums added up (16-bit operands), then out through the LDS as row segments
    ring_barrier();                             // nobody reads the ring any more
    char* const cst = smem + NW * PART;
    auto stage_result = [&](int t, const f32x4& x) __attribute__((always_inline)) {
        const u32x2 w = {E::pack2(x[0], x[1]), E::pack2(x[2], x[3])};
        *reinterpret_cast<u32x2*>(cst + lr * C_STRIDE + (t * 8 + g * 4) * 2) = w;
    };
    if constexpr (F8) {
        if (wave == 0) {
#pragma unroll
            for (int t = 0; t < QUADS; ++t) stage_result(t, f32x4{acc[t * 4], acc[t * 4 + 1], acc[t * 4 + 2], acc[t * 4 + 3]});
        }
    } else {
#pragma unroll
        for (int t = 0; t < QUADS; ++t)
            *reinterpret_cast<f32x4*>(smem + wave * PART + t * 1024 + lane * 16) = f32x4{acc[t * 4], acc[t * 4 + 1], acc[t * 4 + 2], acc[t * 4 + 3]};
        __syncthreads();
        if (wave < QUADS) {
            f32x4 x = *reinterpret_cast<const f32x4*>(smem + wave * 1024 + lane * 16);
#pragma unroll
            for (int w = 1; w < NW; ++w) x += *reinterpret_cast<const f32x4*>(smem + w * PART + wave * 1024 + lane * 16);
            stage_result(wave, x);
        }
    }
    __syncthreads();
    const int r = threadIdx.x / (T / 8), c = threadIdx.x % (T / 8) * 8;
    if (r < min(T, M - m0))
        store_chunk<Stores::ORDINARY>(C + (size_t)(m0 + r) * N + n0 + c, *reinterpret_cast<const u32x4*>(cst + r * C_STRIDE + c * 2), N - n0 - c);
}

template <int IN, int OUT, int T>
int launch_narrow(const GemmLaunchArgs& a)
{
    constexpr int smem = NARROW_STAGES * 16384;
    auto kern = gemm_nt_narrow_kernel<IN, OUT, T>;
    static PerDeviceOnce once;                  // the attribute belongs to the (kernel, device) pair
    if (once.prepare(reinterpret_cast<const void*>(kern), smem) < 0) return -1;
    const char* A = (const char*)a.a;
    const char* B = (const char*)a.b;
    uint16_t* C = (uint16_t*)a.c;
    int M = a.M, N = a.N, row_bytes = a.K * (IN == 2 ? 1 : 2);
    int ntm = (M + T - 1) / T, ntn = (N + T - 1) / T;
    void* args[] = {&A, &B, &C, &M, &N, &row_bytes, &ntm, &ntn};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3((unsigned)(ntm * ntn)), dim3(512), args, smem, (hipStream_t)a.stream);
    return e == hipSuccess ? 0 : -1;
}

template <int IN, int OUT>
int launch_narrow_of(const GemmLaunchArgs& a, int tile)
{
    if constexpr (IN != 2) {
        if (tile == 16) return launch_narrow<IN, OUT, 16>(a);
    }
    return tile == 32 ? launch_narrow<IN, OUT, 32>(a) : -1;
}

}  // namespace

int gemm_narrow_launch(const GemmLaunchArgs& a, int in_type, int tile)
{
    if (in_type == 0) return launch_narrow_of<0, 0>(a, tile);
    if (in_type == 1) return launch_narrow_of<1, 1>(a, tile);
    return a.dtype == 0 ? launch_narrow_of<2, 0>(a, tile) : launch_narrow_of<2, 1>(a, tile);
}

// Which tiles of C a product takes in the place of shape 1: T of gemm_nt_narrow_kernel, or 0 for the 64 x 64 ones.  The smaller ones while they fit the chip in one round,
// however long the rows are; 32 x 32 also two to a CU where the rows are long, for 16-bit operands (for E4M3 one wave does the
// MFMAs, and two such workgroups lose).  us, 64 x 64 / 32 x 32 / 16 x 16, M x N x K:
//    bf16   64 x 64 x 64        4.05 / 3.87 / 3.91         64 x 64 x 16384     43.2 / 22.1 / 12.5
//           256 x 256 x 320     4.12 / 3.86 / 3.91         256 x 256 x 4096    11.1 / 8.3 / 5.1
//           320 x 320 x 1024    5.3 / 3.9 / 4.1            512 x 512 x 4096    14.2 / 8.5 / 13.3
//           704 x 640 x 1536    7.1 / 6.6; x 192 4.07 / 4.05; x 8192 24.5 / 22.6     1024 x 512 x 1536  6.4 / 6.6; x 3072 11.7 / 10.9
//           768 x 768 x 8192    24.6 / 32.0
//    E4M3   64 x 64 x 64        4.08 / 3.82                512 x 512 x 512     3.55 / 3.27; x 16384 23.8 / 16.6
//           640 x 512 x 2048    5.3 / 7.8
static constexpr long long NARROW_LONG_ROW = 4096;     // bytes
int gemm_narrow_tile(int M, int N, long long row_bytes, bool fp8)
{
    auto tiles = [&](int t) { return ((M + t - 1LL) / t) * ((N + t - 1LL) / t); };
    if (!fp8 && tiles(16) <= CHIP_CUS) return 16;
    if (tiles(32) <= CHIP_CUS || (!fp8 && row_bytes >= NARROW_LONG_ROW && tiles(32) <= 2 * CHIP_CUS)) return 32;
    return 0;
}
