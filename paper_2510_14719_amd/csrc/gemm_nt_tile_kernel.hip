// NT matrix products with small tiles of C for gfx950 (MI355X): the same contract as gemm_nt_kernel.hip (16-bit operands)
// and gemm_nt_fp8_kernel.hip (E4M3 operands, 16-bit result), for shapes whose 256 x 256 tiles leave compute units idle
// or whose K is too short to hide the prologue and the epilogue of one big workgroup per compute unit.
//
// One kernel serves every element type, because everything but the MFMA is about bytes: a stage of the LDS ring
// holds 128 bytes (one memory line) of every row of the A tile and of the B tile, so a copy instruction moves 8 whole
// lines, and the fragments of a stage are 8 columns of 16 bytes per row: four k-steps of the 32x32x16 MFMA (16-bit) or
// two of the 32x32x64 MFMA (E4M3).  A row is a multiple of 64 bytes (the contract's K step); in a last stage that is
// only half filled the copies fetch the first half twice and the k-steps of the second half are left out.
//
// Waves: WM x WN of them split the tile, and WK of them split the k-steps of a stage (their accumulators are added
// in the LDS before the epilogue): with one or two workgroups per CU this is what keeps two waves on every SIMD
// when the tile is small.
//
// Ring of S stages.  The fragments of stage j are read into registers during tile j - 1, so at barrier j the slots of
// all stages <= j are free (every wave waits for its reads before the barrier) and stage j + 1 is complete (every
// wave waits for its own copies of it); the copies of stage j + S go out during tile j.
//
// LDS: row r of a stage at r * 128 bytes, its 16-byte column c at slot c ^ ((r / 2) % 8): the 16 rows that one pass of a
// fragment read touches cover all 64 banks.
//
// Epilogue: the product is computed transposed (a lane holds one row m of C and runs of four n).  The 16-bit results go
// through the LDS and leave as whole row segments of the tile (16 bytes per lane): stored straight from the registers, an instruction would
// touch 32 rows with 16 bytes each.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "gemm_launch.h"
#include "gemm_store.h"
#include "gemm_tile_prims.h"
#include "gfx950_prims.h"
#include "launch_once.h"

namespace {

// IN: 0 fp16, 1 bf16, 2 E4M3.  OUT: 0 fp16, 1 bf16.  OCC: workgroups per CU the registers must allow.
template <int IN, int OUT, int BM, int BN, int WM, int WN, int WK, int S, int OCC>
__global__ __launch_bounds__(WM * WN * WK * 64, OCC * WM * WN * WK / 4)
void gemm_nt_tile_kernel(const char* __restrict__ A, const char* __restrict__ B, uint16_t* __restrict__ C,
                         int M, int N, int row_bytes, int ntm, int ntn)
{
    typedef Elem<OUT> E;
    constexpr int NW = WM * WN * WK;
    constexpr int MB = BM / (32 * WM), NB = BN / (32 * WN);      // 32 x 32 blocks of C per wave
    constexpr int KSTEPS = IN == 2 ? 2 : 4;                      // MFMA k-steps per stage
    constexpr int KSW = KSTEPS / WK;                             // ... per wave
    constexpr int HALVES = IN == 2 ? 2 : 1;                      // 16-byte reads per fragment
    constexpr int STAGE_BYTES = (BM + BN) * 128;
    constexpr int PIECES = (BM + BN) / 8, PPW = PIECES / NW;     // 1 KiB copies per stage, per wave
    static_assert(PIECES % NW == 0 && KSTEPS % WK == 0 && (S - 1) * PPW <= 63, "shape of the workgroup");
    constexpr int RED_BYTES = WK == 2 ? NW * MB * NB * 8 * 256 : 0;   // half of every wave's accumulators
    constexpr int C_STRIDE = BN * 2 + 16;                        // bytes per row of the staged result
    static_assert(WK <= 2 && RED_BYTES + BM * C_STRIDE <= S * STAGE_BYTES, "the epilogue reuses the ring");

    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const unsigned lds_base = (unsigned)(size_t)(LDS_AS void*)smem;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int lr = lane & 31, g = lane >> 5;
    const int wm = wave % WM, wn = (wave / WM) % WN, wk = wave / (WM * WN);

    int tm, tn;
    raster_tile(ntm, ntn, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int nk = (row_bytes + 127) >> 7, nfull = row_bytes >> 7;   // stages, and those of them that are whole

    // ---- copies.  Lane L of piece p fetches row 8 p + L / 8 of the stage, into slot L % 8: column (L % 8) ^ swizzle.
    // Tiles that overhang the matrix clamp their rows (the surplus rows are never stored).
    const char* src[PPW];
    unsigned voff[PPW], half_off[PPW];
#pragma unroll
    for (int i = 0; i < PPW; ++i) {
        const int p = wave * PPW + i;
        const bool is_b = p >= BM / 8;
        const int row = (is_b ? p - BM / 8 : p) * 8 + (lane >> 3);
        const int col = (lane & 7) ^ ((row >> 1) & 7);
        src[i] = is_b ? B : A;
        voff[i] = (unsigned)(is_b ? min(n0 + row, N - 1) : min(m0 + row, M - 1)) * (unsigned)row_bytes + col * 16;
        half_off[i] = (col & 4) * 16;
    }
    auto issue_piece = [&](int s, int i) __attribute__((always_inline)) {          // s < nfull
        dma16(src[i] + (size_t)s * 128, voff[i], lds_base + (s % S) * STAGE_BYTES + (wave * PPW + i) * 1024);
    };
    auto issue_piece_any = [&](int s, int i) __attribute__((always_inline)) {      // s < nk
        dma16(src[i] + (size_t)s * 128, s < nfull ? voff[i] : voff[i] - half_off[i],
              lds_base + (s % S) * STAGE_BYTES + (wave * PPW + i) * 1024);
    };

    // ---- fragments
    int frag_off[KSW][HALVES];
#pragma unroll
    for (int k = 0; k < KSW; ++k)
#pragma unroll
        for (int h = 0; h < HALVES; ++h) {
            const int ks = wk * KSW + k;
            const int col = IN == 2 ? ks * 4 + g * 2 + h : ks * 2 + g;
            frag_off[k][h] = lr * 128 + ((col ^ ((lr >> 1) & 7)) * 16);
        }
    struct StageFrags { TileFrag<IN> am[KSW][MB], bn[KSW][NB]; };
    constexpr int READS = KSW * (MB + NB) * HALVES, MFMAS = KSW * MB * NB;
    auto read_one = [&](StageFrags& f, int s, int i) __attribute__((always_inline)) {   // in the order of use
        const int k = i / ((MB + NB) * HALVES), r = (i / HALVES) % (MB + NB), h = i % HALVES;
        const char* st = smem + (s % S) * STAGE_BYTES + frag_off[k][h];
        if (r < NB) f.bn[k][r].h[h] = *reinterpret_cast<const i32x4*>(st + (BM + (wn * NB + r) * 32) * 128);
        else f.am[k][r - NB].h[h] = *reinterpret_cast<const i32x4*>(st + (wm * MB + r - NB) * 32 * 128);
    };

    f32x16 acc[NB][MB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = f32x16(0.f);

    // own copies of every stage but the last `out` ones issued are complete
    auto wait_out = [&](int out) __attribute__((always_inline)) {
        if (S > 3 && out == 2) wait_vmcnt<(S > 3 ? 2 : 0) * PPW>();
        else if (S > 2 && out == 1) wait_vmcnt<(S > 2 ? 1 : 0) * PPW>();
        else wait_vmcnt<0>();
    };
    static_assert(S >= 2 && S <= 4, "wait_out lists the counts");

    // ---- prologue: the whole ring in flight, stage 0 complete for everyone, its fragments requested
#pragma unroll
    for (int s = 0; s < S; ++s)
        if (s < nk) {
#pragma unroll
            for (int i = 0; i < PPW; ++i) issue_piece_any(s, i);
        }
    if (nk >= S) wait_vmcnt<(S - 1) * PPW>(); else wait_out(nk - 1);
    ring_barrier();
    StageFrags X, Y;
#pragma unroll
    for (int i = 0; i < READS; ++i) read_one(X, 0, i);

    // Tile j: the MFMAs on the fragments in `cur`, behind them the requests for the next tile's and the copies
    // of stage j + S.  STEADY: that stage exists and is whole.
    auto tile = [&](int j, const StageFrags& cur, StageFrags& nxt, auto steady_tag) __attribute__((always_inline)) {
        constexpr bool STEADY = decltype(steady_tag)::value;
        if (STEADY) wait_vmcnt<(S - 2) * PPW>(); else wait_out(min(S - 2, nk - 2 - j));
        __builtin_amdgcn_s_waitcnt(0xC07F);     // lgkmcnt(0): this wave's reads of stage j are complete
        ring_barrier();
        const bool half = !STEADY && j >= nfull;                       // a half-filled last stage
        const bool copy = STEADY || j + S < nk, next = STEADY || j + 1 < nk;
#pragma unroll
        for (int q = 0; q < MFMAS; ++q) {
            const int k = q / (MB * NB), mb = (q / NB) % MB, nb = q % NB;
            if (STEADY || !half || wk * KSW + k < KSTEPS / 2)
                acc[nb][mb] = tile_mfma<IN>(cur.bn[k][nb], cur.am[k][mb], acc[nb][mb]);
            __builtin_amdgcn_sched_barrier(0);
            if (next) {
#pragma unroll
                for (int i = q * READS / MFMAS; i < (q + 1) * READS / MFMAS; ++i) read_one(nxt, j + 1, i);
            }
            if (copy) {
#pragma unroll
                for (int i = q * PPW / MFMAS; i < (q + 1) * PPW / MFMAS; ++i) {
                    if (STEADY) issue_piece(j + S, i); else issue_piece_any(j + S, i);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    {
        typedef std::integral_constant<bool, true> steady_t;
        typedef std::integral_constant<bool, false> draining_t;
        int j = 0;
        if (j + 1 + S < nfull) {
            do {
                tile(j, X, Y, steady_t());
                tile(j + 1, Y, X, steady_t());
                j += 2;
            } while (j + 1 + S < nfull);
        }
        if (j + 1 < nk) {
            do {
                tile(j, X, Y, draining_t());
                tile(j + 1, Y, X, draining_t());
                j += 2;
            } while (j + 1 < nk);
        }
        if (j < nk) tile(j, X, Y, draining_t());
    }

    // ---- the waves that split k exchange halves of their accumulators: quads 0, 1 of a block end up with wk = 0, quads
    // 2, 3 with wk = 1.  (All copies have landed: the last tiles waited for everything.)
    char* const cst = smem + RED_BYTES;
    if constexpr (WK == 2) {
        ring_barrier();           // nobody reads the ring any more
        auto red = [&](int w, int blk, int t) __attribute__((always_inline)) -> f32x4* {
            return reinterpret_cast<f32x4*>(smem + ((w * MB * NB + blk) * 2 + t) * 1024 + lane * 16);
        };
#pragma unroll
        for (int blk = 0; blk < MB * NB; ++blk)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float lo = acc[blk % NB][blk / NB][t * 4 + e], hi = acc[blk % NB][blk / NB][8 + t * 4 + e];
                    v[e] = wk == 0 ? hi : lo;
                }
                *red(wave, blk, t) = v;
            }
        __syncthreads();
#pragma unroll
        for (int blk = 0; blk < MB * NB; ++blk)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const f32x4 v = *red(wave ^ (WM * WN), blk, t);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float lo = acc[blk % NB][blk / NB][t * 4 + e], hi = acc[blk % NB][blk / NB][8 + t * 4 + e];
                    acc[blk % NB][blk / NB][t * 4 + e] = (wk == 0 ? lo : hi) + v[e];
                }
            }
    } else {
        ring_barrier();
    }

    // ---- results to the LDS, then out as row segments
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int t = 0; t < 4 / WK; ++t) {
                u32x2 w;
                w[0] = E::pack2(acc[nb][mb][t * 4 + 0], acc[nb][mb][t * 4 + 1]);
                w[1] = E::pack2(acc[nb][mb][t * 4 + 2], acc[nb][mb][t * 4 + 3]);
                const int row = (wm * MB + mb) * 32 + lr, col = (wn * NB + nb) * 32 + (wk * 2 + t) * 8 + g * 4;
                *reinterpret_cast<u32x2*>(cst + row * C_STRIDE + col * 2) = w;
            }
    __syncthreads();
    const int rows = min(BM, M - m0), cols = min(BN, N - n0);
    constexpr int CPR = BN / 8, RPI = NW * 64 / CPR;             // 16-byte chunks per row, rows per round
    const int c = (threadIdx.x % CPR) * 8;
    with_stores(stores_of(C, M, N), [&](auto how) __attribute__((always_inline)) {
#pragma unroll
        for (int r0 = 0; r0 < BM; r0 += RPI) {
            const int r = r0 + threadIdx.x / CPR;
            if (r < rows)
                store_chunk<decltype(how)::value>(C + (size_t)(m0 + r) * N + n0 + c, *reinterpret_cast<const u32x4*>(cst + r * C_STRIDE + c * 2), cols - c);
        }
    });
}

template <int IN, int OUT, int BM, int BN, int WM, int WN, int WK, int S, int OCC>
int launch_tile(const GemmLaunchArgs& a)
{
    constexpr int smem = S * (BM + BN) * 128;
    auto kern = gemm_nt_tile_kernel<IN, OUT, BM, BN, WM, WN, WK, S, OCC>;
    static PerDeviceOnce once;                  // the attribute belongs to the (kernel, device) pair
    if (once.prepare(reinterpret_cast<const void*>(kern), smem) < 0) return -1;
    const char* A = (const char*)a.a;
    const char* B = (const char*)a.b;
    uint16_t* C = (uint16_t*)a.c;
    int M = a.M, N = a.N, row_bytes = a.K * (IN == 2 ? 1 : 2);
    int ntm = (M + BM - 1) / BM, ntn = (N + BN - 1) / BN;
    void* args[] = {&A, &B, &C, &M, &N, &row_bytes, &ntm, &ntn};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3((unsigned)(ntm * ntn)), dim3(WM * WN * WK * 64),
                                         args, smem, (hipStream_t)a.stream);
    return e == hipSuccess ? 0 : -1;
}

// ---- 256 x 256 of C per workgroup, for products that fill the chip with such tiles.  Four waves, one per SIMD, 128 x 128 each (the
// split that reads least from the LDS: 128 KiB per 128-byte step along K, next to 64 KiB of copies written; the MFMAs of
// a step take 2048 cycles), accumulators in the AGPRs.
//
// What bounds a full chip here is power: on operands of zeros a 8192 x 8192 x 8192 product takes two thirds of the time.
// 16-bit operands therefore take the 16 x 16 x 32 MFMA: per flop it reads its operands twice as often as the 32 x 32 x 16 one
// but moves half as much of the fp32 accumulators (the same product, bf16: 761 -> 697 us, although zeros take longer, 503 ->
// 535).  E4M3 operands keep 32 x 32 x 64, where both come out alike and 16 x 16 fragments would not fit the registers.
//
// A step's rows are whole 128-byte lines (layout of the small-tile kernel), so one copy instruction asks the L2 for 8 lines
// and copies can be spread evenly: one per 128 cycles of MFMAs.  (Issued in bursts they fill the CU's
// address path, 16 cycles per copy, and the waves that queue for it cannot issue their MFMAs.)
//
// Ring of five 32 KiB slots for the sequence A_0 B_0 A_1 B_1 A_2 ...: A_j and B_j are the operand tiles of step j.
// Fragments are read one k-step ahead, so step j has been read completely when its last k-step starts.  There is the one
// barrier of a step: behind it the slots of A_j and B_j are free and step j + 1 is complete; B_{j+2} and then A_{j+3} are
// copied into the two slots until the next such point, which waits for B_{j+2} and leaves A_{j+3} in flight.
template <int IN, int OUT>
__global__ __launch_bounds__(256, 1)
void gemm_nt_wide_kernel(const char* __restrict__ A, const char* __restrict__ B, uint16_t* __restrict__ C,
                         int M, int N, int row_bytes, int ntm, int ntn)
{
    typedef Elem<OUT> E;
    constexpr bool B16 = IN != 2;               // 16 x 16 x 32 MFMAs; E4M3: 32 x 32 x 64
    constexpr int KSTEPS = 2, HALVES = IN == 2 ? 2 : 1;          // a k-step is 64 bytes of every row
    constexpr int BS = B16 ? 16 : 32, NB = 128 / BS;             // block size, blocks of each operand per wave
    constexpr int SLOT = 256 * 128, SLOTS = 5;
    constexpr int PPW = 8;                      // copies per wave and operand tile
    constexpr int READS = 2 * NB * HALVES;      // fragment reads per k-step
    constexpr int READ_EVERY = B16 ? 2 : 1;     // MFMAs per read
    constexpr int SPAN = NB * NB * KSTEPS;      // MFMAs between two barriers
    constexpr int COPY_EVERY = SPAN / (2 * PPW);

    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const unsigned lds_base = (unsigned)(size_t)(LDS_AS void*)smem;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int wm = wave & 1, wn = wave >> 1;

    int tm, tn;
    raster_tile(ntm, ntn, tm, tn);
    const int m0 = tm * 256, n0 = tn * 256;
    const int nk = (row_bytes + 127) >> 7, nfull = row_bytes >> 7;   // steps, and those of them that are whole

    // ---- copies: lane L of piece p fetches row 8 p + L / 8 into slot L % 8 of the row (see gemm_nt_tile_kernel)
    unsigned a_off[PPW], b_off[PPW];
    auto piece_col = [&](int i) __attribute__((always_inline)) { return (lane & 7) ^ (((wave * PPW + i) * 4 + (lane >> 4)) & 7); };
#pragma unroll
    for (int i = 0; i < PPW; ++i) {
        const int row = (wave * PPW + i) * 8 + (lane >> 3);
        a_off[i] = (unsigned)min(m0 + row, M - 1) * (unsigned)row_bytes + piece_col(i) * 16;
        b_off[i] = (unsigned)min(n0 + row, N - 1) * (unsigned)row_bytes + piece_col(i) * 16;
    }
    // piece i of the A (B) tile of step s < nk; `whole`: s < nfull is known (else a half step fetches its first half twice)
    auto copy = [&](const char* mat, const unsigned (&off)[PPW], int s, int i, int slot, auto whole) __attribute__((always_inline)) {
        const unsigned o = decltype(whole)::value || s < nfull ? off[i] : off[i] - (piece_col(i) & 4) * 16;
        dma16(mat + (size_t)s * 128, o, lds_base + slot * SLOT + (wave * PPW + i) * 1024);
    };

    // ---- fragments of k-step k, in the order of use (MFMA q of a k-step multiplies block q / NB of A with block q % NB of B)
    struct Frags { TileFrag<IN> am[NB], bn[NB]; };
    auto read_one = [&](Frags& f, int k, int slot_a, int slot_b, int i) __attribute__((always_inline)) {
        const int r = i / HALVES, h = i % HALVES;
        const int row = lane % BS, col = B16 ? k * 4 + (lane >> 4) : k * 4 + (lane >> 5) * 2 + h;
        const int off = row * 128 + ((col ^ ((row >> 1) & 7)) * 16);
        const bool is_a = r == 1 || r > NB;
        const int blk = r == 0 || r == 1 ? 0 : (r <= NB ? r - 1 : r - NB);
        if (is_a) f.am[blk].h[h] = *reinterpret_cast<const i32x4*>(smem + slot_a * SLOT + wm * 16384 + off + blk * (BS * 128));
        else f.bn[blk].h[h] = *reinterpret_cast<const i32x4*>(smem + slot_b * SLOT + wn * 16384 + off + blk * (BS * 128));
    };

    typedef typename std::conditional<B16, f32x4, f32x16>::type block_t;
    block_t acc[NB][NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) acc[nb][mb] = block_t(0.f);

    typedef std::integral_constant<bool, true> yes_t;
    typedef std::integral_constant<bool, false> no_t;
    auto next_slot = [](int s, int by) __attribute__((always_inline)) { s += by; return s >= SLOTS ? s - SLOTS : s; };

    // ---- one k-step: the MFMAs on `cur` (unless `skip`: the missing k-step of a half step, the very last one); between them the reads of the
    // next k-step's fragments (while read_next) and whatever `behind(q)` issues
    auto kstep = [&](const Frags& cur, Frags& nxt, int next_k, int slot_a, int slot_b, bool skip, bool read_next, auto behind) __attribute__((always_inline)) {
        auto between = [&](int q) __attribute__((always_inline)) {
            if (q % READ_EVERY == 0 && q / READ_EVERY < READS && read_next) read_one(nxt, next_k, slot_a, slot_b, q / READ_EVERY);
            behind(q);
        };
        if (skip) {
#pragma unroll
            for (int q = 0; q < NB * NB; ++q) between(q);
            return;
        }
#pragma unroll
        for (int q = 0; q < NB * NB; ++q) {
            const int mb = q / NB, nb = q % NB;
            if constexpr (B16)
                acc[nb][mb] = Elem<IN>::mfma16(__builtin_bit_cast(s16x8, cur.bn[nb].h[0]), __builtin_bit_cast(s16x8, cur.am[mb].h[0]), acc[nb][mb]);
            else
                acc[nb][mb] = tile_mfma<IN>(cur.bn[nb], cur.am[mb], acc[nb][mb]);
            __builtin_amdgcn_sched_barrier(0);
            between(q);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto nothing = [](int) __attribute__((always_inline)) {};

    // ---- prologue: the whole ring in flight; step 0 complete for everyone
#pragma unroll
    for (int s = 0; s < 3; ++s)
        if (s < nk) {
#pragma unroll
            for (int i = 0; i < PPW; ++i) copy(A, a_off, s, i, 2 * s, no_t());
            if (s < 2) {
#pragma unroll
                for (int i = 0; i < PPW; ++i) copy(B, b_off, s, i, 2 * s + 1, no_t());
            }
        }
    if (nk > 2) wait_vmcnt<3 * PPW>(); else if (nk > 1) wait_vmcnt<2 * PPW>(); else wait_vmcnt<0>();
    ring_barrier();
    Frags X, Y;
#pragma unroll
    for (int i = 0; i < READS; ++i) read_one(X, 0, 0, 1, i);
#pragma unroll
    for (int k = 0; k < KSTEPS - 1; ++k)
        kstep(k & 1 ? Y : X, k & 1 ? X : Y, k + 1, 0, 1, false, true, nothing);   // (the launcher keeps nfull >= 1)

    // ---- from the barrier of step p to that of step p + 1: the last k-step of p, the others of p + 1.  STEADY: step p + 3
    // exists and is whole.
    int sa = 0;                                 // slot of A_p (B_p has the next one)
    auto span = [&](int p, auto steady) __attribute__((always_inline)) {
        constexpr bool STEADY = decltype(steady)::value;
        if (STEADY || p + 2 < nk) wait_vmcnt<PPW>(); else wait_vmcnt<0>();   // own copies of step p + 1
        __builtin_amdgcn_s_waitcnt(0xC07F);     // lgkmcnt(0): this wave has read step p
        ring_barrier();
        const int free_a = sa, free_b = next_slot(sa, 1);
        sa = next_slot(sa, 2);
        const int sb = next_slot(sa, 1);
#pragma unroll
        for (int k0 = 0; k0 < KSTEPS; ++k0) {   // k-step k0 of the span reads the fragments of k-step k0 of step p + 1
            kstep(k0 & 1 ? X : Y, k0 & 1 ? Y : X, k0, sa, sb, false, true, [&](int q) __attribute__((always_inline)) {
                const int slot = k0 * NB * NB + q;
                if (slot % COPY_EVERY != COPY_EVERY - 1) return;
                const int i = slot / COPY_EVERY;
                if (i < PPW) {
                    if (STEADY || p + 2 < nk) copy(B, b_off, p + 2, i, free_a, steady);
                } else {
                    if (STEADY || p + 3 < nk) copy(A, a_off, p + 3, i - PPW, free_b, steady);
                }
            });
        }
    };
    int p = 0;
    if (p + 3 < nfull) {
        do { span(p, yes_t()); } while (++p + 3 < nfull);
    }
    if (p + 1 < nk) {
        do { span(p, no_t()); } while (++p + 1 < nk);
    }
    // ---- the last k-step.  Behind the barrier everything has been copied and read: the epilogue may use the ring.
    wait_vmcnt<0>();
    __builtin_amdgcn_s_waitcnt(0xC07F);
    ring_barrier();
    kstep(Y, X, 0, 0, 0, nk > nfull, false, nothing);
    store_wave_block_of<E>(smem + wave * 8192, acc, C, M, N, m0 + wm * 128, n0 + wn * 128, lane);
}

template <int IN, int OUT>
int launch_wide(const GemmLaunchArgs& a)
{
    constexpr int smem = 5 * 256 * 128;
    if (a.K * (IN == 2 ? 1 : 2) < 128) return -1;   // the first step must be whole
    auto kern = gemm_nt_wide_kernel<IN, OUT>;
    static PerDeviceOnce once;                  // the attribute belongs to the (kernel, device) pair
    if (once.prepare(reinterpret_cast<const void*>(kern), smem) < 0) return -1;
    const char* A = (const char*)a.a;
    const char* B = (const char*)a.b;
    uint16_t* C = (uint16_t*)a.c;
    int M = a.M, N = a.N, row_bytes = a.K * (IN == 2 ? 1 : 2);
    int ntm = (M + 255) / 256, ntn = (N + 255) / 256;
    void* args[] = {&A, &B, &C, &M, &N, &row_bytes, &ntm, &ntn};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3((unsigned)(ntm * ntn)), dim3(256), args, smem, (hipStream_t)a.stream);
    return e == hipSuccess ? 0 : -1;
}

// ---- which kernel takes a product.  Estimated time in microseconds of each candidate on a chip of CHIP_CUS CUs, from the
// number of its tiles and of 128-byte steps along K (one step of the kernels above, and the same MFMA time for every
// element type): start-up + rounds * (prologue and epilogue of a tile + steps * time per step).  A round is one tile on
// every CU, also where two workgroups share a CU (shapes 1 and 2: their times per step are those of two tiles in
// turn).  A step is cheaper while part of the chip is idle (step_idle: no other tile running).  Fitted to times measured on
// MI355X, three sets of buffers in turn, bf16 and E4M3.  The fit was last taken over M, N >= 2048 and rows of 512 ... 8192 bytes, where the
// choice is within 2.3 % of the best of the four.  On 251 products drawn over M, N = 16 ... 8192 and rows of 64 ... 32768
// bytes the choice costs more than 5 % in seven, 21 % at the worst; six of these have one to three steps.
// Microseconds at M x N x K, bf16, in the order 256 x 256, 64 x 64, 128 x 128 in pairs, 128 x 128 with split k-steps (the
// choice in brackets):
//    8192 x 8192 x 256      60    105    [56]   83        8192 x 8192 x 2048 [198] 377   239   278
//    8192 x 8192 x 512     [81]   137     83   107        4096 x 4096 x 256  [13.9] 28.3  16.5 22.6
//    3000 x 3000 x 256     13.1  17.6  [13.4] 17.1        3000 x 3000 x 512  [17.0] 21.8  18.8 22.1
//    2048 x 2048 x 256     11.2   8.6   [6.3]  7.1        2048 x 2048 x 4096   70    50    41  [32]
//    1000 x 777 x 512      30    [5.0]   9.3   8.5        64 x 64 x 16384     245   [35]   92   68
// Where shape 1 is chosen the smallest products go on to 32 x 32 or 16 x 16 tiles (gemm_nt_narrow_kernel.hip: 12.5 us for the last one).  Its
// model knows 64 x 64 tiles only, which decides nothing: wherever the smaller tiles apply, 64 x 64 ones are the model's choice too.
struct ShapeModel { int tile; float start, per_tile, step_idle, step_full; };
constexpr ShapeModel T_MODEL[4] = {
    {256, 1.5f, 8.5f, 0.95f, 1.30f},        // 0: gemm_nt_wide_kernel
    {64, 2.0f, 1.0f, 0.13f, 0.185f},        // 1
    {128, 3.5f, 1.6f, 0.41f, 0.41f},        // 2
    {128, 1.0f, 4.5f, 0.28f, 0.48f},        // 3
};
constexpr float T_ALONE = 0.13f;            // shape 2: what a step costs more in a round without a partner

template <int IN, int OUT>
int launch_shape(const GemmLaunchArgs& a, int shape)
{
    // E4M3 products keep one order of summation in every kernel (bit-identical results), so no wave splits their k-steps.
    constexpr bool F8 = IN == 2;
    switch (shape) {
        case 1: return launch_tile<IN, OUT, 64, 64, 2, 2, F8 ? 1 : 2, 4, 2>(a);
        case 2: return launch_tile<IN, OUT, 128, 128, 2, 2, 1, 2, 2>(a);
        case 3: return launch_tile<IN, OUT, 128, 128, F8 ? 4 : 2, 2, F8 ? 1 : 2, 4, 1>(a);
        case 0: return launch_wide<IN, OUT>(a);
        default: return -1;
    }
}

}  // namespace

int gemm_tile_launch(const GemmLaunchArgs& a, int in_type, int shape)
{
    if (in_type == 0) return launch_shape<0, 0>(a, shape);
    if (in_type == 1) return launch_shape<1, 1>(a, shape);
    return a.dtype == 0 ? launch_shape<2, 0>(a, shape) : launch_shape<2, 1>(a, shape);
}

int gemm_default_launch(const GemmLaunchArgs& a, int in_type)
{
    const long long row_bytes = (long long)a.K * (in_type == 2 ? 1 : 2);
    const int shape = gemm_tile_shape(a.M, a.N, row_bytes), narrow = shape == 1 ? gemm_narrow_tile(a.M, a.N, row_bytes, in_type == 2) : 0;
    return narrow ? gemm_narrow_launch(a, in_type, narrow) : gemm_tile_launch(a, in_type, shape);
}

int gemm_tile_shape(int M, int N, long long row_bytes)
{
    const float steps = (float)((row_bytes + 127) / 128);
    int best = -1;
    float best_time = 0.f;
    for (int s = row_bytes < 128 ? 1 : 0; s < 4; ++s) {
        const ShapeModel& m = T_MODEL[s];
        const long long tiles = ((M + m.tile - 1LL) / m.tile) * ((N + m.tile - 1LL) / m.tile), rounds = (tiles + CHIP_CUS - 1) / CHIP_CUS;
        const float load = tiles < CHIP_CUS ? tiles / (float)CHIP_CUS : 1.0f;
        float time = m.start + rounds * (m.per_tile + (m.step_idle + (m.step_full - m.step_idle) * load) * steps);
        if (s == 2 && (rounds & 1)) time += T_ALONE * steps;
        if (best < 0 || time < best_time) {
            best = s;
            best_time = time;
        }
    }
    return best;
}
