// Fused attention forward for gfx950 (MI355X): O = softmax(scale * Q K^T [+ causal mask]) V and
// per-row log-sum-exp, in one kernel with a streaming softmax.
//
// The three stages of one key/value tile follow the paper's Section 3.4.2: T = Q K^T on the matrix
// cores, C = softmax on the vector ALU, U = P V on the matrix cores, and the goal is the one of its
// coarse-grained pipeline (Algorithm 1): keep the matrix cores busy while the vector ALU works.
//
// What carries over from the paper's Hopper design and what does not:
//  * Producer/consumer warp roles are gone.  Every wave issues its share of the global -> LDS copies
//    (direct-to-LDS loads, no register staging) two tiles ahead of their use.  The LDS holds a ring of
//    STAGES tiles, the counterpart of an aref ring of depth D (Section 3.3.2); one s_waitcnt plus one
//    s_barrier per tile play the role of the full/empty credits: a stage is overwritten only after
//    every wave has passed the barrier that follows its last read of it.
//  * The overlap of Algorithm 1 is realised BETWEEN the two waves that share a SIMD: the eight waves of a workgroup
//    form two groups of four (one wave of each group per SIMD) that run the same pipeline half a period apart,
//        group A after barrier j:  [U_{j-1}, T_j] on the matrix cores, then C_j on the vector ALU
//        group B after barrier j:  C_j on the vector ALU, then [U_j, T_{j+1}] on the matrix cores
//    so while one wave of a SIMD streams its MFMAs the other one does its softmax.  The workgroup
//    barrier re-locks the two groups into opposite phases every tile.
//
// Register layout.  The scores are computed transposed, S^T = K Q^T, with the 16x16x32 MFMA: the
// K tile is the A operand (16 keys x 32 features), Q^T the B operand.  A lane then owns ONE query
// (column lane%16 of the result) of each of its wave's 16-query blocks, and four of the 16 keys of a block; the other
// keys of that query sit in the lanes 16, 32 and 48 further on.  The probabilities of two key blocks are already laid out as the
// B operand of the second contraction O^T = V^T P^T (which key stands at which step of a contraction is free, as
// long as V^T follows).  V^T fragments come from the LDS through the transposing 64-bit read of gfx950.
//
// What bounds it at d = 128: the power the matrix cores draw.  On operands of zeros N = 16384, 16 heads, fp16, takes 1200 us
// with either MFMA size, on N(0,1) operands 1845 us with 32x32x16 and 1670 with 16x16x32, which moves half as much of the
// fp32 accumulators per flop (one session; 4 x 16 heads, N = 4096, bf16: 457 / 420; causal, 2 x 32 heads, N = 8192: 918 / 855).
// At d = 64 it is the issue of vector instructions: the softmax of a wave and tile takes 800 cycles by itself (of them 32
// exponentials 10 each, 16 conversions 8 each) and each MFMA of the other waves holds up the vector ALU for 6 to 7, whatever its
// size (256 heads, N = 1024: 81 us / 75).
//
// The row sums are a further row of the second contraction, a block of ones next to V^T (one MFMA per 32 keys and 16 queries):
// the packed dot products that did it on the vector side go through the matrix pipe as well and cost it more (N = 16384 as above:
// 1727 us with them, 1667 without).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "attn_launch.h"
#include "gfx950_prims.h"
#include "key_split.h"
#include "launch_once.h"
#include "tile_schedule.h"

namespace {

// The softmax reference moves only when a row maximum grew by more than this many powers of two.
constexpr float RESCALE_LOG2 = 8.0f;

// LDS fragments requested ahead of their MFMA inside a burst (see mfma_burst).
#ifndef ATTN_FWIN
#define ATTN_FWIN 2
#endif

// 1: launch one workgroup per resident slot and let each walk several tiles; 0: one workgroup per tile.
#ifndef ATTN_PERSISTENT
#define ATTN_PERSISTENT 1
#endif

// 1: the causal d = 64 launch is persistent as well (measured on MI355X: see launch_d).
#ifndef ATTN_PERSISTENT_D64
#define ATTN_PERSISTENT_D64 1
#endif

// 1: small grids take the form that splits the keys of a tile between the wave groups (see key_split.h).
#ifndef ATTN_KEY_SPLIT
#define ATTN_KEY_SPLIT 1
#endif

// Which wave group issues the global -> LDS copies (see COPY_WAVES in the kernel).
#ifndef ATTN_COPY_GROUP
#define ATTN_COPY_GROUP 0
#endif

// 1: in the steady state a wave issues its copies of a stage one at a time between the exponentials of the
// softmax; 0: as one block before the softmax (a wave is held ~270 cycles per tile by that block).  Measured
// on MI355X: spreading them loses 1-2 % (c3, c4, c5), and so does issuing the block at a different point
// of the softmax in each wave of a group: the ~70 cycles per copy instruction are not a queue, so the block stays.
#ifndef ATTN_COPIES_IN_SOFTMAX
#define ATTN_COPIES_IN_SOFTMAX 0
#endif

#ifdef ATTN_TIMING
// Profiling builds only: per-wave cycle totals of the main-loop sections of the first workgroups.
constexpr int DBG_WGS = 1024, DBG_SLOTS = ATTN_TIMING >= 3 ? 32 : 8;
__device__ unsigned long long attn_dbg[DBG_WGS * 8 * DBG_SLOTS];
#if ATTN_TIMING >= 2
#define TSTAMP(var) unsigned long long var; __builtin_amdgcn_sched_barrier(0); \
    asm volatile("s_memtime %0\n\ts_waitcnt lgkmcnt(0)" : "=s"(var) :: "memory"); __builtin_amdgcn_sched_barrier(0)
#if ATTN_TIMING >= 3   // absolute stamps of iterations 100..103
#define TACC(slot, a, b) if (j >= 100 && j < 104) { dbg_acc[8 + (j - 100) * 5 + slot] = (a); if (slot == 3) dbg_acc[8 + (j - 100) * 5 + 4] = (b); }
#else
#define TACC(slot, a, b) dbg_acc[slot] += (b) - (a)
#endif
#else
#define TSTAMP(var)
#define TACC(slot, a, b)
#endif
#else
#define TSTAMP(var)
#define TACC(slot, a, b)
#endif

// Exchange with lane^32 (v_permlane32_swap swaps the upper 32 lanes of its first operand with the
// lower 32 lanes of its second).  Written as inline asm because clang 22 folds the two results of __builtin_amdgcn_permlane32_swap into one
// when both inputs are the same value (fmax(r[0], r[1]) is compiled as r[0]), which silently drops the partner lane.  The s_nop covers
// the VALU-write -> permlane-read hazard the compiler would otherwise handle.
__device__ __forceinline__ void swap32(float& a, float& b) {
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
// The lower half's values of x on every lane, and the upper half's.
__device__ __forceinline__ void both_halves(float x, float& lower, float& upper) {
    lower = x;
    upper = x;
    swap32(lower, upper);
}
// Maximum with lane^16 (v_permlane16_swap: odd rows of 16 lanes of the first operand against even rows of the second).
__device__ __forceinline__ float xor16_max(float x) {
    float a = x, b = x;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    return __builtin_fmaxf(a, b);
}

// (d = 64: the LDS ring is 64 KiB, two workgroups fit a CU; the second launch bound, waves per SIMD, asks the
// compiler for the 128 registers per lane that let their 16 waves be resident together: 256 heads, N = 1024, 88 us without
// it, 75 with it.  The persistent kernel loads the next tile's Q under the epilogue and needs 170; held to 128 it spills and is slower, causal
// 58 -> 61 us, and without its persistence 67.)
// KS = 2 (small grids): the two wave groups of a workgroup work on the SAME NW / 2 * 32 query rows and share out the keys of
// every tile, group A the first half and group B the second, each with a softmax state of its own; at the end
// partner waves (w and w + 4) exchange halves of O and their maxima and sums through the LDS and each stores half of
// the features.  A workgroup then covers 128 rows in about half the time of 256, twice as many of them are there to
// fill the chip, and both groups keep their phases (one on the matrix cores while the other does its softmax).
template <int DTYPE, int D, int NW, int MB, int BN, int STAGES, bool CAUSAL, bool PERSIST, int KS = 1>
__global__ __launch_bounds__(NW * 64, (D == 64 && MB == 1 && !PERSIST) ? 4 : 1)
void attn_fwd_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                     uint16_t* __restrict__ o, float* __restrict__ lse, int N, int nqt, int total,
                     float scale, float scale_log2e, float m_none)
{
    typedef Elem<DTYPE> E;
    constexpr int BM = NW * MB * 32 / KS;       // query rows per workgroup
    constexpr int KB = BN / 16 / KS;            // 16-key blocks of a K/V tile that a wave computes on
    constexpr int QB = MB * 2;                  // 16-query blocks of a wave
    constexpr int KK = D / 32;                  // contraction steps of Q K^T
    constexpr int FB = D / 16;                  // 16-wide feature blocks of O
    constexpr bool AHEAD = KS == 2;             // see fetch_ahead
    constexpr bool BLOCK_BY_BLOCK = KS == 2 && D == 128;                 // see softmax_tile
    constexpr int ROW_BYTES = D * 2;
    constexpr int TILE_BYTES = BN * ROW_BYTES;  // one K or one V tile
    constexpr int STAGE_BYTES = 2 * TILE_BYTES;
    constexpr int RB = BN / 8;                  // 8-row blocks per tile
    constexpr int CHUNKS = TILE_BYTES / 1024;   // 1 KiB wave-transfers per tile
    // Which waves issue the copies: 0 = all eight, 1 = group B only, 2 = group A only.
    constexpr int NG = NW / 4;                  // wave groups: one wave of each group per SIMD
    constexpr int COPY_WAVES = NG == 3 ? 8 : (ATTN_COPY_GROUP == 0 ? NW : NW / 2);
    constexpr int CPW = CHUNKS / COPY_WAVES;    // ... per copying wave
    constexpr int LPG = 2 * CPW;                // copies such a wave issues per stage (K part + V part)
    static_assert(CHUNKS % COPY_WAVES == 0, "tile must split evenly over the copying waves");
    static_assert(STAGES == 4, "the ring protocol below keeps four stages");
    static_assert(KS == 1 || (KS == 2 && NW == 8 && !PERSIST), "the key split pairs the two wave groups");
    static_assert(NW == 8 || NW == 12, "two or three groups of four waves, one wave of each group per SIMD");

#ifdef ATTN_TIMING
    const unsigned long long rt_kernel_entry = __builtin_amdgcn_s_memrealtime();
#endif
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const unsigned lds_base = (unsigned)(size_t)(LDS_AS void*)smem;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform, kept in an SGPR
    const int lane = threadIdx.x & 63;
    const int lc = lane & 15, lg = lane >> 4;   // column of a 16 x 16 block (query), and which four of its rows
    const int group = __builtin_amdgcn_readfirstlane(wave >> 2);   // waves w, w + 4 (, w + 8) share a SIMD
    const bool group_b = group == NG - 1;       // the group that does its softmax first
    const int kb0 = KS == 2 ? group * KB : 0;   // first 16-key block of a tile that this wave computes on

    // ---- which (batch*head, query tile) the workgroup works on: set per round of the tile schedule
    int round = 0;
    int logical __attribute__((unused)), bh, wq0, nt, nt_w;             // nt: K/V tiles the workgroup walks; nt_w: those this wave computes on
    size_t head_off;
    const uint16_t* qh;
    const char *kh, *vh;
    auto set_tile = [&](int tile) __attribute__((always_inline)) {
        tile = __builtin_amdgcn_readfirstlane(tile);   // wave-uniform by construction; keeps all of the below in SGPRs
        logical = tile;
        bh = __builtin_amdgcn_readfirstlane(tile / nqt);   // (the division runs on the vector ALU)
        int qt = tile - bh * nqt;
        if (CAUSAL) qt = nqt - 1 - qt;          // long rows first
        const int q0 = qt * BM;
        wq0 = q0 + (KS == 2 ? wave & 3 : wave) * (MB * 32);   // first query row of this wave
        head_off = (size_t)bh * N * D;
        qh = q + head_off;
        kh = reinterpret_cast<const char*>(k + head_off);
        vh = reinterpret_cast<const char*>(v + head_off);
        nt = (N + BN - 1) / BN;
        if (CAUSAL) {
            const int last_q = min(q0 + BM, N) - 1;
            nt = min(nt, last_q / BN + 1);
        }
        nt_w = nt;
        if (CAUSAL) nt_w = min(nt, (wq0 + MB * 32 - 1) / BN + 1);   // later tiles are wholly hidden from this wave's rows
        if (KS == 2) {                          // the same for this wave's share of the keys (may be 0 for group B)
            const int last_key = (CAUSAL ? min(wq0 + MB * 32, N) : N) - 1 - kb0 * 16;
            nt_w = last_key < 0 ? 0 : min(nt, last_key / BN + 1);
        }
        // All of these are wave-uniform; say so, or values that cross the tile loop end up in vector registers.
        nt = __builtin_amdgcn_readfirstlane(nt);
        nt_w = __builtin_amdgcn_readfirstlane(nt_w);
        wq0 = __builtin_amdgcn_readfirstlane(wq0);
        kh = uniform_ptr(kh);
        vh = uniform_ptr(vh);
    };
    set_tile(tile_schedule(total, (int)gridDim.x, (int)blockIdx.x, 0));   // the launcher keeps grid <= total

    // ---- global -> LDS copies.  Stage s of the ring holds K tile s+1 and V tile s: the pair that one
    // MFMA burst reads (U_s needs V_s, T_{s+1} needs K_{s+1}).  A wave moves CPW 1 KiB pieces of each.
    // K and V tile in LDS: [feature group of 64][row (BN)][128 B], the 16-byte columns of a row permuted.  A piece is 8 rows
    // x 128 bytes, whole memory lines (16 rows x 64 bytes, whose lanes ask for 64 or 16 bytes at a time, cost up to 5 % on calls
    // of few tiles: 4 x 16 heads, N = 1024, d 128, causal 28.5 -> 27.8 us; 2 heads, N = 128, d 64 5.4 -> 5.1): lane L fetches row L/8.  K: column c of row r sits at c ^ (r / 2) % 8, so that the 16 rows
    // that a fragment read takes one column of cover all banks; V: the 32-byte pairs of columns at p ^ (r / 2) % 4, for the 8
    // rows x 32 bytes that half a wave of the transposing read covers.  Inside the sequence the per-lane offset is a constant
    // and the tile/piece offset is added to the scalar base; the clamped form serves tiles that overrun the
    // sequence (their surplus rows are masked or never read).
    const unsigned k_lane_col = ((lane & 7) ^ (lane >> 4)) * 16;                 // of an even piece; odd ones: ^ 64
    const unsigned v_lane_col = ((lane & 7) ^ ((lane >> 4) * 2)) * 16;
    const unsigned k_lane_off = (lane >> 3) * ROW_BYTES + k_lane_col;
    const unsigned v_lane_off = (lane >> 3) * ROW_BYTES + v_lane_col;
    // does this wave issue copies, and its index among the copying waves (three groups: the first eight waves)
    const bool copies = NG == 3 ? wave < 8 : (ATTN_COPY_GROUP == 0 || (ATTN_COPY_GROUP == 1) == group_b);
    const int cwave = (NG == 3 || ATTN_COPY_GROUP == 0) ? wave : (wave & (NW / 2 - 1));
    int piece_src[CPW], piece_dst[CPW];         // wave-uniform: source offset inside a tile, LDS offset inside a K or V slot
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        const int wc = cwave * CPW + i, fg = wc / RB, rb = wc % RB;
        piece_src[i] = rb * 8 * ROW_BYTES + fg * 128;
        piece_dst[i] = wc * 1024;
    }
    auto issue_stage = [&](int s) __attribute__((always_inline)) {             // s = -1 is the stage that only brings K tile 0
        if (!copies) return;
        const unsigned sbase = lds_base + ((s + STAGES) % STAGES) * STAGE_BYTES;
        if (s >= 0 && (s + 2) * BN <= N) {      // K tile s+1 and V tile s lie wholly inside the sequence
            const char* kt = kh + (size_t)(s + 1) * TILE_BYTES;
            const char* vt = vh + (size_t)s * TILE_BYTES;
#pragma unroll
            for (int i = 0; i < CPW; ++i) dma16(kt + piece_src[i], k_lane_off ^ (((cwave * CPW + i) & 1) * 64), sbase + piece_dst[i]);
#pragma unroll
            for (int i = 0; i < CPW; ++i) dma16(vt + piece_src[i], v_lane_off, sbase + TILE_BYTES + piece_dst[i]);
        } else {
#pragma unroll
            for (int i = 0; i < CPW; ++i) {
                const int wc = cwave * CPW + i, fg = wc / RB, rb = wc % RB;
                const int row = min(max((s + 1) * BN + rb * 8 + (lane >> 3), 0), N - 1);
                dma16(kh, (unsigned)(row * ROW_BYTES + fg * 128) + (k_lane_col ^ ((wc & 1) * 64)), sbase + piece_dst[i]);
            }
#pragma unroll
            for (int i = 0; i < CPW; ++i) {
                const int wc = cwave * CPW + i, fg = wc / RB, rb = wc % RB;
                const int row = min(max(s * BN + rb * 8 + (lane >> 3), 0), N - 1);
                dma16(vh, (unsigned)(row * ROW_BYTES + fg * 128 + v_lane_col), sbase + TILE_BYTES + piece_dst[i]);
            }
        }
    };

    // One copy of a stage that lies wholly inside the sequence: K piece i < CPW, else V piece i - CPW.
    auto issue_piece_inside = [&](int s, int i) __attribute__((always_inline)) {
        const unsigned sbase = lds_base + ((s + STAGES) % STAGES) * STAGE_BYTES;
        if (i < CPW) dma16(kh + (size_t)(s + 1) * TILE_BYTES + piece_src[i], k_lane_off ^ (((cwave * CPW + i) & 1) * 64), sbase + piece_dst[i]);
        else dma16(vh + (size_t)s * TILE_BYTES + piece_src[i - CPW], v_lane_off, sbase + TILE_BYTES + piece_dst[i - CPW]);
    };

    // ---- prologue of a tile: three stages in flight, Q fragments into registers
    s16x8 Qf[QB][KK];
    auto prologue = [&]() __attribute__((always_inline)) {
        issue_stage(-1);
        issue_stage(0);
        issue_stage(1);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int row = min(wq0 + qb * 16 + lc, N - 1);
            const uint16_t* qr = qh + (size_t)row * D;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
                Qf[qb][kk] = *reinterpret_cast<const s16x8*>(qr + (kk * 4 + lg) * 8);
        }
    };
    prologue();

    f32x4 O[FB][QB], S[KB][QB];
    u32x4 pw[KB / 2][QB];                       // P of the current tile as packed 16-bit pairs: the B operands of U
    // reference of a row and what it adds to every exponent (-reference * scale * log2 e); both the same in the four lanes of a query
    float m_run[QB], neg_mc[QB];
    f32x4 L[QB];                                // row sums of P: the first element (the others miss the rescaling)
    s16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = E::ONE;

    // per-lane LDS read offsets (the rest of every address is an immediate)
    const int k_lane = (kb0 * 16 + lc) * 128 + ((lg ^ (lc >> 1)) * 16);
    const int v_lane = TILE_BYTES + (kb0 * 16 + 4 * lg + (lc >> 2)) * 128 + ((2 * lg + (lc >> 3)) & 3) * 32 + (lane & 3) * 8;

    // K fragment (A operand of T): keys kb*16 + lane%16, features (kk*4 + lane/16)*8 .. +7
    auto read_kf = [&](const char* const (&sk)[2], int kb, int kk) __attribute__((always_inline)) -> s16x8 {
        return *reinterpret_cast<const s16x8*>(sk[kk & 1] + (kk >> 1) * (BN * 128) + kb * 16 * 128);
    };
    // V^T fragment (A operand of U): features fb*16 + lane%16, the 8 keys of blocks 2t and 2t + 1 that the P
    // operand of the MFMA holds in this lane group, fetched with the transposing LDS read
    auto read_vf = [&](const char* const (&sv)[4], int t, int fb) __attribute__((always_inline)) -> s16x8 {
        const char* a = sv[fb & 3] + (fb >> 2) * (BN * 128) + t * 32 * 128;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(a));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(a + 16 * 128));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };

    // ---- MFMA burst on one stage: U (O^T += V^T P^T with the P in pw) and/or T (S^T = K Q^T), as one
    // stream of MFMAs whose LDS fragments are requested FWIN MFMAs ahead.  The scheduling barriers
    // keep that order: left alone the compiler requests each fragment right before its MFMA.
    // KS = 2: the first fragments of U are requested as soon as their stage is complete, a softmax before the burst that uses them.
    // A split tile is a serial chain of latencies rather than a queue for the matrix cores (8 heads, N = 2309, causal: 33.5 -> 32.0 us;
    // with 256-row tiles no difference).
    s16x8 ahead[ATTN_FWIN];
    auto fetch_ahead = [&](const char* stage_ptr) __attribute__((always_inline)) {
        if (!AHEAD) return;
        const char* const sv[4] = {stage_ptr + v_lane, stage_ptr + (v_lane ^ 32), stage_ptr + (v_lane ^ 64), stage_ptr + (v_lane ^ 96)};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < ATTN_FWIN; ++f) ahead[f] = read_vf(sv, f / FB, f % FB);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mfma_burst = [&](auto do_u, auto do_t, const char* stage_ptr) __attribute__((always_inline)) {
        constexpr int NU = decltype(do_u)::value ? KB / 2 * FB : 0;
        constexpr int NT = decltype(do_t)::value ? KB * KK : 0;
        constexpr int NF = NU + NT;
        constexpr int FWIN = ATTN_FWIN < NF ? ATTN_FWIN : NF;
        const char* const sk[2] = {stage_ptr + k_lane, stage_ptr + (k_lane ^ 64)};
        const char* const sv[4] = {stage_ptr + v_lane, stage_ptr + (v_lane ^ 32), stage_ptr + (v_lane ^ 64), stage_ptr + (v_lane ^ 96)};
        s16x8 fr[NF];
        constexpr bool HAVE = AHEAD && NU > 0;
        if (HAVE) {
#pragma unroll
            for (int f = 0; f < FWIN; ++f) fr[f] = ahead[f];
        }
        auto fetch = [&](int f) __attribute__((always_inline)) {
            if (f < NU) fr[f] = read_vf(sv, f / FB, f % FB);
            else fr[f] = read_kf(sk, (f - NU) % KB, (f - NU) / KB);
        };
        auto run_mfma = [&](int f) __attribute__((always_inline)) {
            if (f < NU) {
                const int t = f / FB, fb = f % FB;
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) O[fb][qb] = E::mfma16(fr[f], __builtin_bit_cast(s16x8, pw[t][qb]), O[fb][qb]);
                if (fb == FB - 1) {
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) L[qb] = E::mfma16(ones, __builtin_bit_cast(s16x8, pw[t][qb]), L[qb]);
                }
            } else {
                const int kb = (f - NU) % KB, kk = (f - NU) / KB;
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) S[kb][qb] = E::mfma16(fr[f], Qf[qb][kk], kk == 0 ? f32x4(0.f) : S[kb][qb]);
            }
        };
        if (!HAVE) {
#pragma unroll
            for (int f = 0; f < FWIN; ++f) fetch(f);
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if (f + FWIN < NF) fetch(f + FWIN);
            run_mfma(f);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- C of tile j: mask, streaming softmax of S into pw, running reference, rescaling of O and the row sums.
    // Base-2 exponentials with the scale folded into the exponent.  The running reference m only
    // moves when a row maximum grew by more than 2^RESCALE_LOG2 (the probabilities then stay below
    // that factor), so everything about it is behind a rarely taken branch; `first`: the wave's first tile, where it is set.
    // With `spread` the wave's copies of stage j + 2 (known to lie inside the sequence) go out between the
    // exponentials, evenly spaced.
    // `part`: 0 = the whole tile; 1 = mask, maximum, reference, rescaling and the first half of the keys;
    // 2 = the second half (the middle group of three splits its softmax around its burst).
    auto softmax_tile = [&](int j, auto spread, auto part, auto first) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first)::value;
        constexpr bool SPREAD = decltype(spread)::value;
        constexpr int PART = decltype(part)::value;
        constexpr int NPAIR = KB * QB * 2, NCOPY = 2 * CPW, PER = NPAIR / NCOPY;
        static_assert(!SPREAD || (PER >= 1 && PER * NCOPY == NPAIR), "copies spread evenly over the exponentials");
        const int kv0 = j * BN;                 // first key of the tile; the wave's own start at block kb0
        if (PART != 2 && ((kv0 + BN > N) || (CAUSAL && kv0 + BN - 1 > wq0))) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const int qi = wq0 + qb * 16 + lc;
                const int lim = CAUSAL ? min(qi, N - 1) : N - 1;   // last visible key
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) {
                    // (Whole tiles pass over the blocks that every row of theirs sees: under the mask the elements to compare are what a short row
                    // spends its time on.  us without / with: d 128, 1600 heads, N 64 36.5 / 35.4; 2 x 32 heads, N 8192 880 / 867; d 64, 256 heads,
                    // N 1024 57.5 / 56.8.  In split tiles the tests cost more than they save: 8 heads, N 2309 32.2 / 32.9.)
                    if (CAUSAL && KS == 1 && kv0 + (kb0 + kb) * 16 + 15 <= min(wq0 + qb * 16, N - 1)) continue;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int key = kv0 + (kb0 + kb) * 16 + lg * 4 + i;
                        if (key > lim) S[kb][qb][i] = -__builtin_inff();
                    }
                }
            }
        }
        if (PART != 2) {
            // A lane looks at its own part of the keys only: some lane of a row exceeds the limit exactly when the row does.
            float mx[QB];
            bool over = false;
            unsigned long long over_of[QB] = {}, any = 0;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                mx[qb] = S[0][qb][0];
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) mx[qb] = __builtin_fmaxf(mx[qb], S[kb][qb][i]);
                if (FIRST) continue;
                const bool o = __builtin_fmaf(mx[qb], scale_log2e, neg_mc[qb]) > RESCALE_LOG2;
                if (BLOCK_BY_BLOCK) over_of[qb] = __builtin_amdgcn_ballot_w64(o);
                any |= over_of[qb];
                over |= o;
            }
            // (of the row sums only the first element is read, so only that one is rescaled: 43.5 -> 43.1 us at 24 heads, N 1596, causal, where
            // keys eight times as long as the others keep moving the reference)
            if (BLOCK_BY_BLOCK) {
                // Only the 16-query blocks in which a row exceeds the limit, each by itself; such a block takes the present maximum of all its rows,
                // which it is rescaled for anyway.  A split tile is a chain of latencies, and this is the shorter one (such keys, us, with the
                // form below / so: 7 heads, N 1851, causal 33.9 / 32.8, 8 heads, N 2309, causal 41.0 / 39.5, 4 heads, N 5000 78.7 / 75.7; other keys 26.8 / 26.9,
                // 32.0 / 32.1, 63.8 / 64.0, at the worst, 8 heads, N 900, 17.3 / 17.6); whole
                // tiles gain from it with such keys (24 heads, N 1596, causal 43.1 / 42.8) what they lose with others (35.8 / 36.1), and
                // split ones at d = 64 lose (27 heads, N 700, causal 12.3 / 12.5, 10.9 / 11.1).
                if (FIRST || any != 0) {
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) {
                        if (!FIRST && over_of[qb] == 0) continue;
                        const float m_old = m_run[qb];
                        float a, b;
                        both_halves(xor16_max(__builtin_fmaxf(mx[qb], m_old)), a, b);
                        m_run[qb] = __builtin_fmaxf(a, b);
                        neg_mc[qb] = -m_run[qb] * scale_log2e;
                        if (FIRST) continue;
                        const float alpha = __builtin_amdgcn_exp2f((m_old - m_run[qb]) * scale_log2e);
                        L[qb][0] *= alpha;
#pragma unroll
                        for (int fb = 0; fb < FB; ++fb) O[fb][qb] = O[fb][qb] * alpha;
                    }
                }
            } else if (FIRST || __builtin_amdgcn_ballot_w64(over) != 0) {
                // Two 16-query blocks at a time: after the first exchange the lower half of the wave carries the first, the upper half the second.
                // (Where keys eight times as long keep moving the reference, 2 x 32 heads, N 8192, causal: 982 us with each block by itself, 947 so.)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    float &m0 = m_run[2 * mb], &m1 = m_run[2 * mb + 1];
                    float a = mx[2 * mb], b = mx[2 * mb + 1];
                    swap32(a, b);
                    const float row_max = xor16_max(__builtin_fmaxf(a, b));
                    const float m_old = lane < 32 ? m0 : m1;
                    const bool moves = FIRST ? row_max > m_none : __builtin_fmaf(row_max, scale_log2e, lane < 32 ? neg_mc[2 * mb] : neg_mc[2 * mb + 1]) > RESCALE_LOG2;
                    const float m_use = moves ? row_max : m_old;
                    both_halves(m_use, m0, m1);
                    neg_mc[2 * mb] = -m0 * scale_log2e;
                    neg_mc[2 * mb + 1] = -m1 * scale_log2e;
                    if (FIRST) continue;
                    float alpha[2];
                    both_halves(__builtin_amdgcn_exp2f((m_old - m_use) * scale_log2e), alpha[0], alpha[1]);
                    const unsigned long long moved = __builtin_amdgcn_ballot_w64(moves);
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        if ((unsigned)(moved >> (32 * h)) == 0) continue;
                        L[2 * mb + h][0] *= alpha[h];
#pragma unroll
                        for (int fb = 0; fb < FB; ++fb) O[fb][2 * mb + h] = O[fb][2 * mb + h] * alpha[h];
                    }
                }
            }
        }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            if ((PART == 1 && kb >= KB / 2) || (PART == 2 && kb < KB / 2)) continue;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(S[kb][qb][2 * t], scale_log2e, neg_mc[qb]));
                    const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(S[kb][qb][2 * t + 1], scale_log2e, neg_mc[qb]));
                    const unsigned w = E::pack2(p0, p1);
                    pw[kb / 2][qb][kb % 2 * 2 + t] = w;
                    const int n = (kb * QB + qb) * 2 + t;
                    if (SPREAD && n % PER == PER / 2) {
                        __builtin_amdgcn_sched_barrier(0);
                        if (copies) issue_piece_inside(j + 2, n / PER);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
        }
    };

    // At barrier j every wave's share of stages <= j has landed (each wave waits for its own copies up
    // to stage j, leaving only stage j+1's in flight) and nobody reads stage j-2 any more, so that
    // stage takes the copies of stage j+2.
    auto wait_stage = [&](int j) __attribute__((always_inline)) {
        if (copies) {
            if (j + 1 < nt) wait_vmcnt<LPG>(); else wait_vmcnt<0>();
        }
        __builtin_amdgcn_s_barrier();
    };
    auto stage_ptr = [&](int s) __attribute__((always_inline)) -> const char* { return smem + ((s + STAGES) % STAGES) * STAGE_BYTES; };

    // ---- epilogue: normalise, write O (16-bit) and LSE (natural log).  Expanded at the end of each
    // group's code path, so that the accumulators of the two paths never have to meet in one register set.
    // A lane holds one query row, a row of O is 2 D bytes: stored straight from the registers, an instruction touches 32
    // rows with 16 bytes each.  The rows go through a piece of the ring that nobody reads any more, private to the
    // wave (so no barrier), and leave as whole 64- to 256-byte segments.
    // `region`: LDS offset of the wave's piece, 32 rows x F features; a row's 16-byte chunks are stored permuted so that
    // the 8-byte writes and the 16-byte reads cover all banks.
    // O is written through the L2 unless it is small (store_through; with KS = 1 it never is).  Ordinary stores / written through / past the caches, several
    // sets of buffers in turn, us: 512 heads, N 256, d 64 18.0 / 16.7 / 16.7, with an elementwise kernel that reads O behind
    // it 25.7 / 24.2 / 24.9, with a product 39.9 / 38.5 / 39.6; 64 heads, N 512, d 128, causal 15.2 / 14.3 / 14.4, elementwise 19.8 / 18.8 / 19.2;
    // 256 heads, N 1024, d 64 89.1 / 87.9 / 87.9, 98.6 / 97.5 / 98.3, 104.9 / 103.9 / 108.8.  Small: 8 heads, N 256, d 64 6.89 / 7.15 / 6.89.
    constexpr int EPI_F = NW == 12 ? D / 4 : (PERSIST || KS == 2 ? D / 2 : D);   // features staged at a time
    constexpr int EPI_BYTES = 32 * EPI_F * 2;
    auto epilogue = [&](size_t ep_head_off, int ep_bh, int ep_wq0, unsigned region) __attribute__((always_inline)) {
    constexpr int CH = EPI_F / 8, RPB = 16 / CH;                         // 16-byte chunks per staged row, rows per 256 bytes
    uint16_t* oh = o + ep_head_off;
    float* lh = lse + (size_t)ep_bh * N;
    char* const st = smem + region;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int row0 = ep_wq0 + mb * 32;
        const float l_row = lg ? L[mb * 2 + 1][0] : L[mb * 2][0], m_row = lg ? m_run[mb * 2 + 1] : m_run[mb * 2];
        if (lane < 32 && row0 + lane < N && !(KS == 2 && group_b)) lh[row0 + lane] = m_row * scale + __builtin_logf(l_row);
        const float inv[2] = {1.0f / L[mb * 2][0], 1.0f / L[mb * 2 + 1][0]};
#pragma unroll
        for (int part = 0; part < D / EPI_F; ++part) {
            if (KS == 2 && (part != 0) != group_b) continue;
            asm volatile("" ::: "memory");      // (order of the LDS accesses: another lane's row is read)
#pragma unroll
            for (int f = 0; f < CH / 2; ++f)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 x = O[part * (CH / 2) + f][mb * 2 + h] * inv[h];
                    const u32x2 w = {E::pack2(x[0], x[1]), E::pack2(x[2], x[3])};
                    const int row = h * 16 + lc, c = f * 2 + (lg >> 1);
                    *reinterpret_cast<u32x2*>(st + row * (CH * 16) + ((c ^ ((row / RPB) & (CH - 1))) * 16) + (lg & 1) * 8) = w;
                }
            asm volatile("" ::: "memory");
            auto rows_out = [&](auto through) __attribute__((always_inline)) {
#pragma unroll
                for (int p = 0; p < CH / 2; ++p) {                       // (the LDS accesses of a wave complete in order)
                    const int row = (p * 64 + lane) / CH, c = lane % CH;
                    const u32x4 w = *reinterpret_cast<const u32x4*>(st + row * (CH * 16) + ((c ^ ((row / RPB) & (CH - 1))) * 16));
                    uint16_t* dst = oh + (size_t)(row0 + row) * D + part * EPI_F + c * 8;
                    if (row0 + row < N) {
                        if (decltype(through)::value) store_through(dst, w);
                        else *reinterpret_cast<u32x4*>(dst) = w;
                    }
                }
            };
            if (KS == 1 || total > SMALL_RESULT / (BM * D * 2)) rows_out(std::true_type{}); else rows_out(std::false_type{});
        }
    }
    };

    // ---- end of a tile: when the schedule has another tile for this workgroup, its prologue is issued
    // first (after a barrier: every wave is then done reading the ring), so that its copies and Q
    // loads are in flight while the epilogue of the finished tile normalises and stores.  The epilogue stages its rows in
    // slots that hold neither a stage still being read (nt - 1, or nt - 2) nor one being filled: slot 2 under the next
    // prologue (stages -1, 0, 1), else those of the stages nt and nt + 1, which no copy targets; with KS = 2 above the exchange area.
    // ---- KS = 2: O, row sum and reference of this wave become those of all keys, for the half of the features that it
    // stores.  The reference of a wave without any visible key is m_none, its sums are 0.
    constexpr int XCHG_FLOATS = QB * (FB / 2 * 4 + 2);                   // floats per lane
    auto merge_groups = [&](auto upper) __attribute__((always_inline)) {
        constexpr int SEND = decltype(upper)::value ? 0 : FB / 2, KEEP = FB / 2 - SEND;   // feature blocks
        constexpr int FLOATS = XCHG_FLOATS;
        static_assert(NW * FLOATS * 256 <= STAGES * STAGE_BYTES, "the exchange reuses the ring");
        char* const mine = smem + wave * (FLOATS * 256);
        const char* const other = smem + (wave ^ 4) * (FLOATS * 256);
        __syncthreads();                        // nobody reads the ring any more
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
            for (int t = 0; t < FB / 2; ++t)
                *reinterpret_cast<f32x4*>(mine + (qb * (FB / 2) + t) * 1024 + lane * 16) = O[SEND + t][qb];
            *reinterpret_cast<f32x2*>(mine + QB * (FB / 2) * 1024 + qb * 512 + lane * 8) = f32x2{m_run[qb], L[qb][0]};
        }
        __syncthreads();
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const f32x2 ml = *reinterpret_cast<const f32x2*>(other + QB * (FB / 2) * 1024 + qb * 512 + lane * 8);
            const float m = __builtin_fmaxf(m_run[qb], ml[0]);
            const float w0 = __builtin_amdgcn_exp2f((m_run[qb] - m) * scale_log2e), w1 = __builtin_amdgcn_exp2f((ml[0] - m) * scale_log2e);
            L[qb][0] = L[qb][0] * w0 + ml[1] * w1;
            m_run[qb] = m;
#pragma unroll
            for (int t = 0; t < FB / 2; ++t) {
                const f32x4 x = *reinterpret_cast<const f32x4*>(other + (qb * (FB / 2) + t) * 1024 + lane * 16);
                O[KEEP + t][qb] = O[KEEP + t][qb] * w0 + x * w1;
            }
        }
    };

    bool more = true;
    auto finish_tile = [&]() __attribute__((always_inline)) {
        const size_t ep_head_off = head_off;
        const int ep_bh = bh, ep_wq0 = wq0;
        const int next = PERSIST ? tile_schedule(total, (int)gridDim.x, (int)blockIdx.x, ++round) : -1;
        more = next >= 0;
        unsigned region;
        if (PERSIST) {
            static_assert(!PERSIST || NW * EPI_BYTES <= STAGE_BYTES, "one free slot");
            region = 2 * STAGE_BYTES + wave * EPI_BYTES;
        } else if (KS == 2) {
            constexpr int ABOVE = NW * XCHG_FLOATS * 256;        // what merge_groups used
            static_assert(PERSIST || KS != 2 || ABOVE + NW * EPI_BYTES <= STAGES * STAGE_BYTES, "above the exchange area");
            region = ABOVE + wave * EPI_BYTES;
        } else {
            static_assert(PERSIST || KS == 2 || NW / 2 * EPI_BYTES <= STAGE_BYTES, "two free slots");
            region = ((nt + wave / (NW / 2)) % STAGES) * STAGE_BYTES + wave % (NW / 2) * EPI_BYTES;
        }
        if (more) {
            __builtin_amdgcn_s_barrier();
            set_tile(next);
            prologue();
        } else if (PERSIST) {
            __builtin_amdgcn_s_barrier();       // (slot 2 may hold one of the last two stages)
        }
        epilogue(ep_head_off, ep_bh, ep_wq0, region);
    };

#ifdef ATTN_TIMING
    unsigned long long dbg_acc[DBG_SLOTS] = {};
    unsigned long long rt0 = 0, ct0 = 0;
#endif
    do {
    // (the tile's coordinates are derived afresh from the round number: only that number and the Q
    // fragments cross from one tile to the next, everything else restarts from scalar registers)
    set_tile(tile_schedule(total, (int)gridDim.x, (int)blockIdx.x, __builtin_amdgcn_readfirstlane(round)));
    // Use the Q fragments once here: the compiler then waits for their loads before the loop instead
    // of inside it, where its vmcnt(0) would also wait for the K/V copies issued a moment earlier.
    // (The Q loads were issued after the copies of the prologue, so this wait also covers stages -1, 0, 1.)
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) asm volatile("" :: "v"(Qf[qb][kk]));
    wait_vmcnt<0>();
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        m_run[qb] = m_none;                     // (see launch)
        neg_mc[qb] = -m_none * scale_log2e;
        L[qb] = f32x4(0.f);
#pragma unroll
        for (int fb = 0; fb < FB; ++fb) O[fb][qb] = f32x4(0.f);
    }
    __builtin_amdgcn_s_barrier();               // stages -1, 0, 1 are complete for every wave
#ifdef ATTN_TIMING
    rt0 = __builtin_amdgcn_s_memrealtime(); ct0 = __builtin_readcyclecounter();
#endif
    // Each group's steady state is one loop with a single code path (the first and last tile and the
    // idle tail of a causal wave are peeled off), so the accumulators stay in place across iterations.
    constexpr std::integral_constant<int, 0> WHOLE{};
    constexpr std::integral_constant<int, 1> FIRST_HALF{};
    constexpr std::integral_constant<int, 2> SECOND_HALF{};
    if (NG == 3 && group == 1) {
        // the middle group of three, iteration j: second half of C_j, then [U_j, T_{j+1}], then the first half of
        // C_{j+1}; both contractions read stage j.  Its burst falls between those of the first group (right after
        // the barrier) and of the last (after its whole softmax): three bursts per SIMD and tile, back to back.
        mfma_burst(std::false_type{}, std::true_type{}, stage_ptr(-1));                  // T_0
        softmax_tile(0, std::false_type{}, FIRST_HALF, std::true_type{});
        int j = 0;
        if (j + 1 < nt_w) {
            do {                                // bottom-tested: see group A
                wait_stage(j);
                if (j + 2 < nt) issue_stage(j + 2);
                softmax_tile(j, std::false_type{}, SECOND_HALF, std::false_type{});
                mfma_burst(std::true_type{}, std::true_type{}, stage_ptr(j));
                softmax_tile(j + 1, std::false_type{}, FIRST_HALF, std::false_type{});
            } while (++j + 1 < nt_w);
        }
        wait_stage(j);                                                                   // j == nt_w - 1
        if (j + 2 < nt) issue_stage(j + 2);
        softmax_tile(j, std::false_type{}, SECOND_HALF, std::false_type{});
        mfma_burst(std::true_type{}, std::false_type{}, stage_ptr(j));                   // U of the last tile
        for (++j; j < nt; ++j) {                                                         // idle tail of a causal wave
            wait_stage(j);
            if (j + 2 < nt) issue_stage(j + 2);
        }
        finish_tile();
    } else if (!group_b) {
        // group A, iteration j: [U_{j-1}, T_j] then C_j; both contractions read stage j-1
        wait_stage(0);
        mfma_burst(std::false_type{}, std::true_type{}, stage_ptr(-1));                  // T_0
        fetch_ahead(stage_ptr(0));
        if (2 < nt) issue_stage(2);
        softmax_tile(0, std::false_type{}, WHOLE, std::true_type{});
        auto iter_a = [&](int j, auto spread) __attribute__((always_inline)) {
            TSTAMP(t0);
            wait_stage(j);
            TSTAMP(t1);
            mfma_burst(std::true_type{}, std::true_type{}, stage_ptr(j - 1));
            fetch_ahead(stage_ptr(j));
            TSTAMP(t2);
            if (!decltype(spread)::value && j + 2 < nt) issue_stage(j + 2);
            TSTAMP(t3);
            softmax_tile(j, spread, WHOLE, std::false_type{});
            TSTAMP(t4);
            TACC(0, t0, t1); TACC(1, t1, t2); TACC(2, t2, t3); TACC(3, t3, t4);
        };
        // (bottom-tested on purpose: with the exit test at the top the accumulators' loop-carried
        // value is also live on the exit edge, the first MFMA of an iteration then cannot update it
        // in place, and the compiler copies all 64 accumulator registers back every iteration)
        int j = 1;
        // iterations whose stage j + 2 exists and lies wholly inside the sequence spread its copies
        const int j_spread = ATTN_COPIES_IN_SOFTMAX ? min(nt_w, min(nt - 2, N / BN - 3)) : 0;
        if (j < j_spread) {
            do {
                iter_a(j, std::true_type{});
            } while (++j < j_spread);
        }
        if (j < nt_w) {
            do {
                iter_a(j, std::false_type{});
            } while (++j < nt_w);
        }
        if (j < nt) wait_stage(j);                                                       // j == nt_w
        mfma_burst(std::true_type{}, std::false_type{}, stage_ptr(j - 1));               // U of the last tile
        if (j < nt && j + 2 < nt) issue_stage(j + 2);
        for (++j; j < nt; ++j) {                                                         // idle tail of a causal wave
            wait_stage(j);
            if (j + 2 < nt) issue_stage(j + 2);
        }
        if constexpr (KS == 2) merge_groups(std::false_type{});
        finish_tile();
    } else if (KS == 2 && nt_w == 0) {
        // no key of this wave's share is visible to its rows: it only copies
        for (int j = 0; j < nt; ++j) {
            wait_stage(j);
            if (j + 2 < nt) issue_stage(j + 2);
        }
        if constexpr (KS == 2) merge_groups(std::true_type{});
        finish_tile();
    } else {
        // group B, iteration j: C_j then [U_j, T_{j+1}]; both contractions read stage j
        mfma_burst(std::false_type{}, std::true_type{}, stage_ptr(-1));                  // T_0
        auto iter_b = [&](int j, auto spread) __attribute__((always_inline)) {
            TSTAMP(t0);
            wait_stage(j);
            fetch_ahead(stage_ptr(j));
            TSTAMP(t1);
            if (!decltype(spread)::value && j + 2 < nt) issue_stage(j + 2);
            TSTAMP(t2);
            softmax_tile(j, spread, WHOLE, std::false_type{});
            TSTAMP(t3);
            mfma_burst(std::true_type{}, std::true_type{}, stage_ptr(j));
            TSTAMP(t4);
            TACC(0, t0, t1); TACC(2, t1, t2); TACC(3, t2, t3); TACC(1, t3, t4);
        };
        int j = 0;
        const int j_spread = ATTN_COPIES_IN_SOFTMAX ? min(nt_w - 1, min(nt - 2, N / BN - 3)) : 0;
        if (j < j_spread) {
            do {
                iter_b(j, std::true_type{});
            } while (++j < j_spread);
        }
        if (j + 1 < nt_w) {
            do {
                iter_b(j, std::false_type{});
            } while (++j + 1 < nt_w);
        }
        wait_stage(j);                                                                   // j == nt_w - 1
        fetch_ahead(stage_ptr(j));
        if (j + 2 < nt) issue_stage(j + 2);
        softmax_tile(j, std::false_type{}, WHOLE, std::false_type{});
        mfma_burst(std::true_type{}, std::false_type{}, stage_ptr(j));                   // U of the last tile
        for (++j; j < nt; ++j) {                                                         // idle tail of a causal wave
            wait_stage(j);
            if (j + 2 < nt) issue_stage(j + 2);
        }
        if constexpr (KS == 2) merge_groups(std::true_type{});
        finish_tile();
    }
    } while (more);
#ifdef ATTN_TIMING
    if (blockIdx.x < DBG_WGS && lane == 0) {
        dbg_acc[5] = nt;
        dbg_acc[6] = __builtin_amdgcn_s_memrealtime() - rt0;   // 100 MHz ticks
        dbg_acc[7] = __builtin_readcyclecounter() - ct0;
#if ATTN_TIMING == 1
        dbg_acc[0] = rt0;                                        // absolute start of the main loop
        dbg_acc[1] = __builtin_amdgcn_s_getreg((31 << 11) | (0 << 6) | 4);    // HW_ID
        dbg_acc[2] = __builtin_amdgcn_s_getreg((31 << 11) | (0 << 6) | 20);   // XCC_ID
        dbg_acc[3] = logical;
        dbg_acc[4] = rt_kernel_entry;
#endif
        for (int i = 0; i < DBG_SLOTS; ++i) attn_dbg[(blockIdx.x * 8 + wave) * DBG_SLOTS + i] = dbg_acc[i];
    }
#endif

#ifdef ATTN_TIMING
    if (blockIdx.x < DBG_WGS && lane == 0) attn_dbg[(blockIdx.x * 8 + wave) * DBG_SLOTS + 5] = __builtin_amdgcn_s_memrealtime();
#endif
}

template <int DTYPE, int D, int NW, int MB, int BN, int STAGES, bool CAUSAL, bool PERSIST, int KS = 1>
int launch(const AttnLaunchArgs& a)
{
    constexpr int BM = NW * MB * 32 / KS;
    constexpr int smem = STAGES * 2 * BN * D * 2;
    auto kern = attn_fwd_kernel<DTYPE, D, NW, MB, BN, STAGES, CAUSAL, PERSIST, KS>;
    static PerDeviceOnce once;                  // the attribute belongs to the (kernel, device) pair
    const int dev = once.prepare(reinterpret_cast<const void*>(kern), smem);
    if (dev < 0) return -1;
    const int nqt = (a.N + BM - 1) / BM;
    const long long total = (long long)nqt * a.B * a.H;
    // Persistent launch: as many workgroups as the chip holds at once (one per CU at d = 128: the LDS
    // ring takes 128 KiB), each walking its share of the tile schedule.
    long long grid = total;
    if (PERSIST) {
        const int cus = once.compute_units(dev);
        if (cus < 8) return -1;
        const long long resident = (long long)cus * ((160 * 1024) / smem);
        if (grid > resident) grid = resident;
    }
    const float log2e = 1.4426950408889634f;
    const uint16_t* q = (const uint16_t*)a.q;
    const uint16_t* k = (const uint16_t*)a.k;
    const uint16_t* v = (const uint16_t*)a.v;
    uint16_t* o = (uint16_t*)a.o;
    float* lse = a.lse;
    int N = a.N, nqt_arg = nqt, total_arg = (int)total;
    float scale = a.scale, scale_log2e = a.scale * log2e;
    // The softmax reference before the first finite score.  Not -inf: where the first keys that a wave works on all score
    // -inf, (-inf) - (-inf) would turn the row into NaN.  The most negative float whose scaled value is finite gives those
    // keys the weight exp2(-inf) = 0 and moves to the first finite score.
    float m_none = scale_log2e > 1.f ? -0x1.fffff0p127f / scale_log2e : -__FLT_MAX__;
    void* args[] = {&q, &k, &v, &o, &lse, &N, &nqt_arg, &total_arg, &scale, &scale_log2e, &m_none};
    // the launch's own status, not hipGetLastError(): that one also reports stale errors of unrelated calls
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3((unsigned)grid), dim3(NW * 64),
                                         args, smem, (hipStream_t)a.stream);
    return e == hipSuccess ? 0 : -1;
}

// Whether this build has the form that splits keys, and the rule.
constexpr bool has_split(int d) { return ATTN_KEY_SPLIT && (d == 64 || ATTN_CFG_NW == 8) && ATTN_CFG_STAGES == 4 && !(ATTN_CFG_PIPE && d == 128); }
bool splits_keys(int d, int N, long long heads, bool causal) { return has_split(d) && attn_splits_keys(d, N, heads, causal, false); }

template <int DTYPE, int D>
int launch_d(const AttnLaunchArgs& a)
{
    constexpr int NW = D == 128 ? ATTN_CFG_NW : 8, MB = D == 64 ? ATTN_CFG_MB_D64 : ATTN_CFG_MB, BN = ATTN_CFG_BN, STAGES = ATTN_CFG_STAGES;
    if (a.rows ? a.rows == 128 : splits_keys(D, a.N, (long long)a.B * a.H, a.causal != 0))
        return a.causal ? launch<DTYPE, D, 8, 1, BN, STAGES, true, false, 2>(a) : launch<DTYPE, D, 8, 1, BN, STAGES, false, false, 2>(a);
    // When the persistent form is used.  d = 128: always; with the mask it balances the tile lengths, and the next prologue
    // goes on under the epilogue (4 x 16 heads, N = 4096, no mask, bf16: 447.7 -> 445.6 us, N = 16384, 16 heads, fp16 1773 -> 1767;
    // 16 x 16 heads, N = 512, 43.3 -> 43.4).  d = 64: with the mask (61 -> 58 us at 256 heads, N = 1024); without it two workgroups
    // share a CU and cover each other's prologue and epilogue, and the next tile's Q fragments would cost the registers that
    // let them co-reside.
    if (D == 128 && ATTN_PERSISTENT)
        return a.causal ? launch<DTYPE, D, NW, MB, BN, STAGES, true, true>(a) : launch<DTYPE, D, NW, MB, BN, STAGES, false, true>(a);
    if (D == 64 && ATTN_PERSISTENT_D64 && a.causal) return launch<DTYPE, D, NW, MB, BN, STAGES, true, true>(a);
    return a.causal ? launch<DTYPE, D, NW, MB, BN, STAGES, true, false>(a) : launch<DTYPE, D, NW, MB, BN, STAGES, false, false>(a);
}

}  // namespace

int attn_launch(const AttnLaunchArgs& a)
{
    if (ATTN_CFG_PIPE && a.d == 128) return attn_pipe_launch(a);
    if (a.dtype == 0) return a.d == 128 ? launch_d<0, 128>(a) : launch_d<0, 64>(a);
    return a.d == 128 ? launch_d<1, 128>(a) : launch_d<1, 64>(a);
}

#ifdef ATTN_TIMING
extern "C" int attn_dbg_read(unsigned long long* host, int n)
{
    return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(attn_dbg), sizeof(unsigned long long) * n);
}
#endif

int attn_launch_call_rows(int d, int N, long long heads, int causal)
{
    if (splits_keys(d, N, heads, causal != 0)) return 128;
    return attn_launch_tile_param(d, causal, 0);
}

bool attn_launch_has_rows(int d, int causal, int rows) { return rows == attn_launch_tile_param(d, causal, 0) || (rows == 128 && has_split(d)); }

int attn_launch_tile_param(int d, int causal, int which)
{
    (void)causal;
    if (d != 64 && d != 128) return -1;
    if (ATTN_CFG_PIPE && d == 128) {
        switch (which) {
            case 0: return 256;
            case 1: return 64;
            case 2: return 5;
            case 3: return ATTNP_CFG_NW * 64;
            default: return -1;
        }
    }
    switch (which) {
        case 0: return (d == 128 ? ATTN_CFG_NW : 8) * (d == 64 ? ATTN_CFG_MB_D64 : ATTN_CFG_MB) * 32;
        case 1: return ATTN_CFG_BN;
        case 2: return ATTN_CFG_STAGES;
        case 3: return (d == 128 ? ATTN_CFG_NW : 8) * 64;
        default: return -1;
    }
}
