// Which attention calls take 128-row query tiles with the keys of a tile shared out between the halves of a workgroup (KS = 2
// in the kernels) instead of 256-row tiles: the split ones where the chip is not full, or would be filled unevenly.
//
// A split tile takes a bit more than half the time of a whole one, and there are twice as many.  So they pay while they fit
// the chip in one round, one workgroup per CU.  With the mask and long rows the 256-row tiles of one round leave most CUs waiting
// for those with the longest rows; split tiles in two rounds even that out where short tiles of the first round make room
// for long ones of the second.  Workgroups go to the XCDs in turn and every XCD walks a contiguous range of tiles, heads from long
// rows to short: where the range is half a head, one head or two (4, 8 or 16 heads) the rounds always pair well, else mostly while
// the second round is short or the rows are many.
//
// Measured on MI355X, whole / split tiles, us (d 128 unless stated; more in the table of tests/test_key_split.py):
//   16-bit   1 head, N 16384 296 / 193; 32 heads, N 1024 30 / 25; 2 heads, N 128 8.2 / 7.8, d 64 5.4 / 5.2; 64 heads, N 1024 42 / 50
//            causal: 8 heads, N 7168 144 / 114; 16 heads, N 3584 76 / 64; 4 heads, N 15616 315 / 306; 12 heads, N 2816 56 / 41;
//            17 heads, N 3840 85 / 106; 9 heads, N 6144 125 / 142; 21 heads, N 2560 55 / 62; d 64: 14 heads, N 2816 50 / 43;
//            28 heads, N 2048 38 / 40
//   E4M3     1 head, N 16384 218 / 121; d 64: 100 heads, N 256 7.0 / 6.1, 100 heads, N 128 4.9 / 5.1; 85 heads, N 320 10.7 / 11.5;
//            85 heads, N 352 12.3 / 11.1; 64 heads, N 1024 24 / 33
//            causal: 85 heads, N 320 11.6 / 12.9; 64 heads, N 448 13.1 / 14.5; 51 heads, N 577 15.4 / 15.4; 8 heads, N 7424 105 / 72;
//            18 heads, N 3584 56 / 67; 5 heads, N 10325 141 / 118; d 64: 64 heads, N 4096 156 / 138; 64 heads, N 2048 57 / 52
#pragma once

#include "tile_schedule.h"                      // CHIP_CUS

// heads = batch size x heads.
inline bool attn_splits_keys(int d, int N, long long heads, bool causal, bool fp8)
{
    const long long tiles = (N + 127LL) / 128 * heads;                   // 128-row tiles
    if (tiles <= CHIP_CUS) {
        if (!fp8) return true;
        if (d == 64) return N > 128;                                     // (a stage holds 128 keys)
        if (N <= 256) return false;
        return N > (causal ? 512 : 320) || tiles <= (causal && N > 320 ? 128 : 64);   // (the exchange spills at d = 128)
    }
    if (!causal) return false;
    if (d == 64 && fp8) return N >= 2048 && tiles <= 8 * CHIP_CUS;       // (two workgroups per CU, no spills)
    if (N <= 2048 || tiles > 2 * CHIP_CUS) return false;
    if (d == 64 || heads == 4 || heads == 8 || heads == 16) return true;
    if (tiles <= CHIP_CUS * 5 / 4) return true;
    if (fp8) return N > 7168 || (N > 4096 && tiles <= 400) || (N > 3072 && tiles <= 360);
    return (N > 4500 && tiles <= 360) || (N + 255LL) / 256 * heads > CHIP_CUS;        // (or whole tiles take two rounds as well)
}
