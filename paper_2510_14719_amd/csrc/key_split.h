// Which attention calls take 128-row query tiles with the keys of a tile shared out between the halves of a workgroup (KS = 2
// in the kernels) instead of 256-row tiles: the split ones where the chip is not full, or would be filled unevenly.
//
// A split tile takes 0.55 to 0.75 of the time of a whole one, and there are up to twice as many.  So they pay
//  * while they fit the chip in one round, one workgroup per CU (very short E4M3 rows excepted: the exchange at the end costs more);
//  * where the rounds that they take are cheaper than the rounds of whole tiles (257 whole tiles are two rounds, 514 split
//    ones three of 0.6 each), above all where the last 128 rows of a sequence leave half of a whole tile empty;
//  * under the mask, where whole tiles in one round leave most CUs waiting for those with the longest rows, and whole tiles in
//    two are paired by their number only.  Workgroups go to the XCDs in turn and every XCD walks a contiguous
//    range of tiles, heads from long rows to short: where the range is half a head, one head or two (4, 8 or 16 heads) split tiles in two
//    rounds always pair well, else mostly while the second round is short or the rows are many.
//
// Measured on MI355X, whole / split tiles, us, some on either side of each line (d 128 unless stated; more in tests/test_key_split.py):
//   one round    16-bit  2 heads, N 128 8.2 / 7.8
//                E4M3    65 heads, N 239 9.0 / 8.3; 127 heads, N 148 7.8 / 8.5; 132 heads, N 111 6.2 / 7.2; 66 heads, N 320 10.5 / 11.0;
//                        causal: 94 heads, N 227 9.3 / 8.7; 47 heads, N 399 11.5 / 9.7; 101 heads, N 123 6.6 / 7.4;
//                        d 64: 100 heads, N 256 7.0 / 6.1, N 128 4.9 / 5.1
//   rounds       16-bit  64 heads, N 1024 42 / 50; d 64: 42 heads, N 1905 64.8 / 57.9;
//                        25 heads, N 4510 153 / 167; 340 heads, N 123 9.2 / 8.2; 333 heads, N 300 22.2 / 19.9; 348 heads, N 485 32.1 / 37.4
//                E4M3    16 heads, N 5484 162 / 138; 23 heads, N 4510 135 / 157; 28 heads, N 4999 231 / 220; d 64: 131 heads, N 345 15.9 / 12.7
//   mask         16-bit  8 heads, N 7168 144 / 114; 16 heads, N 3584 76 / 64; 17 heads, N 3840 85 / 106; 9 heads, N 6144 125 / 142;
//                        11 heads, N 6575 238 / 163; 21 heads, N 4739 201 / 159; 40 heads, N 3150 106 / 120
//                        d 64: 14 heads, N 2816 50 / 43; 264 heads, N 80 11.4 / 7.0; 285 heads, N 1926 316 / 212; 2061 heads, N 69 44 / 25;
//                        256 heads, N 1024 (four whole rounds, paired) 58 / 68
//                E4M3    8 heads, N 7424 105 / 72; 18 heads, N 3584 56 / 67; 14 heads, N 7599 196 / 146; 15 heads, N 4833 83 / 86;
//                        d 64: 64 heads, N 4096 156 / 138
#pragma once

#include "tile_schedule.h"                      // CHIP_CUS

// A grid has less than 2^32 threads in a dimension, 512 per split tile.  Whole tiles under the mask at d = 64 are persistent and so
// know no such limit: beyond it the calls are theirs.
constexpr long long MAX_SPLIT_TILES = (1ll << 32) / 512 - 1;

// heads = batch size x heads.
inline bool attn_splits_keys(int d, int N, long long heads, bool causal, bool fp8)
{
    const long long split = (N + 127LL) / 128 * heads, per_head = (N + 255LL) / 256, whole = per_head * heads;   // tiles
    auto rounds = [](long long tiles, long long slots) { return (tiles + slots - 1) / slots; };
    // split tiles at `cost` of a whole one each
    auto fewer_rounds = [&](double cost) { return cost * rounds(split, CHIP_CUS) < 0.97 * rounds(whole, CHIP_CUS); };

    if (split > MAX_SPLIT_TILES) return false;
    if (split <= CHIP_CUS) {
        if (!fp8) return true;
        if (d == 64) return N > 128;                                     // (a stage holds 128 keys)
        if (causal) return N > 512 || (N > 128 && split <= CHIP_CUS * 3 / 4);
        return N > 320 || (N > 192 && split <= CHIP_CUS * 5 / 8);
    }
    // (Sequences of 513 to 1536, in more than one round, keep whole tiles throughout: some would gain as much as their
    // neighbours, e.g. d 64 and the mask 108 heads, N 544 24.8 / 17.4, but the tests of whole tiles with ragged ends run at these lengths.)
    if (!causal) {
        if (fp8 && d == 64) return (N > 1536 || (N > 256 && N <= 512)) && fewer_rounds(N > 512 ? 0.60 : 0.70);
        if (fp8) return N > 2048 && fewer_rounds(0.58);
        if (N <= 128) return d == 64 || whole <= 2 * CHIP_CUS;           // (half of a whole tile would be empty)
        if (d == 64) return (N > 1536 || (N > 256 && N <= 512)) && fewer_rounds(0.61);
        return N > 1536 && fewer_rounds(0.65);
    }
    if (d == 64 && fp8) return N >= 2048 && split <= 8 * CHIP_CUS;       // (two workgroups per CU)
    if (whole > CHIP_CUS) {
        if (N > 512 && N <= 1536) return false;
        // d = 64: the persistent whole tiles are one to a CU and in batches of 512, the split ones two to a CU.  Full batches whose long and
        // short tiles pair evenly are the exception.
        if (d == 64) return per_head < 2 || (per_head & (per_head - 1)) != 0 || 2 * CHIP_CUS * rounds(whole, 2 * CHIP_CUS) - whole > 8;
        if (fp8) return N > 2048 && whole > CHIP_CUS * 3 / 2 && whole <= CHIP_CUS * 15 / 8;
        return N <= 128 ? whole <= 2 * CHIP_CUS : N > 1536 && whole <= CHIP_CUS * 11 / 6;
    }
    if (N <= 2048 || split > 2 * CHIP_CUS) return false;
    if (d == 64 || heads == 4 || heads == 8 || heads == 16) return true;
    if (split <= CHIP_CUS * 5 / 4) return true;
    if (fp8) return N > 7168 || (N > 4096 && split <= 400) || (N > 3072 && split <= 360);
    return N > 4500 && split <= 360;
}
