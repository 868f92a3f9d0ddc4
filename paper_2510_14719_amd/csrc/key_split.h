// Which attention calls take 128-row query tiles with the keys of a tile shared out between the halves of a workgroup (KS = 2
// in the kernels) instead of 256-row tiles: the split ones where the chip is not full, or would be filled unevenly.
//
// A split tile takes 0.5 to 0.9 of the time of a whole one (the exchange at its end weighs on short rows), and there are up to twice
// as many.  So they pay
//  * while they fit the chip in one round, one workgroup per CU (very short E4M3 rows excepted);
//  * without the mask, where the rounds that they take are cheaper than the rounds of whole tiles (257 whole tiles are two rounds, 514 split
//    ones three): `cost` is the time of one of their rounds over one of whole tiles, fitted to 300 calls of 64 to 9000 keys;
//  * under the mask, where whole tiles in one round leave most CUs waiting for those with the longest rows, and whole tiles in
//    two are paired by their number only.  Workgroups go to the XCDs in turn and every XCD walks a contiguous
//    range of tiles, heads from long rows to short: where the range is half a head, one head or two (4, 8 or 16 heads) split tiles in two
//    rounds always pair well, else mostly while the second round is short or the rows are many.
//
// Measured on MI355X, whole / split tiles, us, some on either side of each line (d 128 unless stated, N(0,1) inputs; more in
// tests/test_key_split.py):
//   one round    16-bit  2 heads, N 128 7.9 / 7.4
//                E4M3    65 heads, N 239 9.1 / 8.5; 127 heads, N 148 7.8 / 8.5; causal: 100 heads, N 150 8.0 / 7.7; 101 heads, N 123 6.7 / 7.4;
//                        d 64: 100 heads, N 200 7.1 / 6.1, N 100 4.9 / 5.1
//   no mask      16-bit  70 heads, N 865 51 / 35; 109 heads, N 722 47 / 46; 77 heads, N 1944 159 / 166; 64 heads, N 1024 32 / 39;
//                        N <= 128: 268 heads, N 71 15.3 / 14.1; 900 heads, N 96 31.7 / 30.4; 1500 heads, N 128 58 / 61; 400 heads, N 64 11.7 / 12.3; 700 heads, N 20 14.7 / 13.8;
//                        the same with the mask: 900 heads, N 66 29.5 / 27.9; 400 heads, N 64 12.2 / 12.6
//                        d 64: 187 heads, N 596 35 / 29; 174 heads, N 775 44 / 43; 85 heads, N 1154 41 / 47; 340 heads, N 123 9.6 / 8.9
//                E4M3    44 heads, N 1390 51 / 35; 67 heads, N 1140 43 / 44; 120 heads, N 583 29 / 33;
//                        d 64: 73 heads, N 841 28 / 20; 106 heads, N 759 25 / 27
//   mask         16-bit  8 heads, N 7168 144 / 100; 16 heads, N 3584 75 / 57; 17 heads, N 3840 82 / 101; 9 heads, N 6144 122 / 136;
//                        11 heads, N 6575 230 / 159; 21 heads, N 4739 191 / 151; 40 heads, N 3150 109 / 122; 140 heads, N 343 25 / 21;
//                        whole tiles between two rounds and many are a matter of their number: 96 heads, N 947 38 / 50; 108 heads, N 1095 83 / 63;
//                        21 heads, N 7252 403 / 292; 56 heads, N 6057 484 / 526 (whole ones are taken)
//                        d 64: 73 heads, N 847 36 / 18; 266 heads, N 1285 158 / 102; 600 heads, N 437 54 / 55; 285 heads, N 1926 310 / 218;
//                        22 heads, N 1729 33 / 28; 92 heads, N 393 11.7 / 12.4; 256 heads, N 1024 (four whole rounds, paired) 61 / 70
//                E4M3    8 heads, N 7424 103 / 65; 18 heads, N 3584 53 / 61; 14 heads, N 7599 179 / 132; 15 heads, N 4833 79 / 83;
//                        d 64: 64 heads, N 4096 151 / 141; 50 heads, N 1280 20 / 24
#pragma once

#include "tile_schedule.h"                      // CHIP_CUS

// A grid has less than 2^32 threads in a dimension, 512 per split tile.  Whole tiles under the mask at d = 64 are persistent and so
// know no such limit: beyond it the calls are theirs.
constexpr long long MAX_SPLIT_TILES = (1ll << 32) / 512 - 1;

// heads = batch size x heads.
inline bool attn_splits_keys(int d, int N, long long heads, bool causal, bool fp8)
{
    const long long split = (N + 127LL) / 128 * heads, per_head = (N + 255LL) / 256, whole = per_head * heads;   // tiles
    auto rounds = [](long long tiles) { return (tiles + CHIP_CUS - 1) / CHIP_CUS; };

    if (split > MAX_SPLIT_TILES) return false;
    if (split <= CHIP_CUS) return !fp8 || N > (d == 64 || causal ? 128 : 192);
    // One tile per head, half of it or more empty where it is a whole one: split tiles while the rounds are few.  (From 33 to 64
    // keys, a single tile of keys to share out, whole tiles are the faster ones.)
    if (!fp8 && d == 128 && N <= 128) return (N <= 32 || N > 64) && whole <= 4 * CHIP_CUS;
    if (!causal) {
        if (!fp8 && N <= 128) return true;
        const double cost = fp8 ? (d == 64 ? 0.51 : 0.525) + 230. / (N + 300) : d == 64 ? 0.56 + 10. / N : 0.60 + 45. / N;
        return cost * rounds(split) < 0.97 * rounds(whole);
    }
    if (d == 64 && fp8) return N >= 2048 && split <= 8 * CHIP_CUS;       // (two workgroups per CU)
    if (whole > CHIP_CUS) {
        // d = 64: the persistent whole tiles are one to a CU and in batches of 512, the split ones two to a CU.  Full batches whose long and
        // short tiles pair evenly are the exception.
        if (d == 64) return per_head < 2 || (per_head & (per_head - 1)) != 0 || (whole + 2 * CHIP_CUS - 1) / (2 * CHIP_CUS) * (2 * CHIP_CUS) - whole > 8;
        if (fp8) return N > 2048 && whole > CHIP_CUS * 3 / 2 && whole <= CHIP_CUS * 15 / 8;
        return (N > 128 && split <= 2 * CHIP_CUS) || (N > 1536 && whole <= CHIP_CUS * 11 / 6);
    }
    if (d == 64) return N > 512;
    if (N <= 2048 || split > 2 * CHIP_CUS) return false;
    if (heads == 4 || heads == 8 || heads == 16 || split <= CHIP_CUS * 5 / 4) return true;
    if (fp8) return N > 7168 || (N > 4096 && split <= 400) || (N > 3072 && split <= 360);
    return N > 4500 && split <= 360;
}
