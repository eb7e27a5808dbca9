// Which GEMM kernel takes which rows of a problem: host arithmetic only, no HIP.
#pragma once

#include <stdint.h>

namespace rs {

enum class GemmTile { Slim64x64, Slim128x64, Slim128x128, Slim256x128, Ring, Direct, Persistent };

// The kernel for the first `rows` rows; rows < M: the rows behind them are a problem of their own.
struct GemmChoice {
    GemmTile tile;
    int64_t rows;
};

// Choice by shape: the smallest tile of 64 x 64, 128 x 64, 128 x 128, 256 x 128 (slim kernels) and 256 x 256
// (persistent kernel) that gives every CU at most one workgroup.  A workgroup streams its operands at
// the pace of one CU whatever else runs, so a smaller tile is faster as long as it does not put two
// workgroups on some CUs; at 48 slices of K the steps are 12 / 20 / 24 / 34 / 59 us per launch (768 x 3072).
// Chains of the four layers of a block, sizes on both sides of the steps (us per layer against the
// next smaller / larger tile): 768 x 3072 at 1182 rows (228 tiles of 64 x 64) -22.5 / -16.0 against the 128 x 128
// ring kernel, at 1576 rows (300) -12.0 / -15.2; at 3152 rows (150 of 128 x 128) -11.1 / -0.3; at 8471
// rows (204 of 256 x 128) -4.5 / -24.7; 384 x 1152 at 12608 rows (250 of 256 x 256) 18.9 us persistent, 24 ring.
// Beyond one round:
//  - K <= 384: a tile is mostly epilogue; the ring kernels (two workgroups per CU, one's epilogue under the
//    other's K loop): 1536 x 384 at 25216 rows -5 us of 62 against the persistent kernel.
//  - K < 2048 and up to 1.45 rounds of 256 x 256 tiles: the 256 x 128 tiles, whose last round costs half as much
//    (768 x 768 at 25216 rows -7 us of 53, 2304 x 768 at 10047 rows -4 of 50; at 1.59 rounds +5).
//  - otherwise the persistent kernel; with K >= 2048 and a last round at most half full the rows that make up
//    whole rounds go to it and the rows behind them to the tile that suits them, in a second launch
//    (a round is long there: 768 x 3072 at 50432 rows -19 us of 260).  A row panel of more tiles than the whole
//    rounds hold (N > 256 * cus) cannot be cut that way and stays whole.
inline GemmChoice gemm_choose(int64_t M, int64_t N, int K, int64_t cus) {
    auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    if (tiles(64, 64) <= cus) return {GemmTile::Slim64x64, M};
    if (tiles(128, 64) <= cus) return {GemmTile::Slim128x64, M};
    if (tiles(128, 128) <= cus) return {GemmTile::Slim128x128, M};
    if (tiles(256, 128) <= cus) return {GemmTile::Slim256x128, M};
    const int64_t t = tiles(256, 256), rounds = t / cus, rem = t - rounds * cus;
    if (rounds == 0 || rem == 0) return {GemmTile::Persistent, M};
    if (K <= 384) return {GemmTile::Ring, M};
    if (K < 2048 && 100 * t <= 145 * cus) return {GemmTile::Slim256x128, M};
    if (K < 2048 || 2 * rem > cus) return {GemmTile::Persistent, M};
    const int64_t m1 = rounds * cus / ((N + 255) / 256) * 256;  // row panels that fill whole rounds: fewer than all of them
    return {GemmTile::Persistent, m1 > 0 ? m1 : M};
}

// The same for weights in fragment order (a block's layers; `res`: with a residual in the epilogue).  The small slim tiles as above; the
// direct kernel (128 x 256 tiles, two workgroups per CU) takes the place of most of what the ring and the persistent kernel
// do: its workgroups hand a free slot on, and a CU with only one runs it faster, so that a last round half full costs about
// half of one.  us, the best of the others / direct: 768 x 768 at 50432 rows 85 / 72, at 25216 48 / 38; 768 -> 3072 at 50432 287 / 242, at 6280 52 / 39;
// 384 -> 1536 at 50432 95 / 84, at 12608 37 / 29.
//  - up to one 256 x 128 slim tile per CU (eight waves, residual rows requested early): those.  Only without a residual, at 768 <= K < 1536
//    and more than 0.7 tiles per CU, the direct kernel where it too has at most one tile per CU.  slim / direct in a block: with
//    residual 768 x 768 at 9244 rows 18.0 / 19.4, 1024 x 1024 at 8036 22.4 / 23.1, 1344 -> 256 at 24600 25.3 / 28.1; without 768 -> 2304 at 3368
//    18.1 / 16.8, 1024 -> 3072 at 2064 19.5 / 18.5, but 1088 -> 832 at 9100 (288 direct tiles) 23.6 / 31.6, 832 x 832 there 19.7 / 27.3.
//  - N <= 128 beyond that: a 256-wide tile would be half empty or more.  The ring kernel's 128 x 128 tiles to K = 512, the slim tiles from there.
//    us, ring / slim / direct: 64 x 64 at 91520 rows 10.3 / 14.7 / 14.7, at 372288 32 / 39 / 42; 256 -> 64 at 91520 18.4 / 23.7 / 29.3; 128 x 128 at 75680
//    14.5 / 18.2 / 18.2; 448 -> 128 at 86840 25.4 / 30.1 / 35.2; 512 -> 128 at 300320 118 / 119 / 134; 1024 -> 128 at 165252 114 / 112 / 125; 2048 -> 64
//    at 121512 150 / 145 / 159.
//  - N is no multiple of 256 and the direct kernel would have more than two tiles per CU, the slim one at most two: slim.  slim /
//    direct: 1088 x 1088 at 13664 41.1 / 47.5, 832 -> 576 at 23564 39.8 / 43.8, 1280 -> 320 at 33000 41.8 / 50.7, 256 -> 1344 at 10944 21.3 / 24.0.
//  - K >= 2048 and a last round of 256 x 256 tiles at most a sixth full: a few tiles alone cost the direct kernel two thirds of a
//    round.  The rows of whole rounds go to the persistent kernel, those behind them to the tile that suits them, in a second launch.
//    us, cut / direct: 4096 -> 1024 at 16388 rows 130 / 145, 18000 136 / 147, 20000 (0.23) 159 / 150, 33200 249 / 272; 3072 -> 768 at 23000
//    103 / 115, 25216 (0.16) 112 / 116, 27392 (0.25) 137 / 124, 45568 202 / 213, 48000 (0.2) 213 / 215; 2560 -> 640 at 22000 89 / 96; 2048 -> 512 at
//    33000 82.5 / 84.4; 1792 -> 448 there 71.3 / 72.7, at 36000 76.2 / 75.1.  A row panel of more tiles than the whole rounds hold stays whole.
//  - K >= 1536 and a last round more than half full (0.6 below K = 3072): the persistent kernel, which moves two thirds of the
//    bytes per flop.  persistent / direct: 3072 -> 768 at 41216 rows (0.89) 170 / 182, 33536 (0.54) 155 / 167, 21760 89.5 / 90.2, 12552 63.5 / 71.9, 28800
//    (0.32) 147 / 124; 1536 -> 384 at 25216 40.1 / 44.0, 50432 (0.54) 91 / 83; 2048 -> 512 at 50000 (0.53) 129 / 123; 2560 -> 640 at 33684 (0.55) 139 / 136.
inline GemmChoice gemm_choose_frag(int64_t M, int64_t N, int K, int64_t cus, bool res) {
    auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    if (tiles(64, 64) <= cus) return {GemmTile::Slim64x64, M};
    if (tiles(128, 64) <= cus) return {GemmTile::Slim128x64, M};
    if (tiles(128, 128) <= cus) return {GemmTile::Slim128x128, M};
    const int64_t slim = tiles(256, 128), direct = tiles(128, 256);
    if (slim <= cus) return {!res && K >= 768 && K < 1536 && 10 * slim > 7 * cus && direct <= cus ? GemmTile::Direct : GemmTile::Slim256x128, M};
    if (N <= 128) return {K <= 512 ? GemmTile::Ring : GemmTile::Slim256x128, M};
    if (slim <= 2 * cus && direct > 2 * cus) return {GemmTile::Slim256x128, M};
    const int64_t t = tiles(256, 256), rem = t % cus;
    if (K >= 2048 && t > cus && rem > 0 && 6 * rem <= cus) {
        const int64_t m1 = (t - rem) / ((N + 255) / 256) * 256;  // row panels that fill whole rounds
        if (m1 > 0) return {GemmTile::Persistent, m1};
    }
    return {K >= 1536 && (rem == 0 || 10 * rem > (K < 3072 ? 6 : 5) * cus) ? GemmTile::Persistent : GemmTile::Direct, M};
}

// fp32: the rows of one launch, in whole tiles of `bm` x 64: it has 256 threads per tile, tiles rounded up to a multiple of
// 8, and holds less than 2^32 of them.
inline int64_t gemm_f32_launch_rows(int N, int bm) { return (((int64_t)1 << 24) - 8) / ((N + 63) / 64) * bm; }

// fp32: tiles shared by the waves (64 x 64), with 3 or 4 workgroups per CU, or (0) 32 x 64 tiles with K split over the waves.  Same results
// either way.
//  - The shared tiles where they fill the chip: four rounds of one tile per CU, 1.5 where K is short (the sum through LDS of the split tiles
//    is a large part of a tile then), and in between where the last round is at least 0.9 full, a tile being a long unit of work at long K.
//    us, shared / split (tiles in brackets): K = 192: 3152 x 576 (450) 9.5 / 12.0, 10088 x 192 (474) 9.8 / 12.5, 6304 x 192 (297) 9.3 / 9.7, 1576 x 768
//    with GELU (300) 11.9 / 11.8; K = 768: 10088 x 192 (474) 27.7 / 30.0, 20000 x 192 (939) 50.6 / 56.2, 12608 x 192 (591) 38.7 / 36.8, 8192 x 192 (384)
//    27.0 / 23.4, 788 x 192 (39) 15.9 / 9.5; 3072 -> 768 at 4000 rows (756) 143 / 150, at 2000 (384) 97 / 77.
//  - Not a single column of them at long K between four and 5.5 rounds, which reads its rows in 128-byte pieces that no other tile
//    shares: 2048 -> 64 at 76800 rows (1200) 247 (three per CU) / 215, at 82560 256 / 232, at 96000 262 / 259; at 48640 (760) 121 / 146, at 114560 (1790) 278 / 290.
//  - Three per CU between four and five rounds, where a fourth leaves a lone tile behind, and at long K.  us, three / four: 2048 -> 2304
//    at 2176 rows (1224) 161 / 187, 768 -> 192 at 25600 (1200) 66 / 76, 1024 x 1024 at 4800 (1200) 83 / 91, 4096 -> 1024 at 7168 (1792) 433 / 473;
//    beyond, at K = 768 and 192, three cost 1 to 2 and 5 %.
struct GemmF32Choice {
    int per_cu;
};
inline GemmF32Choice gemm_f32_choose(int64_t M, int N, int K, int64_t cus) {
    const int64_t tiles = ((M + 63) / 64) * (N / 64);
    const bool fills = tiles >= 4 * cus || (K <= 384 && 2 * tiles >= 3 * cus) || (tiles > cus && 10 * tiles >= 9 * cus * ((tiles + cus - 1) / cus));
    if (!fills || (N == 64 && K > 1024 && tiles > 4 * cus && 2 * tiles < 11 * cus)) return {0};
    return {tiles > 4 * cus && (tiles < 5 * cus || K > 1024) ? 3 : 4};
}

}  // namespace rs
