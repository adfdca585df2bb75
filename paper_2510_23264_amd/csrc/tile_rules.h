// Which tile a matrix product takes.  Host arithmetic without any GPU type, so that tests can compile it alone.
#pragma once
#include <cmath>

namespace pahq {

// Tiles of bm x bn of n_probs problems of M x N, and how often they fill 256 compute units.
inline long long tile_count(int n_probs, int M, int N, int bm, int bn) {
  return (long long)((M + bm - 1) / bm) * ((N + bn - 1) / bn) * n_probs;
}
inline double tile_rounds(int n_probs, int M, int N, int bm, int bn) { return (double)((tile_count(n_probs, M, N, bm, bn) + 255) / 256); }

// Which tile a launch of the exact-sum kernels takes.  With r = tiles per compute unit, rounded up, the time of a launch
// is close to a + b r in units of a 128 x 128 tile of a full chip; a is what a tile's dependent steps take when nothing
// else runs beside it.  (a, b) are fits to timings of M 128 .. 50000, N 64 .. 12288, K 128 .. 11008.  The choice is within
// 5 % of the best of the six at most of these sizes.  Measured, us (128 x 128 or 256 x 128, which was the rule before,
// against what is taken now): 1024 x 512 x 2048 23.8 -> 8.8, 1024 x 2048 x 512 12.4 -> 7.6, 3000 x 768 x 3072 35 -> 26,
// 8192 x 512 x 2048 32 -> 25, 512 x 4096 x 11008 102 -> 61, 9000 x 2304 x 768 50 -> 45.  From five tiles of 256 x 128 per unit
// on that kernel is the fastest whatever the remainder (50000 x 3072 x 768: 261 against 355 and more).
// A smaller tile reads more per product, which the fit does not know: where the larger one's tiles fill the chip already
// (r > 1) and rows of K are longer than 1024 bytes, it is taken only if it promises 6 %.  Of 38 such sizes that promise less
// 26 took 4 % longer or more with it and 4 that much less (2178 x 3264 x 1408 in bfloat16 33 -> 44, 7143 x 2880 x 3840 177 ->
// 192); with shorter rows it is the other way round (59 sizes: 4 and 33, 860 x 7104 x 128 0.95 of the larger tile's time).
// 256 x 256 (wide: plain problems with rows of whole cache lines, gemm8_wide_ok): one workgroup per unit; because the clock rises
// where units run out of tiles, a last round costs between its share and a whole one, and an epilogue counts for more the fewer
// slabs a tile has, most of all one that reads a residual, during which the matrix cores idle.  It is taken where it promises 6 %.
// Of random plain sizes (10 to 5000 such tiles) that take it, time over that of the other tiles, without a residual: 71 in codes
// 0.86 in the mean, 1.01 at most, 132 in bfloat16 0.70 and 0.99.  With one: 41 in codes 0.91 and 1.03, 99 in bfloat16 0.73 and 1.01;
// by the rule without a residual 42 more in codes, 1.01 in the mean (2144 x 6560 x 512 30 -> 38 us, 98571 x 416 x 384 97 -> 110),
// and 15 in bfloat16 of few tiles and short rows, 1.07 (2564 x 11104 x 256 bytes 46 -> 57, 12679 x 1664 x 1024 55 -> 60).
// K: bytes of an operand row.
enum ExactTile { TILE_256x256, TILE_256x128, TILE_128x128, TILE_64x128, TILE_128x64, TILE_64x64, TILE_32x64 };
inline ExactTile pick_exact_tile(int n_probs, int M, int N, int K, bool b16, bool kl, bool wide, bool residual) {
  auto per_cu = [&](int bm, int bn) { return tile_rounds(n_probs, M, N, bm, bn); };
  const bool narrow = N <= 64 && !kl;
  ExactTile best = narrow ? TILE_128x64 : TILE_128x128;
  double r = narrow ? per_cu(128, 64) : per_cu(128, 128);
  double cost = narrow ? 0.37 + 0.48 * r : 0.5 + 0.85 * r;
  bool large = false;
  if (!narrow && !b16 && !kl && M >= 8192 && N >= 128) {
    const double rp = per_cu(256, 128);
    if (rp >= 5 || 0.1 + 1.8 * rp <= cost) { best = TILE_256x128; r = rp; cost = 0.1 + 1.8 * rp; large = rp >= 5; }
  }
  if (!large) {
    if (r > 1 && K > 1024) cost *= 0.94;
    auto consider = [&](ExactTile t, double c) { if (c < cost) { best = t; cost = c; } };
    if (!narrow) consider(TILE_64x128, 0.37 + 0.48 * per_cu(64, 128));
    if (!kl) {         // (the parts of a row of the KL epilogue are 64 columns of one wave)
      consider(TILE_64x64, 0.3 + 0.26 * per_cu(64, 64));
      consider(TILE_32x64, 0.27 + 0.17 * per_cu(32, 64));
    }
  }
  if (wide) {
    const double t = (double)tile_count(n_probs, M, N, 256, 256) / 256;
    const double per_round = b16 ? 1.2 + 40.0 / K : 1.25 + (residual ? 300.0 : 120.0) / K;
    const bool short_rows = b16 && residual && K <= 1024 && t < 2;
    if (!short_rows && 0.6 + per_round * (std::ceil(t) + t) <= 0.94 * cost) best = TILE_256x256;
  }
  return best;
}

// Tiles of gemm_f32_x_k; _STEP4: four slabs of 32 k per wait.
enum F32Tile { F32_128x128, F32_64x64, F32_32x64_STEP4, F32_32x64, F32_32x32_STEP4, F32_32x32 };

// K: length of the sums.  (us)
// - from two tiles of 64 x 64 per unit on those, or 128 x 128 (half the reads from LDS) where their last round leaves no more
//   idle (16384 x 2048 x 512 284 / 276, 15616 x 512 x 2048 293 / 265, but 5000 x 2048 x 512 93 / 107 and 2048 x 2048 x 512, one
//   tile of 128 x 128 per unit, 41 / 44; 64 x 64 overlap from round to round, so their last round counts half) and the sums are
//   long enough to hide the large tile's epilogue, which two waves per SIMD carry alone: 102400 x 768 x 64 145 / 136, with a
//   residual 189 / 208, with a second output too 363 / 379; 24576 x 1024 x 256 113 / 111, 115 / 120, 158 / 177, x 512 214 / 204,
//   216 / 213.  (A second output goes with K = d_head only.)  Of 54 random launches whose 128 x 128 tiles fill the chip six take
//   them, at 0.96 to 0.99 of the time of 64 x 64; 37 of the others would take longer with them, by up to 1.4.
// - one workgroup per unit or less: a wave's chain of waiting, reading and multiplying is what is seen, and four slabs per wait
//   shorten it (32 x 64 / the same in fours / 32 x 32 / the same in fours): 1184 x 128 x 4096 three times 55 / 49 / 53 / 51,
//   256 x 128 x 4096 three times 56 / 49 / 50 / 35, 512 x 512 x 512 10.3 / 9.4 / 8.2 / 7.6.  While there are few steps, one that is
//   not full costs more than it saves: 128 x 16 x 64 three times 3.3 / 3.6 / 2.9 / 3.2, 1600 x 64 x 64 three times
//   3.6 / 4.0 / 3.5 / 3.8, 512 x 512 x 192 5.2 / 5.3 / 4.3 / 4.5, but x 128 4.4 / 4.1 / 3.7 / 3.6; from 13 slabs on it no longer
//   does (512 x 512 x 416 7.9 / 7.7 / 6.2 / 6.1).
// - between the two 32 x 64 or, where they fill the units more evenly, 32 x 32: 1024 x 768 x 512 14.8 / 13.8,
//   1216 x 512 x 512 14.3 / 13.1, but 540 x 1536 x 1024 23.5 / 26.8.
inline F32Tile pick_f32_tile(int n_probs, int M, int N, int K) {
  auto rounds = [&](int bm, int bn) { return tile_rounds(n_probs, M, N, bm, bn); };
  auto tiles = [&](int bm, int bn) { return tile_count(n_probs, M, N, bm, bn); };
  if (tiles(64, 64) >= 512)
    return K >= 512 && tiles(128, 128) > 256 && 3.9 * rounds(128, 128) <= 0.5 * (rounds(64, 64) + tiles(64, 64) / 256.0) ? F32_128x128 : F32_64x64;
  const int slabs = K / 32;
  const bool fours = slabs % 4 == 0 || slabs > 12;
  if (tiles(32, 32) <= 256) return fours ? F32_32x32_STEP4 : F32_32x32;
  if (tiles(32, 64) <= 256) return fours ? F32_32x64_STEP4 : F32_32x32;
  return 1.1 * rounds(32, 32) < 2 * rounds(32, 64) ? F32_32x32 : F32_32x64;
}

}  // namespace pahq
