// Which tile of the fp32 product kernel a launch takes.  Host arithmetic without any GPU type, so that tests can compile it alone.
#pragma once

namespace pahq {

// Tiles of bm x bn of n_probs problems of M x N, and how often they fill 256 compute units.
inline long long tile_count(int n_probs, int M, int N, int bm, int bn) {
  return (long long)((M + bm - 1) / bm) * ((N + bn - 1) / bn) * n_probs;
}
inline double tile_rounds(int n_probs, int M, int N, int bm, int bn) { return (double)((tile_count(n_probs, M, N, bm, bn) + 255) / 256); }

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
