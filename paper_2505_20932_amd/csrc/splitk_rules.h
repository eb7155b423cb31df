// Which tile of the small-problem int8 kernel (qlinear_splitk.hip) takes a layer.  Host arithmetic on sizes only, no HIP: the
// launcher and a CPU test share it.
#pragma once

#include <stdint.h>

#include "fast_rules.h"

namespace cwac {

// Its tiles: 16 tn channels x 16 tm tokens, K split over w wavefronts with rings of d units of 128 bytes of K.
struct SplitkTile {
  int tn, tm, w, d;
};
constexpr SplitkTile kSplitk[] = {{0, 0, 0, 0}, {1, 1, 4, 4}, {2, 1, 4, 3}, {2, 2, 4, 2}, {4, 4, 4, 2}};

// The tile (index into kSplitk), 0 where the tile kernels are faster.
inline int splitk_tile(int64_t m, int n, int k) {
  // Measured against the 64 x 64 tile kernel and among 15 tiles / wavefront counts / ring depths, weights cold
  // (microseconds at m x n x k, tile kernel -> this one):
  //   m <= 16: 16 x 16 tiles.  16 x 4096 x 4096 29.2 -> 6.7, 16 x 12288 x 4096 30.6 -> 13.1 (3.9 TB/s),
  //     16 x 4096 x 11008 70.0 -> 12.7.
  if (m <= 16) return 1;
  const int64_t t32 = tiles_of(m, n, 32, 32), t64 = tiles_of(m, n, 64, 64);
  //   17 .. 32 tokens of a layer whose 32 x 32 tiles would leave compute units idle: 32 channels x 16 tokens.
  //     32 x 4096 x 4096 29.1 -> 7.2 (32 x 32 tiles: 9.0); 32 x 11008 x 4096 16.5 against 15.4 with 32 x 32 tiles.
  if (m <= 32 && t32 <= 192) return 2;
  //   64 x 64 tiles halve the operand traffic of 32 x 32 ones, but only one workgroup fits a compute unit: where
  //     they fill one round and K is long.  200 x 4096 x 4096 28.8 -> 13.0 (18.2 with 32 x 32 tiles),
  //     200 x 4096 x 11008 67.9 -> 24.8 (40.9), 64 x 12288 x 4096 30.5 -> 17.3 (18.9); but 394 x 768 x 3072 (84 tiles)
  //     9.6 against 7.5, 1576 x 768 x 3072 (300 tiles) 17.8 against 15.8, 197 x 3072 x 768 6.9 against 6.7.
  if (t32 > 512 && t64 <= 256 && k >= 1024) return 4;
  //   32 x 32 tiles: 197 x 768 x 768 5.7 -> 3.5, 197 x 768 x 3072 16.7 -> 5.0, 197 x 1152 x 384 4.5 -> 3.2.  The tile
  //     kernel's time grows with K, this one's with the rounds of tiles: level at 2.3 rounds for K = 768
  //     (788 x 768: 6.7 / 6.8) and 4.4 for K = 1536 (3000 x 384: 10.9 / 10.7); ahead at 4.7 rounds for K = 3072
  //     (1576 x 768: 15.8 / 18.0) and 6 for 4096 (128 x 12288: 30.0 / 31.6), behind at 9.4 (200 x 11008: 41.0 / 33.4).
  //     Rows that are no whole number of 64-byte pieces cost the direct-to-LDS loads more than the tile kernel's: four
  //     rounds there (350 x 3040 x 1776, 4.1 rounds: 11.8 / 12.9; 547 x 2352 x 3472, 5.2: 20.1 / 23.4; 286 x 5120 x 8944,
  //     5.6: 62.5 / 72.4; 1712 at 3.9 rounds: 0.89 of the tile kernel's time).
  //     Two workgroups fit a compute unit, so its time steps at two and four rounds: short of four it stays ahead from
  //     K = 680 on, with a shorter K in proportion (256 x 3072 x 768, 3 rounds: 7.1 / 5.9; 300 x 2304 x 768, 2.8: 7.2 / 6.0;
  //     788 x 1280 x 1280, 3.9: 9.9 / 8.2; 300 x 2048 x 512, 2.5: 5.9 / 5.3; 394 x 1152 x 384, 1.8: 4.7 / 3.6; level at
  //     1024 x 768 x 768, 3 rounds, and 512 x 1536 x 384, 3).
  const double rounds = (double)t32 / 256.0, four = (double)k / 170.0 < 4.0 ? (double)k / 170.0 : 4.0;
  double most = 1.0 + (double)k / 480.0;
  if (most < four) most = four;
  const double cap = (k % 64) != 0 ? 4.0 : 6.0;
  return rounds <= (most < cap ? most : cap) ? 3 : 0;
}

// A layer with a code table behind its int8 output, where the plain forward takes the 64 x 64 register-staged tile: 0 that tile and
// a lookup pass, 1 this kernel, 2 the direct-to-LDS kernel, both of which look up in their epilogue.  The pass costs 2 to 2.5 us, so
// such a layer leaves the tile earlier (microseconds, register-staged tile and lookup / split-K / direct-to-LDS):
// 394 x 1536 x 384 6.6 / 4.7 / 5.3, 591 x 1536 x 384 (3.6 rounds of 32 x 32 tiles) 7.3 / 5.2 / 5.4, 788 x 1536 x 384 (4.7) 7.8 / 6.6 /
// 5.5, 592 x 2048 x 512 (4.8) 8.6 / 7.0 / 5.8.  Four rounds, more from K = 640 to where the 128 x 128 tiles get a deep ring
// (quarter_ring): 160 x 6656 x 768 (4.1) 10.0 / 7.6 / 8.3, 250 x 5120 x 768 (5.0) 10.1 / 8.5 / 8.3, 250 x 5120 x 1024 (5.0) 11.2 / 8.9 /
// 9.3, 224 x 6656 x 1024 (5.7) 11.3 / 9.6 / 9.3, 197 x 5120 x 1280 (4.4) 12.2 / 9.7 / 10.8, 250 x 6144 x 1280 (6.0) 12.5 / 10.8 / 10.9,
// 224 x 6144 x 1536 (5.3) 13.5 / 11.0 / 10.2.
inline int table_form(int64_t m, int n, int k) {
  const int64_t t32 = tiles_of(m, n, 32, 32);
  const double rounds = k >= 640 && k < 1536 ? 4.0 + (double)(k - 640) / 320.0 : 4.0;
  if ((double)t32 > 256.0 * rounds && m >= 128 && n >= 256 && (k % 64) == 0) return 2;
  return t32 <= 1536 ? 1 : 0;
}

}  // namespace cwac
