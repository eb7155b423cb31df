// Which tile of the direct-to-LDS int8 kernel takes a layer.  Host arithmetic on sizes only, no HIP: the launchers and a CPU
// test share it.
#pragma once

#include <stdint.h>

#include "cwac.h"

namespace cwac {

inline int64_t tiles_of(int64_t m, int n, int bm, int bn) { return ((m + bm - 1) / bm) * (((int64_t)n + bn - 1) / bn); }

// True where it takes 128 x 128 tiles (layers with few tiles and a long K loop).
inline bool fast_prefers_quarter_tile(int64_t m, int n) {
  // Layers with too few 128 x 256 tiles to occupy the chip: a tile's duration is the K loop of one
  // wavefront, so 128 x 128 tiles of four 64 x 64 wavefronts (half the MFMAs per wavefront and K step,
  // twice the tiles) finish sooner.  Thresholds from measurements on LLM layer shapes at 256-2048
  // tokens and ResNet-50 stage 5: ahead from 96 such tiles on, until 160 half tiles exist.
  const int64_t t_half = tiles_of(m, n, 128, 256), t_q = tiles_of(m, n, 128, 128);
  return n >= 128 && t_half < 160 && t_q >= 96;
}

// True where a convolution of at least 256 rows takes 128 x 128 tiles however few they are: with up to one tile per compute unit
// a layer lasts as long as one tile's K loop, and that of the deep ring (quarter_ring: 2) is the faster one.  3 x 3, 64 x 64
// register-staged tile / this, us: 392 x 256 x 2304 14.9 / 13.2, 3136 x 256 x 2304 15.4 / 13.3, 294 x 512 x 4608 26.0 / 21.0,
// 2205 x 512 x 4608 27.3 / 21.6.
inline bool conv_quarter_tile(int64_t m, int n, int k, int c_in) {
  return (c_in % 128) == 0 && k >= 1536 && n >= 256 && tiles_of(m, n, 128, 128) <= 256;
}

// K step and ring depth of the 128 x 128 tile (four wavefronts of 64 x 64; `kstep`: K or the channels of a filter tap).
// Measured, microseconds at m x n x k, int8 output unless noted:
//   0: 64-byte steps, three stages, three workgroups per compute unit: where steps of 128 do not divide K, and for
//      4-byte outputs in more than two rounds of tiles (their stores weigh as much as the K loop: 12608 x 3072 x 768 fp32
//      52.8 / 54.6 with 1).
//   1: 128-byte steps, two stages, two workgroups per compute unit: half the barriers.  4616 x 768 x 768 9.0 -> 8.1,
//      7252 x 512 x 512 7.1 -> 6.5, 2000 x 3072 x 768 11.8 -> 10.0.
//   2: 128-byte steps, three stages, one workgroup per compute unit: one round of tiles and a long K, where nothing
//      else covers a stage's round trip.  4616 x 768 x 3072 19.6 -> 16.1, 1000 x 4096 x 4096 30.7 -> 23.2,
//      7252 x 512 x 2048 14.6 -> 12.8 (14.4 with 1), 6272 x 256 x 1024 8.5 -> 8.6 (8.4 with 1).  Eight wavefronts in two groups
//      that share a stage's k-steps (on another machine, four / eight): 4616 x 768 x 3072 17.0 / 16.5, 7252 x 512 x 2048 14.2 / 13.7,
//      512 x 4096 x 11008 39.2 / 36.2, 3 x 3 convolutions 6272 x 256 x 2304 13.9 / 13.2, 6272 x 512 x 4608 24.9 / 23.0.  The time is
//      about 6 us + 0.35 us per stage; four stages 0 to 2 % slower; with two stages (1) eight wavefronts 4 to 40 % slower.
inline int quarter_ring(int64_t m, int n, int k, int kstep, bool wide) {
  const int64_t tiles = tiles_of(m, n, 128, 128);
  if ((kstep % 128) != 0 || (wide && tiles > 512)) return 0;
  return tiles <= 256 && k >= 1536 ? 2 : 1;
}

// The 128-token x 256-channel tile on one workgroup per compute unit with 128-byte steps and three stages: one round of
// tiles and a long K.  2048 x 4096 x 4096 42.9 -> 35.1, 500 x 11008 x 4096 39.8 -> 33.2, 2000 x 4096 x 11008 fp32 105.8 -> 88.7.
inline bool half_deep(int64_t m, int n, int k) {
  return (k % 128) == 0 && k >= 3072 && tiles_of(m, n, 128, 256) <= 256;
}

// The tile shape (CWAC_SHAPE_*) it picks by itself for a linear layer with n >= 256.
inline int fast_linear_shape(int64_t m, int n, int k, int out_bytes) {
  // The automatic tile shape of a linear layer with n >= 256, from measurements on the ViT / Swin / LLM
  // layer shapes (K 512 .. 11008, 196 .. 3072 tiles of 256 x 256).
  //  * Few tiles and a long K loop: 128 x 128 tiles (fast_prefers_quarter_tile).
  //  * Less than a round of 256 x 256 tiles: 128 x 256 tiles where they are one round and K is long (half_deep), else
  //    128 x 128 tiles where those are at most two rounds, two workgroups to a compute unit (2000 x 3072 x 768, 384 of
  //    them: 10.0 us, persistent tile 13.6; 1979 x 3952 x 1280, 496: 16.2 / 21.1; 16337 x 448 x 1664, 512: 18.2 / 23.4), or
  //    where K is too short for a tile's loop to matter (8031 x 816 x 128: 9.2 / 12.6; 3106 x 2656 x 128: 8.2 / 9.1; level
  //    at K = 384), else the persistent tile (3152 x 3072 x 768, 600 of them: 14.3, 128 x 128 tiles 15.2; 12608 x 768 x
  //    3072 fp32, 594: 39.4 / 45.7).
  //  * Otherwise the persistent 256 x 256 tile (which splits the tiles of a thin last round in two).
  //    With 4-byte outputs and a short K loop the tile's store burst weighs as much as its K loop: there the 128 x 128
  //    tile (three workgroups per compute unit, four times as many tiles, stores spread out) finishes sooner.  fp32, two sets of
  //    54 and 110 layers from 160 to 2364 tiles, each on its own machine, persistent / 128 x 128: K = 384 and 512 1.00 to 1.25
  //    (12608 x 2304 x 384 34.5 / 31.5, 25216 x 1152 x 512 39.9 / 32.0); K = 640 to 768 to two rounds 1.00 to 1.26 (12608 x 2304 x 768
  //    44.7 / 39.2), beyond them from 0.96 up on the second machine (25216 x 2304 x 768,
  //    3.5 rounds: 76.8 / 79.4; 20000 x 2304 x 768, 2.8: 62.7 / 64.8); K = 1024 ahead where the last 256 channels are at most half
  //    used (25216 x 1152 51.8 / 46.9), else 0.96 to 1.00 (7252 x 4096 49.1 / 50.6, 30000 x 1024 49.4 / 51.6), beyond two rounds 0.86 to
  //    1.05; K = 1536 0.77 to 1.02.  In any case to K = 1024 where the last round leaves a good part of the chip idle (33000 x 1152 x
  //    1024: 68.8 / 60.5).  All of that but for one round of tiles whose 128 x 128 ones just miss one of their own (three to a compute
  //    unit, 768): 12608 x 1024 x 1024, 800 of them, 24.2 / 26.1, 3152 x 4096 x 512, 832, 20.0 / 20.9, 9000 x 1536 x 384, 864, 18.9 / 19.7;
  //    level at 4616 x 3072 x 768, 912 (ragged channels stay: 12608 x 1000 x 768, 792, 1.06).
  //  * 128 to 255 tokens: 128-token tiles, the only ones that the rows fill.
  if (fast_prefers_quarter_tile(m, n)) return CWAC_SHAPE_128_128;
  if ((k % 128) != 0) return CWAC_SHAPE_128_PAIR;
  if (m < 256) return half_deep(m, n, k) ? CWAC_SHAPE_128_PAIR : CWAC_SHAPE_128_128;
  const int64_t t256 = tiles_of(m, n, 256, 256);
  if (t256 < 160) {
    if (half_deep(m, n, k)) return CWAC_SHAPE_128_PAIR;
    return tiles_of(m, n, 128, 128) <= 512 || k <= 256 ? CWAC_SHAPE_128_128 : CWAC_SHAPE_256_PERSIST;
  }
  const double fill = (double)t256 / (double)(256 * ((t256 + 255) / 256));  // busy share of the rounds
  const bool half_used = tiles_of(1, n, 1, 128) % 2 != 0;
  const int64_t t_q = tiles_of(m, n, 128, 128);
  const bool just_missed = t256 < 256 && (n % 128) == 0 && t_q > 768 && t_q <= 880;
  if (out_bytes > 1 && k <= 1024 && !just_missed && (fill < 0.85 || k <= 512 || (t256 <= 512 && (k <= 768 || half_used)))) return CWAC_SHAPE_128_128;
  return CWAC_SHAPE_256_PERSIST;
}

}  // namespace cwac
