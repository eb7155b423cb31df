// Which form of the attention kernel (block_glue.hip) takes a call.  Host arithmetic on sizes only, no HIP: the launcher and
// a CPU test share it.
#pragma once

#include <stdint.h>

namespace cwac {

constexpr int kAttnSplit = 0;       // a head's keys split over a workgroup's wavefronts
                                    // 1 .. 7: a workgroup holds all keys of a head, that many tiles of 32
constexpr int kAttnChunks = 8;      // keys in chunks of 128, blocks of 128 queries
constexpr int kAttnChunksWide = 9;  // ... blocks of 32 attention_wide_waves queries

// Wavefronts (32 queries each) of a wide block.
constexpr int attention_wide_waves(int head_dim) { return head_dim == 64 ? 7 : 8; }

// pairs: images times heads.
inline int attention_form(int tokens, int64_t pairs, int head_dim, bool bias) {
  const int tiles = (tokens + 31) / 32;
  // The keys split over a workgroup's wavefronts while there is at most one such workgroup to a compute unit - its LDS leaves
  // room for one (us, a workgroup per head or 128 queries / split: 3 x 12 x 197 tokens, 252 of them, 7.6 / 5.9; 8 x 3 x 257, 216,
  // 8.4 / 6.8; 12 x 577, 228, 13.4 / 9.2) - and more than four key tiles (12 x 144, five: 5.9 / 5.3; 12 x 128, four: 4.6 / 4.8), or four
  // of 32-wide heads with a bias (4 x 128 4.8 / 4.5, 16 x 100 4.75 / 4.67; 64-wide 16 x 112 5.3 / 5.4, 32-wide without 16 x 128 3.9 / 4.2).
  if ((tiles > 4 || (tiles == 4 && bias && head_dim == 32)) && pairs * tiles <= 256) return kAttnSplit;
  if (tiles <= 7) return tiles;
  // Every workgroup reads and converts all keys of its head, so one wide block beats two blocks of 128 on the same compute unit;
  // but two wide ones that do not fit it together follow one another.  What counts are the query tiles that the fullest
  // compute unit gets.  us, blocks of 128 / wide:
  //   64-wide heads, at most two wide blocks to a compute unit: 8 x 12 x 257 tokens 11.9 / 10.9, 8 x 12 x 400 16.6 / 14.3, 4 x 12 x
  //   1025 33.1 / 28.7, 12 x 4096 110 / 94, 8 x 12 x 1025 (16 query tiles / 14) 58.2 / 53.5; the same share or more blocks: 8 x
  //   12 x 577 (8 / 14) 21.1 / 32.2, 32 x 12 x 400 (24 / 21) 39.8 / 40.7.
  //   32-wide heads, where reading the keys weighs more: also at an equal share (32 x 16 x 400, 32: 39.0 / 32.9; 16 x 4096, 8:
  //   76.4 / 67.9), and with many blocks in any case (32 x 16 x 785, 56 / 64: 121 / 97; 128 x 16 x 257, 96 / 128: 73.0 / 71.8); but
  //   8 x 16 x 577 (12 / 16) 20.0 / 20.2, 32 x 16 x 257 (24 / 32) 21.7 / 22.6.
  //   With a bias the wide blocks are -7 to 30 % slower (more registers per wavefront).
  if (bias) return kAttnChunks;
  const auto load = [&](int waves) { return (pairs * ((tiles + waves - 1) / waves) + 255) / 256 * waves; };
  const int64_t narrow = load(4), wide = load(attention_wide_waves(head_dim));
  const bool pays = head_dim == 64 ? wide < narrow && wide <= 14 : wide <= narrow || narrow > 32;
  return pays ? kAttnChunksWide : kAttnChunks;
}

}  // namespace cwac
