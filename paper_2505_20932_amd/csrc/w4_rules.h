// Which tile of the weight-streaming INT4 kernel takes a layer, and whether that kernel does.  Host arithmetic on sizes
// only, no HIP: the launcher (w4a16.hip) and a CPU test share it.
#pragma once

#include <stdint.h>

namespace cwac {

// Tiles of the weight-streaming kernel: 32 nb output channels x mp tokens per workgroup of nw wavefronts, rings of `depth`
// units of 64 input channels.  Wavefronts and ring depth as measured best: eight wavefronts where their rings fit the
// LDS (two per SIMD, so that one's LDS reads run under the other's MFMAs), two slots each (three: within 3 %; four of 8
// rows: 4 % slower).  us: a round of one workgroup per compute unit at k = 4096, measured with cold weights at
// n = 4096 .. 12288 and k = 4096 and 11008; the choice among the tiles takes it to grow with k.  short_us, long_us: a round
// costs short_us + long_us k / 4096 (launches of 1 to 16 rounds, k = 128 .. 4096, n = 512 .. 131072; rms 6 to 8 %): what a
// workgroup does besides its K loop weighs as much as the loop where k is a few hundred.
struct W4StreamTile {
  int nb, mp, nw, depth;
  double us, short_us, long_us;
};
constexpr W4StreamTile kW4Stream[] = {{1, 8, 8, 2, 4.2, 0.5, 2.7},  {1, 16, 8, 3, 4.2, 0.7, 3.2},  {1, 32, 8, 2, 5.0, 1.6, 4.5},
                                      {2, 32, 8, 2, 8.5, 2.5, 6.8}, {1, 64, 8, 2, 8.0, 2.1, 7.3},  {2, 64, 4, 2, 12.3, 2.9, 10.2},
                                      {2, 128, 4, 2, 21.5, 5.1, 17.0},
                                      // the first two with four wavefronts (chosen by w4_stream_tile, not by cost)
                                      {1, 8, 4, 2, 4.2, 0.5, 2.7},  {1, 16, 4, 2, 4.2, 0.7, 3.2}};
constexpr int kW4StreamTiles = (int)(sizeof(kW4Stream) / sizeof(kW4Stream[0]));
constexpr int kW4StreamByCost = 7;  // the tiles that the estimate chooses among

// rounds of one workgroup per compute unit
inline double w4_stream_rounds(const W4StreamTile &t, int64_t m, int n) {
  const int64_t wgs = ((m + t.mp - 1) / t.mp) * (((int64_t)n + 32 * t.nb - 1) / (32 * t.nb));
  return (double)((wgs + 255) / 256);
}

// The tile (index into kW4Stream).  What the tiles trade: fewer tokens per workgroup read the weights more often, fewer
// channels the activations, and each halves when its factor doubles, until there is less than a round of workgroups.
inline int w4_stream_tile(int64_t m, int n, int k) {
  // Up to 16 tokens, more than a round of workgroups and at most two units of K for each of eight wavefronts: four of them.
  // Eight / four, us: 16 x 24576 x 128 5.1 / 3.8, 16 x 131072 x 512 22.9 / 14.0, 1 x 131072 x 1024 23.7 / 19.2,
  // 8 x 12288 x 1024 4.8 / 4.7; level at 8 x 8192 x 1024 (4.0 / 4.0), behind at 1 x 49152 x 2048 (14.1 / 15.1).
  if (m <= 16 && n > 8192 && k <= 1024) return m <= 8 ? kW4StreamByCost : kW4StreamByCost + 1;
  if (m <= 8) return 0;
  int best = 1;
  double cost = 1e30;
  for (int i = 1; i < kW4StreamByCost; ++i) {
    const double c = w4_stream_rounds(kW4Stream[i], m, n) * kW4Stream[i].us * (double)k / 4096.0;
    if (c < cost) {
      cost = c;
      best = i;
    }
  }
  return best;
}

// Whether up to 16 tokens run in tiles of 16 channels instead (w4a16_stream16_kernel).  With m x n, the channels that the fullest of
// 256 compute units gets are what counts: fewer with 16-channel tiles up to n = 4096 (16 against 32) and from 8224 to 12288
// (48 against 64).  Gain over the 32-channel tiles, k = 128 .. 8192: n <= 4096 11 to 56 %, 8224 .. 12288 with up to 8 tokens 0 to
// 24 %; with up to 8 tokens and n = 4128 .. 8192, where both give 32, 0 to 22 % to k = 1024, -1 to 6 % at 1536 and, but for the
// narrowest, -5 to 4 % from 2048 on (us, 32 / 16 channels: 1 x 6144 x 2048 4.57 / 4.74, 4 x 8192 x 4096 6.05 / 6.39, 8 x 4128 x 4096
// 5.94 / 5.76).  Wider layers lose up to 33 %, and 9 to 16 tokens wider than 4096 up to 40 %: their activations are read by twice the
// workgroups.
inline bool w4_stream16_pays(int64_t m, int n, int k) {
  if (n <= 4096) return m <= 16;
  return m <= 8 && n <= 12288 && (n > 8192 || k <= (n <= 4608 ? 4096 : 1536));
}

// 128-token tiles of the tiled kernel in a launch up to which it takes them (one per compute unit)
constexpr int64_t kW4HalfTileUpTo = 256;

// Pieces that the tiles of the last round are cut into (512-channel tiles of the tiled kernel, one per compute unit and round).
// A thin last round in pieces (us, whole tiles / pieces): rest 8, 1400 x 12288 x 4096 190 / 164; rest 32, 3000 x 6144 x 2048
// 98 / 82; rest 64, 3000 x 12288 x 4096 298 / 273; rest 96, 2048 x 11008 x 4096 189 / 174; rest 128, 2048 x 12288 x 4096 200 / 189.
// Quarters rather than halves to 64: rest 8 164 / 169, rest 64 273 / 276; level at 68.  More than 128 tiles would need two
// rounds of halves, 2 x 2/3 of a tile.
inline int w4_pieces(int64_t tiles) {
  const int64_t rest = tiles % 256;
  return tiles <= 256 || rest == 0 || rest > 128 ? 1 : rest <= 64 ? 4 : 2;
}

// Whether the weight-streaming kernel takes the layer, with the tile above.  Up to 32 tokens always: the layer is its weight
// stream, and a tile of the tiled kernel would compute 128 token rows for them.  Tiled -> streaming, 1 / 16 / 32 tokens:
// 131072 x 4096 99 / 104 / 104 us -> 58 / 76 / 91, 151936 x 4096 173 / 177 / 178 -> 64 / 88 / 108.
// Above 32, against one round of the tiled kernel's 128-token tiles: each walks all of k by itself, but a wide layer with a
// short k needs one round where the streaming kernel needs several.  Both estimates were fitted to 900 launches; the tiled
// one is taken 5 % low, since the tiled kernel loses less where the two are close.  Measured, tiled -> streaming:
// 128 x 4096 x 4096 55 -> 10.0, 400 x 4096 x 4096 55.5 -> 24.1, 256 x 4096 x 11008 119 -> 34.1, 200 x 12288 x 4096
// 56.7 -> 41.3; level at 400 x 12288 x 4096 (68.9 / 68.5); behind at 200 x 24576 x 128 (7.3 / 16.8), 384 x 12288 x 384
// (10.8 / 20.3) and 128 x 32768 x 768 (16.4 / 19.5).
inline bool w4_stream_pays(int64_t m, int n, int k, int tile) {
  if (m <= 32) return true;
  if (((m + 127) / 128) * (((int64_t)n + 255) / 256) > kW4HalfTileUpTo) return false;
  const W4StreamTile &t = kW4Stream[tile];
  const double dk = (double)k, dn = (double)n;
  const double stream = 1.0 + w4_stream_rounds(t, m, n) * (t.short_us + t.long_us * dk / 4096.0);
  const double tiled = 3.7 + 0.0125 * dk + 0.44e-6 * (double)m * dn + 6.0e-8 * dn * dk;
  return stream < 0.95 * tiled;
}

}  // namespace cwac
