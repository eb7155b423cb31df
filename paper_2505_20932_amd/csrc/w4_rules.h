// Which tile of the weight-streaming INT4 kernel takes a layer, and whether that kernel does.  Host arithmetic on sizes
// only, no HIP: the launcher (w4a16.hip) and a CPU test share it.
#pragma once

#include <stdint.h>

namespace cwac {

// Tiles of the weight-streaming kernel: 32 nb output channels x mp tokens per workgroup of nw wavefronts, rings of `depth`
// units of 64 input channels.  Wavefronts and ring depth as measured best: eight wavefronts where their rings fit the
// LDS (two per SIMD, so that one's LDS reads run under the other's MFMAs), two slots each (three: within 3 %; four of 8
// rows: 4 % slower).  us: a round of one workgroup per compute unit at k = 4096, measured with cold weights at
// n = 4096 .. 12288 and k = 4096 and 11008; taken to grow with k.
struct W4StreamTile {
  int nb, mp, nw, depth;
  double us;
};
constexpr W4StreamTile kW4Stream[] = {{1, 8, 8, 2, 4.2},  {1, 16, 8, 3, 4.2}, {1, 32, 8, 2, 5.0},  {2, 32, 8, 2, 8.5},
                                      {1, 64, 8, 2, 8.0}, {2, 64, 4, 2, 12.3}, {2, 128, 4, 2, 21.5}};
constexpr int kW4StreamTiles = (int)(sizeof(kW4Stream) / sizeof(kW4Stream[0]));

struct W4StreamChoice {
  int tile = 0;         // index into kW4Stream
  double cost = 1e30;   // estimated microseconds
};

// What the tiles trade: fewer tokens per workgroup read the weights more often, fewer channels the activations, and each
// halves when its factor doubles, until there is less than a round of workgroups.  2 us go to launch and epilogue.
inline W4StreamChoice w4_stream_choice(int64_t m, int n, int k) {
  W4StreamChoice best;
  for (int i = m <= 8 ? 0 : 1; i < (m <= 8 ? 1 : kW4StreamTiles); ++i) {
    const W4StreamTile &t = kW4Stream[i];
    const int64_t wgs = ((m + t.mp - 1) / t.mp) * (((int64_t)n + 32 * t.nb - 1) / (32 * t.nb));
    const double cost = 2.0 + (double)((wgs + 255) / 256) * t.us * (double)k / 4096.0;
    if (cost < best.cost) {
      best.cost = cost;
      best.tile = i;
    }
  }
  return best;
}

// 128-token tiles of the tiled kernel in a launch up to which it takes them (one per compute unit)
constexpr int64_t kW4HalfTileUpTo = 256;

// Whether the weight-streaming kernel takes the layer.  Up to 32 tokens always: the layer is its weight stream, and a tile
// of the tiled kernel would compute 128 token rows for them.  Tiled -> streaming, 1 / 16 / 32 tokens: 131072 x 4096
// 99 / 104 / 104 us -> 58 / 76 / 91, 151936 x 4096 173 / 177 / 178 -> 64 / 88 / 108.  Above 32, against the tiled kernel's first round of 128-token
// tiles, which costs 3 + 0.0127 k: a tile walks all of k by itself.  Measured, tiled -> streaming: 128 x 4096 x 4096
// 55 -> 10.0, 400 x 4096 x 4096 55.5 -> 24.1, 256 x 4096 x 11008 119 -> 34.1, 200 x 12288 x 4096 56.7 -> 41.3; level at
// 400 x 12288 x 4096 (68.9 / 68.5).
inline bool w4_stream_pays(int64_t m, int n, int k, const W4StreamChoice &c) {
  if (m <= 32) return true;
  return ((m + 127) / 128) * (((int64_t)n + 255) / 256) <= kW4HalfTileUpTo && c.cost < 3.0 + 0.0127 * (double)k;
}

}  // namespace cwac
