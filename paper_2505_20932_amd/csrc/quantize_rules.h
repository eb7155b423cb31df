// Launch sizes of the row quantizer (quantize.hip).  Host arithmetic on sizes only, no HIP: the launcher and a CPU test share it.
#pragma once

#include <stdint.h>

namespace cwac {

// Threads that a row of k values takes; `vec`: in vectors of 4 (k % 4 == 0, aligned), else 256 threads at any length.
// A wavefront to k = 1024, four to 4096, sixteen beyond.  Four instead of sixteen: 16 x 11008 3.8 us against 3.0, 4096 x 11008 35.0
// against 32.4, level at 5000 x 5120; sixteen instead of four: 512 x 4096 4.3 against 3.1.  Fewer than 512 rows of more
// than 512 values: four wavefronts, one vector per lane (one wavefront / four, us per call of a replayed graph: 8 x 1000 3.19 / 3.03,
// 64 x 1024 3.30 / 3.11, 197 x 896 3.35 / 3.16, 197 x 640 3.18 / 3.15; 512 x 640 3.24 / 3.33, 1000 x 1000 3.80 / 3.90).
inline int quantize_row_threads(int64_t rows, int k, bool vec) {
  if (!vec || k > 16384) return 256;
  if (k <= 1024) return k > 512 && rows < 512 ? 256 : 64;
  return k <= 4096 ? 256 : 1024;
}

// Rows of one launch (a grid counts fewer than 2^32 threads); more rows take several.
inline int64_t quantize_rows_per_launch(int64_t rows, int k, bool vec) {
  return ((int64_t)1 << 31) / quantize_row_threads(rows, k, vec);
}

}  // namespace cwac
