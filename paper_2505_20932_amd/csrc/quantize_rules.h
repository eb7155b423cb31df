// Launch sizes of the row quantizer (quantize.hip).  Host arithmetic on sizes only, no HIP: the launcher and a CPU test share it.
#pragma once

#include <stdint.h>

namespace cwac {

// Threads that a row of k values takes; `vec`: in vectors of 4 (k % 4 == 0, aligned), else 256 threads at any length.
inline int quantize_row_threads(int k, bool vec) {
  return !vec || k > 16384 ? 256 : k <= 1024 ? 64 : k <= 4096 ? 256 : 1024;
}

// Rows of one launch (a grid counts fewer than 2^32 threads); more rows take several.
inline int64_t quantize_rows_per_launch(int k, bool vec) { return ((int64_t)1 << 31) / quantize_row_threads(k, vec); }

}  // namespace cwac
