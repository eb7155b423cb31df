// Quantizers of Sec. 3.2 (Eq. 1-2) and the weight column sums used by the
// zero-point term of Eq. 7.  All arithmetic is single fp32 operations with
// IEEE division and round-half-to-even, so codes are reproducible bit for bit.
#include <float.h>
#include <math.h>

#include "cwac_internal.h"
#include "quantize_rules.h"

namespace cwac {
namespace {

constexpr int kRangeBlocks = 1024;
constexpr int kThreads = 256;

// ---- min / max (inputs of Eq. 2): two deterministic stages ------------------
__global__ __launch_bounds__(kThreads) void range_partial_kernel(const float *__restrict__ x,
                                                                 int64_t count, int vec_ok,
                                                                 float *__restrict__ partial) {
  float lo = FLT_MAX, hi = -FLT_MAX;
  const int64_t tid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t nthreads = (int64_t)gridDim.x * kThreads;
  if (vec_ok) {
    const int64_t nvec = count >> 2;
    const float4 *xv = reinterpret_cast<const float4 *>(x);
    for (int64_t i = tid; i < nvec; i += nthreads) {
      const float4 v = xv[i];
      lo = fminf(fminf(lo, v.x), fminf(v.y, fminf(v.z, v.w)));
      hi = fmaxf(fmaxf(hi, v.x), fmaxf(v.y, fmaxf(v.z, v.w)));
    }
    for (int64_t i = (nvec << 2) + tid; i < count; i += nthreads) {
      lo = fminf(lo, x[i]);
      hi = fmaxf(hi, x[i]);
    }
  } else {
    for (int64_t i = tid; i < count; i += nthreads) {
      lo = fminf(lo, x[i]);
      hi = fmaxf(hi, x[i]);
    }
  }
  lo = wave_min(lo);
  hi = wave_max(hi);
  __shared__ float s_lo[kThreads / kWave], s_hi[kThreads / kWave];
  const int w = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) {
    s_lo[w] = lo;
    s_hi[w] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < kThreads / kWave; ++i) {
      lo = fminf(lo, s_lo[i]);
      hi = fmaxf(hi, s_hi[i]);
    }
    partial[2 * blockIdx.x] = lo;
    partial[2 * blockIdx.x + 1] = hi;
  }
}

__global__ __launch_bounds__(kThreads) void range_final_kernel(const float *__restrict__ partial,
                                                               int nblocks,
                                                               float *__restrict__ minmax) {
  float lo = FLT_MAX, hi = -FLT_MAX;
  for (int i = threadIdx.x; i < nblocks; i += kThreads) {
    lo = fminf(lo, partial[2 * i]);
    hi = fmaxf(hi, partial[2 * i + 1]);
  }
  lo = wave_min(lo);
  hi = wave_max(hi);
  __shared__ float s_lo[kThreads / kWave], s_hi[kThreads / kWave];
  const int w = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) {
    s_lo[w] = lo;
    s_hi[w] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < kThreads / kWave; ++i) {
      lo = fminf(lo, s_lo[i]);
      hi = fmaxf(hi, s_hi[i]);
    }
    minmax[0] = lo;
    minmax[1] = hi;
  }
}

// ---- x / s as IEEE division rounds it, without the division's scaling and fix-up steps ------------------------
// With y = RN(1 / s), a first quotient x * y is within 1.5 units in the last place; one residual step
// makes it a neighbour of x / s, the second one RN(x / s) (Markstein's theorem: the residuals are exact and no
// quotient of two 24-bit numbers lies closer than 2^-48 to a midpoint).  The residuals must not underflow where the
// quotient decides a code (|x / s| >= 1/4): scales inside [2^-90, 2^100]; others take the division itself.
// Five instructions instead of eleven; measured with it in the row quantizer below.
constexpr float kQuotMin = 8.0779356694631609e-28f, kQuotMax = 1.2676506002282294e30f;  // 2^-90, 2^100
__device__ __forceinline__ float quotient(float x, float s, float y) {
  float q = x * y;
  q = __builtin_fmaf(__builtin_fmaf(-q, s, x), y, q);
  return __builtin_fmaf(__builtin_fmaf(-q, s, x), y, q);
}

// Four whole numbers in [-128, 127], given as v + 1.5 * 2^23 (whose addition is the rounding), as bytes.
__device__ __forceinline__ uint32_t pack_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  return __builtin_amdgcn_perm(b, a, 0x0c0c0400u) | __builtin_amdgcn_perm(d, c, 0x04000c0cu);
}
constexpr float kRound = 12582912.0f;

// ---- Eq. 1, per-tensor parameters, b-bit codes in signed 8-bit storage ------
// zu = unsigned zero-point, levels = 2^b - 1, half = 2^(b-1)
struct ActQ {
  float s, zu, levels;
  int half;
  // fast form: y = RN(1 / s), 0 where s is outside its range; |x| is first limited to 1024 s (far outside the clip), so
  // that an infinity has a residual; a NaN takes the lower bound, as fmaxf and fminf have it
  float y, limit;
};
__device__ __forceinline__ int act_code(float x, const ActQ &a) {
  float v = rintf(__fdiv_rn(x, a.s)) + a.zu;
  v = fmaxf(v, 0.0f);
  v = fminf(v, a.levels);
  return static_cast<int>(v) - a.half;
}
__device__ __forceinline__ uint32_t act_codes4(const float4 &v, const ActQ &a) {
  const float x[4] = {v.x, v.y, v.z, v.w};
  uint32_t w[4];
  if (a.y != 0.0f) {  // uniform
    const int z = (int)a.zu - a.half;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float q = quotient(__builtin_amdgcn_fmed3f(x[i], -a.limit, a.limit), a.s, a.y);
      w[i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_fmed3f(q, -a.zu, a.levels - a.zu) + kRound) + (uint32_t)z;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = (uint32_t)act_code(x[i], a);
  }
  return pack_bytes(w[0], w[1], w[2], w[3]);
}

// Rows without gaps: a thread's U loads (256 vectors apart, so that every access is a whole line) go out before
// its first code.
template <int U>
__global__ __launch_bounds__(kThreads) void quantize_act_flat_kernel(const float4 *__restrict__ x, int64_t total, ActQ a,
                                                                     uint32_t *__restrict__ q) {
  for (int64_t at = (int64_t)blockIdx.x * (kThreads * U) + threadIdx.x; at < total; at += (int64_t)gridDim.x * (kThreads * U)) {
    float4 v[U];
#pragma unroll
    for (int j = 0; j < U; ++j)
      if (at + j * kThreads < total) v[j] = x[at + j * kThreads];
#pragma unroll
    for (int j = 0; j < U; ++j)
      if (at + j * kThreads < total) q[at + j * kThreads] = act_codes4(v[j], a);
  }
}

__global__ __launch_bounds__(kThreads) void quantize_act_vec_kernel(const float *__restrict__ x,
                                                                    int64_t ldx, int64_t rows,
                                                                    int kv, ActQ a,
                                                                    int8_t *__restrict__ q,
                                                                    int64_t ldq) {
  const int64_t total = rows * kv;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * kThreads) {
    const int64_t r = i / kv;
    const int c = static_cast<int>(i - r * kv) * 4;
    *reinterpret_cast<uint32_t *>(q + r * ldq + c) = act_codes4(*reinterpret_cast<const float4 *>(x + r * ldx + c), a);
  }
}

__global__ __launch_bounds__(kThreads) void quantize_act_kernel(const float *__restrict__ x,
                                                                int64_t ldx, int64_t rows, int k,
                                                                ActQ a, int8_t *__restrict__ q,
                                                                int64_t ldq) {
  const int64_t total = rows * k;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * kThreads) {
    const int64_t r = i / k;
    const int64_t c = i - r * k;
    q[r * ldq + c] = static_cast<int8_t>(act_code(x[r * ldx + c], a));
  }
}

// ---- symmetric per-row quantizer ---------------------
__device__ __forceinline__ int sym_code(float x, float s, float qmax) {
  float v = rintf(__fdiv_rn(x, s));
  v = fmaxf(v, -qmax);
  v = fminf(v, qmax);
  return static_cast<int>(v);
}
__device__ __forceinline__ float row_scale(float amax, float qmax) {
  const float s = __fdiv_rn(amax, qmax), floor_s = FLT_MIN * 256.0f;
  return s >= floor_s ? s : floor_s;
}
// Four codes of a row; y = RN(1 / s), or 0 where s is outside the range of the fast quotient (uniform).  A finite
// scale means finite values (or NaN, which takes the lower bound).
__device__ __forceinline__ uint32_t sym_codes4(const float4 &v, float s, float y, float qmax) {
  const float x[4] = {v.x, v.y, v.z, v.w};
  uint32_t w[4];
  if (y != 0.0f) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      w[i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_fmed3f(quotient(x[i], s, y), -qmax, qmax) + kRound);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = (uint32_t)sym_code(x[i], s, qmax);
  }
  return pack_bytes(w[0], w[1], w[2], w[3]);
}

typedef float f4 __attribute__((ext_vector_type(4)));
template <bool STREAM>
__device__ __forceinline__ float4 load4(const float *p) {
  const f4 *at = reinterpret_cast<const f4 *>(p);
  const f4 v = STREAM ? __builtin_nontemporal_load(at) : *at;
  return make_float4(v[0], v[1], v[2], v[3]);
}

// The row in registers: WPR wavefronts per row, NV vectors of 4 per thread (k <= 256 WPR NV), so every value is read once.
// Bound: HBM for many rows - 4 bytes in, 1 out per value -, one round trip for a few.  Microseconds, with
// every row read twice and IEEE division / now: 16 x 4096 3.4 / 2.7, 16 x 11008 6.0 / 3.0, 2048 x 4096 9.1 / 6.5,
// 16384 x 4096 71 / 53 (6.4 TB/s), 16384 x 11008 238 / 145 (6.2 TB/s), 3072 x 768 4.6 / 3.0.
// STREAM: non-temporal loads.
template <int WPR, int NV, int THREADS, bool STREAM>
__global__ __launch_bounds__(THREADS) void quantize_rows_reg_kernel(const float *__restrict__ x, int64_t ldx, int rows, int k,
                                                                    float qmax, float *__restrict__ scale,
                                                                    int8_t *__restrict__ q, int64_t ldq) {
  constexpr int RPB = THREADS / (64 * WPR);  // rows per workgroup
  const int tid = WPR == 1 ? (int)(threadIdx.x & 63) : (int)threadIdx.x;
  const int64_t row = (int64_t)blockIdx.x * RPB + (WPR == 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0);
  if (WPR == 1 && row >= rows) return;  // whole wavefronts; no barrier below for WPR == 1
  const float *xr = x + row * ldx;
  int8_t *qr = q + row * ldq;
  float4 v[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int c = 4 * (tid + j * (64 * WPR));
    v[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (c < k) v[j] = load4<STREAM>(xr + c);
  }
  float amax = 0.0f;
#pragma unroll
  for (int j = 0; j < NV; ++j)
    amax = fmaxf(fmaxf(amax, fabsf(v[j].x)), fmaxf(fabsf(v[j].y), fmaxf(fabsf(v[j].z), fabsf(v[j].w))));
  amax = wave_max(amax);
  if constexpr (WPR > 1) {
    __shared__ float s_max[WPR];
    if ((threadIdx.x & 63) == 0) s_max[threadIdx.x >> 6] = amax;
    __syncthreads();
    amax = s_max[0];
#pragma unroll
    for (int i = 1; i < WPR; ++i) amax = fmaxf(amax, s_max[i]);
  }
  const float s = row_scale(amax, qmax);
  const float y = s >= kQuotMin && s <= kQuotMax ? __fdiv_rn(1.0f, s) : 0.0f;
  if (tid == 0) scale[row] = s;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int c = 4 * (tid + j * (64 * WPR));
    if (c < k) *reinterpret_cast<uint32_t *>(qr + c) = sym_codes4(v[j], s, y, qmax);
  }
}

// Any layout and length: one workgroup per row, the row read twice.
__global__ __launch_bounds__(kThreads) void quantize_rows_sym_kernel(
    const float *__restrict__ x, int64_t ldx, int k, int vec_ok, float qmax,
    float *__restrict__ scale, int8_t *__restrict__ q, int64_t ldq) {
  const int64_t row = blockIdx.x;
  const float *xr = x + row * ldx;
  int8_t *qr = q + row * ldq;
  float amax = 0.0f;
  if (vec_ok) {
    for (int c = threadIdx.x * 4; c < k; c += kThreads * 4) {
      const float4 v = *reinterpret_cast<const float4 *>(xr + c);
      amax = fmaxf(fmaxf(amax, fabsf(v.x)), fmaxf(fabsf(v.y), fmaxf(fabsf(v.z), fabsf(v.w))));
    }
  } else {
    for (int c = threadIdx.x; c < k; c += kThreads) amax = fmaxf(amax, fabsf(xr[c]));
  }
  amax = wave_max(amax);
  __shared__ float s_max[kThreads / kWave];
  if ((threadIdx.x & (kWave - 1)) == 0) s_max[threadIdx.x / kWave] = amax;
  __syncthreads();
  amax = s_max[0];
  for (int i = 1; i < kThreads / kWave; ++i) amax = fmaxf(amax, s_max[i]);
  const float s = row_scale(amax, qmax);
  if (threadIdx.x == 0) scale[row] = s;
  if (vec_ok) {
    const float y = s >= kQuotMin && s <= kQuotMax ? __fdiv_rn(1.0f, s) : 0.0f;
    for (int c = threadIdx.x * 4; c < k; c += kThreads * 4)
      *reinterpret_cast<uint32_t *>(qr + c) = sym_codes4(*reinterpret_cast<const float4 *>(xr + c), s, y, qmax);
  } else {
    for (int c = threadIdx.x; c < k; c += kThreads)
      qr[c] = static_cast<int8_t>(sym_code(xr[c], s, qmax));
  }
}

// ---- colsum[n] = sum_k w_q[n,k]: one wavefront per row ----------------------
__global__ __launch_bounds__(kThreads) void colsum_kernel(const int8_t *__restrict__ w,
                                                          int64_t ldw, int n, int k, int vec_ok,
                                                          int32_t *__restrict__ colsum) {
  const int row = blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave;
  if (row >= n) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int8_t *wr = w + (int64_t)row * ldw;
  int s = 0;
  if (vec_ok) {
    for (int c = lane * 16; c < k; c += kWave * 16) {
      const int4 v = *reinterpret_cast<const int4 *>(wr + c);
      const int words[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int j = 0; j < 4; ++j)
        s += (words[j] << 24 >> 24) + (words[j] << 16 >> 24) + (words[j] << 8 >> 24) +
             (words[j] >> 24);
    }
  } else {
    for (int c = lane; c < k; c += kWave) s += wr[c];
  }
  s = wave_sum(s);
  if (lane == 0) colsum[row] = s;
}

template <int WPR, int NV, int THREADS>
cwac_status rows_reg(const float *x, int64_t ldx, int rows, int k, float qmax, float *scale, int8_t *q, int64_t ldq,
                     hipStream_t st) {
  const unsigned grid = (unsigned)ceil_div(rows, THREADS / (64 * WPR));
  // Values that the last-level cache (256 MiB) cannot hold are streamed past it: 16384 x 11008 152 us against 145,
  // 16384 x 4096 59 against 53; smaller ones may be there already: 4096 x 11008 (172 MiB) 32 against 39 streamed.
  if constexpr (WPR > 1) {
    if ((int64_t)rows * k * 4 >= ((int64_t)256 << 20)) {
      quantize_rows_reg_kernel<WPR, NV, THREADS, true><<<grid, THREADS, 0, st>>>(x, ldx, rows, k, qmax, scale, q, ldq);
      return launch_status();
    }
  }
  quantize_rows_reg_kernel<WPR, NV, THREADS, false><<<grid, THREADS, 0, st>>>(x, ldx, rows, k, qmax, scale, q, ldq);
  return launch_status();
}

// k % 4 == 0 and k <= 16384, rows and codes aligned for vectors of 4.
cwac_status launch_rows_reg(const float *x, int64_t ldx, int rows, int k, float qmax, float *scale, int8_t *q, int64_t ldq,
                            hipStream_t st) {
  const int vecs = (k + 255) / 256;  // per lane, were the row one wavefront's
  if (vecs <= 4 && quantize_row_threads(rows, k, true) == 256) return rows_reg<4, 1, 256>(x, ldx, rows, k, qmax, scale, q, ldq, st);
  if (vecs <= 1) return rows_reg<1, 1, 256>(x, ldx, rows, k, qmax, scale, q, ldq, st);
  if (vecs <= 2) return rows_reg<1, 2, 256>(x, ldx, rows, k, qmax, scale, q, ldq, st);
  if (vecs <= 4) return rows_reg<1, 4, 256>(x, ldx, rows, k, qmax, scale, q, ldq, st);
  if (vecs <= 8) return rows_reg<4, 2, 256>(x, ldx, rows, k, qmax, scale, q, ldq, st);
  if (vecs <= 16) return rows_reg<4, 4, 256>(x, ldx, rows, k, qmax, scale, q, ldq, st);
  if (vecs <= 32) return rows_reg<16, 2, 1024>(x, ldx, rows, k, qmax, scale, q, ldq, st);
  if (vecs <= 48) return rows_reg<16, 3, 1024>(x, ldx, rows, k, qmax, scale, q, ldq, st);
  return rows_reg<16, 4, 1024>(x, ldx, rows, k, qmax, scale, q, ldq, st);
}

}  // namespace
}  // namespace cwac

using namespace cwac;

extern "C" size_t cwac_range_workspace(int64_t count) {
  (void)count;
  return (size_t)kRangeBlocks * 2 * sizeof(float);
}

extern "C" cwac_status cwac_range_f32(const float *x, int64_t count, float *minmax,
                                      void *workspace, size_t workspace_bytes, void *stream) {
  if (!x || !minmax) return CWAC_E_NULL;
  if (count < 1) return CWAC_E_SHAPE;
  if (!workspace || workspace_bytes < cwac_range_workspace(count)) return CWAC_E_WORKSPACE;
  if (!aligned(x, 4) || !aligned(minmax, 4) || !aligned(workspace, 8)) return CWAC_E_ALIGN;
  const int vec_ok = aligned(x, 16);
  int blocks = (int)(ceil_div(count, (int64_t)kThreads * 16) < kRangeBlocks
                         ? ceil_div(count, (int64_t)kThreads * 16)
                         : kRangeBlocks);
  float *partial = static_cast<float *>(workspace);
  range_partial_kernel<<<blocks, kThreads, 0, as_stream(stream)>>>(x, count, vec_ok, partial);
  range_final_kernel<<<1, kThreads, 0, as_stream(stream)>>>(partial, blocks, minmax);
  return launch_status();
}

extern "C" cwac_status cwac_qparams_from_range(float mn, float mx, int32_t bits, float *s,
                                               int32_t *z) {
  if (!s || !z) return CWAC_E_NULL;
  if (bits < 2 || bits > 8) return CWAC_E_SHAPE;
  // Eq. 2 in fp32; volatile keeps each operation a separately rounded fp32 op.
  const float levels = (float)((1 << bits) - 1);
  volatile float diff = mx - mn;
  volatile float scale = diff / levels;
  const float floor_s = FLT_MIN * (float)(1 << bits);
  if (!(scale >= floor_s)) scale = floor_s;
  volatile float ratio = -mn / scale;
  float zf = rintf(ratio);
  if (zf < 0.0f) zf = 0.0f;
  if (zf > levels) zf = levels;
  *s = scale;
  *z = (int32_t)zf;
  return CWAC_OK;
}

extern "C" cwac_status cwac_quantize_act_bits(const float *x, int64_t ldx, int64_t rows, int32_t k,
                                              float s, int32_t z, int32_t bits, int8_t *q,
                                              int64_t ldq, void *stream) {
  if (!x || !q) return CWAC_E_NULL;
  if (bits < 2 || bits > 8) return CWAC_E_SHAPE;
  const int half = 1 << (bits - 1);
  if (rows < 0 || k < 1 || ldx < k || ldq < k || !(s > 0.0f) || z < -half || z > half - 1)
    return CWAC_E_SHAPE;
  if (!aligned(x, 4)) return CWAC_E_ALIGN;
  if (rows == 0) return CWAC_OK;
  ActQ a;
  a.s = s;
  a.zu = (float)(z + half);
  a.levels = (float)((1 << bits) - 1);
  a.half = half;
  a.y = s >= kQuotMin && s <= kQuotMax ? 1.0f / s : 0.0f;
  a.limit = a.y != 0.0f ? 1024.0f * s : 0.0f;
  const bool vec = (k % 4 == 0) && (ldx % 4 == 0) && (ldq % 4 == 0) && aligned(x, 16) &&
                   aligned(q, 4);
  if (vec && ldx == k && ldq == k) {
    const int64_t total = rows * (k / 4);
    const float4 *xv = reinterpret_cast<const float4 *>(x);
    uint32_t *qv = reinterpret_cast<uint32_t *>(q);
    // one vector per thread while that is at most four workgroups of 256 to a compute unit (latency), else four
    if (total <= 1024 * kThreads) {
      quantize_act_flat_kernel<1><<<(unsigned)ceil_div(total, kThreads), kThreads, 0, as_stream(stream)>>>(xv, total, a, qv);
    } else {
      const int64_t blocks = ceil_div(total, 4 * kThreads);
      quantize_act_flat_kernel<4><<<(unsigned)(blocks < (1 << 23) ? blocks : (1 << 23)), kThreads, 0, as_stream(stream)>>>(
          xv, total, a, qv);
    }
    return launch_status();
  }
  const int64_t work = vec ? rows * (k / 4) : rows * (int64_t)k;
  const int64_t want = ceil_div(work, kThreads);
  const int blocks = (int)(want < 65536 ? want : 65536);
  if (vec)
    quantize_act_vec_kernel<<<blocks, kThreads, 0, as_stream(stream)>>>(x, ldx, rows, k / 4, a, q,
                                                                         ldq);
  else
    quantize_act_kernel<<<blocks, kThreads, 0, as_stream(stream)>>>(x, ldx, rows, k, a, q, ldq);
  return launch_status();
}

extern "C" cwac_status cwac_quantize_act(const float *x, int64_t ldx, int64_t rows, int32_t k,
                                         float s, int32_t z, int8_t *q, int64_t ldq,
                                         void *stream) {
  return cwac_quantize_act_bits(x, ldx, rows, k, s, z, 8, q, ldq, stream);
}

extern "C" cwac_status cwac_quantize_rows_sym_bits(const float *x, int64_t ldx, int64_t rows,
                                                   int32_t k, int32_t bits, float *scale,
                                                   int8_t *q, int64_t ldq, void *stream) {
  if (!x || !q || !scale) return CWAC_E_NULL;
  if (bits < 2 || bits > 8) return CWAC_E_SHAPE;
  if (rows < 0 || rows > 0x7fffffff || k < 1 || ldx < k || ldq < k) return CWAC_E_SHAPE;
  if (!aligned(x, 4) || !aligned(scale, 4)) return CWAC_E_ALIGN;
  if (rows == 0) return CWAC_OK;
  const int vec = (k % 4 == 0) && (ldx % 4 == 0) && (ldq % 4 == 0) && aligned(x, 16) &&
                  aligned(q, 4);
  const float qmax = (float)((1 << (bits - 1)) - 1);
  hipStream_t st = as_stream(stream);
  const int64_t most = quantize_rows_per_launch(rows, k, vec);
  for (int64_t row = 0; row < rows; row += most) {
    const int n = (int)(rows - row < most ? rows - row : most);
    const float *xr = x + row * ldx;
    int8_t *qr = q + row * ldq;
    cwac_status status;
    if (vec && k <= 16384) {
      status = launch_rows_reg(xr, ldx, n, k, qmax, scale + row, qr, ldq, st);
    } else {
      quantize_rows_sym_kernel<<<(unsigned)n, kThreads, 0, st>>>(xr, ldx, k, vec, qmax, scale + row, qr, ldq);
      status = launch_status();
    }
    if (status != CWAC_OK) return status;
  }
  return CWAC_OK;
}

extern "C" cwac_status cwac_quantize_rows_sym(const float *x, int64_t ldx, int64_t rows,
                                              int32_t k, float *scale, int8_t *q, int64_t ldq,
                                              void *stream) {
  return cwac_quantize_rows_sym_bits(x, ldx, rows, k, 8, scale, q, ldq, stream);
}

extern "C" cwac_status cwac_colsum(const int8_t *w_q, int64_t ldw, int32_t n, int32_t k,
                                   int32_t *colsum, void *stream) {
  if (!w_q || !colsum) return CWAC_E_NULL;
  if (n < 1 || k < 1 || ldw < k) return CWAC_E_SHAPE;
  if (!aligned(colsum, 4)) return CWAC_E_ALIGN;
  const int vec = (k % 16 == 0) && (ldw % 16 == 0) && aligned(w_q, 16);
  const int rows_per_block = kThreads / kWave;
  colsum_kernel<<<(unsigned)ceil_div(n, rows_per_block), kThreads, 0, as_stream(stream)>>>(
      w_q, ldw, n, k, vec, colsum);
  return launch_status();
}
