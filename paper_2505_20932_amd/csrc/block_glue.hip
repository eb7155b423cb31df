// The non-linear glue between the W8A8 linear layers of a pre-norm Transformer block (the part
// of the block that per-layer compensation steps around, Sec. 3.2): residual add + layer
// normalization + quantizer, the GELU of the MLP as a 256-entry code table, and multi-head
// self-attention on the requantized output of the qkv layer.  Every linear layer consumes int8
// codes and requantizes to int8 codes (Eq. 10); the residual stream is binary16.
//
// Arithmetic, in fp32 unless stated (no contraction: each line is one rounding):
//   residual   t = h + s_r * (float)(c - z_r);  h1 = RN16(t);  the layer norm reads h1
//   layer norm mean = sum(x) * (1 / C);  var = sum((x - mean)^2) * (1 / C);  y = fma((x - mean) * rsq(var + eps), gamma, beta)
//   quantizer  code = clip(rne(fma(y, 1 / s, z)), -128, 127)                            (Eq. 1)
//   attention  S = (K - z)(Q - z)^T exactly (integers below 2^24 in the fp32 MFMA accumulators);
//              P = 1024 p = exp2(fma(S, s^2 / sqrt(d) * log2 e, 10 - that * max S));  O = (sum_j RN16(P_j) (V_j - z)) * s / sum_j P_j,
//              keys taken in groups of 64 with a running maximum (earlier partial sums rescaled whenever it rises); the order of
//              all sums follows from the number of tokens alone
//   GELU table entry(c) = clip(rne(GELU(s_in (c - z_in)) / s_out + z_out)) evaluated in fp64 (erf form)
#include <hip/hip_runtime.h>

#include <math.h>

#include "attention_rules.h"
#include "cwac_internal.h"

namespace cwac {
namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v4i __attribute__((ext_vector_type(4)));

// sum over aligned groups of LPR lanes (the same value in every lane of a group), without LDS: neighbours, pairs,
// quads and halves of 16 lanes by DPP, 16s and 32s by the half-wave exchanges
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int LPR, bool PAIRED = false>
__device__ __forceinline__ float group_sum(float v) {
  if constexpr (!PAIRED) v += dpp<0xb1>(v);  // quad_perm 1,0,3,2 (PAIRED: neighbours hold their common sum already)
  v += dpp<0x4e>(v);   // quad_perm 2,3,0,1
  v += dpp<0x141>(v);  // row_half_mirror: the other quad of 8
  v += dpp<0x140>(v);  // row_mirror: the other half of 16
  if constexpr (LPR >= 32) {
    const uint32_t mine = __builtin_bit_cast(uint32_t, v);
    const auto both = __builtin_amdgcn_permlane16_swap(mine, mine, false, false);
    const uint32_t a = both[0], b = both[1];
    v = __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
  }
  if constexpr (LPR >= 64) {
    const uint32_t mine = __builtin_bit_cast(uint32_t, v);
    const auto both = __builtin_amdgcn_permlane32_swap(mine, mine, false, false);
    const uint32_t a = both[0], b = both[1];
    v = __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
  }
  return v;
}

// Four int8 codes (one word) -> (code - z) as four binary16 values, exactly: a byte u = code + 128 under
// the high byte 0x64 is the binary16 number 1024 + u, and (1024 + u) - (1152 + z) is an integer below
// 2048 in magnitude.  `bias` = 1152 + z in both halves.
__device__ __forceinline__ void codes_to_h4(uint32_t w, h2 bias, h2 &lo, h2 &hi) {
  const uint32_t u = w ^ 0x80808080u;
  lo = __builtin_bit_cast(h2, __builtin_amdgcn_perm(0x64646464u, u, 0x04010400u)) - bias;
  hi = __builtin_bit_cast(h2, __builtin_amdgcn_perm(0x64646464u, u, 0x04030402u)) - bias;
}

__device__ __forceinline__ h8 codes_to_h8(uint2 c, h2 bias) {
  h2 a, b, d, e;
  codes_to_h4(c.x, bias, a, b);
  codes_to_h4(c.y, bias, d, e);
  return h8{a[0], a[1], b[0], b[1], d[0], d[1], e[0], e[1]};
}

// Four values of Eq. 1 before rounding -> four codes in a word.  The rounding is an addition: what is clamped to
// whole bounds first rounds to the same code.
__device__ __forceinline__ uint32_t pack_codes(const float (&v)[4]) {
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    w[i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_fmed3f(v[i], -128.0f, 127.0f) + 12582912.0f);
  return __builtin_amdgcn_perm(w[1], w[0], 0x0c0c0400u) | __builtin_amdgcn_perm(w[3], w[2], 0x04000c0cu);
}

// ------------------------------------------------------------------------------------------
// Residual add + layer norm + quantizer: LPR lanes per token row, the row in registers (NV vectors of V channels
// per lane), two-pass mean / variance with the sums taken over the lanes' registers by DPP and half-wave
// exchanges (no LDS).  HBM bytes per element: 2 (h) [+ 1 (codes) + 2 (h1)] + 1 (x_q).
//
// The order of a row's sums follows from C alone, never from the number of rows: a token's codes do not depend on
// the batch that it comes in.  It is the order of vectors of 8 channels on 16, 32 or 64 lanes, whichever pair LPR x NV has
// the fewest idle lanes (32 x 3 for C = 768) - or, where it leaves none idle and that one would, of vectors of 4 on 64 lanes
// (C = 1280 and 1792).
//
// Many rows: workgroups of 256 threads, bound by HBM and, close behind, by the ~16 vector instructions per element;
// gamma and beta pass through LDS, staged while the row's loads are in flight.  Few rows (few wavefronts to a compute
// unit): the serial chain of one row is what takes the time.  So a workgroup is one wavefront, gamma and beta go straight
// into registers, and a vector of 8 is split over a PAIR of lanes: either takes half the elements, and the chain of a sum
// goes from the first to the second lane of the pair with every vector.
// Residual + norm, microseconds, with shuffles through LDS, an integer rounding chain and a row loop / with a wavefront per
// row of 4 channels per lane for few rows, whose sums had an order of their own / now: 197 x 768 4.2 / 3.1 / 3.2, 2308 x 768
// 5.7 / 5.5 / 4.8, 7252 x 512 7.1 / 7.4 / 6.8, 4616 x 768 7.9 / 7.1 / 6.6, 25216 x 768 27.2 / 25.4 / 25.5.
// ------------------------------------------------------------------------------------------
struct LnParams {
  const _Float16 *h;
  int64_t ldh;
  const int8_t *r;
  int64_t ldr;
  float s_r;
  int z_r;
  _Float16 *h_out;
  int64_t ldho;
  const float *gamma, *beta;
  float eps, inv_s_x, inv_c;  // 1 / s_x and 1 / c, rounded once on the host
  int z_x;
  int8_t *x_q;
  int64_t ldxq;
  int64_t m;
  int c;
};

template <int V>
struct LnVec;
template <>
struct LnVec<8> {
  typedef h8 Half;
  typedef uint2 Codes;
  static __device__ __forceinline__ uint32_t word(const uint2 &c, int i) { return i ? c.y : c.x; }
  static __device__ __forceinline__ uint2 pack(const uint32_t (&w)[2]) { return make_uint2(w[0], w[1]); }
};
template <>
struct LnVec<4> {
  typedef h4 Half;
  typedef uint32_t Codes;
  static __device__ __forceinline__ uint32_t word(const uint32_t &c, int) { return c; }
  static __device__ __forceinline__ uint32_t pack(const uint32_t (&w)[1]) { return w[0]; }
};

// The sum of a row: `add` adds an element to a chain.
template <int LPR, int NV, int V, bool PAIRS, typename F>
__device__ __forceinline__ float row_sum(F &&add) {
  float s = 0.0f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
#pragma unroll
    for (int e = 0; e < V; ++e) s = add(s, j, e);
    if constexpr (PAIRS) {  // what counts: the first lane's four, the second lane's on top of them, then both go on from there
      s = dpp<0xa0>(s);     // quad_perm 0,0,2,2
#pragma unroll
      for (int e = 0; e < V; ++e) s = add(s, j, e);
      s = dpp<0xf5>(s);  // quad_perm 1,1,3,3
    }
  }
  return group_sum<LPR, PAIRS>(s);
}

// FULL: every lane's every vector is inside the row (C = V * LPR * NV): no masks.
template <int LPR, int NV, int V, int THREADS, bool FULL, bool PAIRS = false>
__global__ __launch_bounds__(THREADS) void residual_ln_quant_kernel(const LnParams p) {
  constexpr bool kLds = THREADS > 64;  // gamma and beta through LDS
  static_assert(!kLds || V == 8, "the two halves of a vector of 8 lie apart in LDS");
  static_assert(!PAIRS || (V == 4 && LPR >= 32), "half a vector of 8 to a lane, on twice its lanes");
  const int lane = threadIdx.x & (LPR - 1);  // position inside the row's group of LPR lanes
  const int nvec = p.c / V;
  const int64_t row = ((int64_t)blockIdx.x * THREADS + threadIdx.x) / LPR;
  // Groups past the last row read it again and store nothing (h_out may be h): the exchanges run with every lane.
  const bool live = row < p.m;
  const int64_t at = live ? row : p.m - 1;
  typename LnVec<V>::Half hv[NV];
  typename LnVec<V>::Codes cw[NV];
  const _Float16 *hp = p.h + at * p.ldh;
  const int8_t *rp = p.r + at * p.ldr;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int v = (FULL || lane + LPR * j < nvec) ? lane + LPR * j : 0;
    hv[j] = *reinterpret_cast<const typename LnVec<V>::Half *>(hp + V * v);
  }
  if (p.r) {
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int v = (FULL || lane + LPR * j < nvec) ? lane + LPR * j : 0;
      cw[j] = *reinterpret_cast<const typename LnVec<V>::Codes *>(rp + V * v);
    }
  }
  // gamma and beta in LDS: the first and the second four channels of every vector side by side, so that the
  // lanes of a 16-byte read cover all banks
  __shared__ __attribute__((aligned(16))) float s_gb[kLds ? 4096 : 4];
  float4 gr[kLds ? 1 : NV][V / 4], br[kLds ? 1 : NV][V / 4];
  if (p.x_q) {
    if constexpr (kLds) {
      for (int i = threadIdx.x; i < p.c / 4; i += THREADS) {
        const int to = ((i & 1) << 10) + 4 * (i >> 1);
        *reinterpret_cast<float4 *>(s_gb + to) = *reinterpret_cast<const float4 *>(p.gamma + 4 * i);
        *reinterpret_cast<float4 *>(s_gb + 2048 + to) = *reinterpret_cast<const float4 *>(p.beta + 4 * i);
      }
      __syncthreads();
    } else {
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const int v = (FULL || lane + LPR * j < nvec) ? lane + LPR * j : 0;
#pragma unroll
        for (int q = 0; q < V / 4; ++q) {
          gr[j][q] = *reinterpret_cast<const float4 *>(p.gamma + V * v + 4 * q);
          br[j][q] = *reinterpret_cast<const float4 *>(p.beta + V * v + 4 * q);
        }
      }
    }
  }
  float x[NV][V];
  const float zr = (float)p.z_r + 128.0f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int v = lane + LPR * j;
    const bool ok = FULL || v < nvec;
#pragma unroll
    for (int e = 0; e < V; ++e) x[j][e] = (float)hv[j][e];
    if (p.r) {
      typename LnVec<V>::Half ho;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const uint32_t u = LnVec<V>::word(cw[j], e >> 2) ^ 0x80808080u;  // code + 128 in every byte
        const float t = x[j][e] + p.s_r * ((float)((u >> (8 * (e & 3))) & 0xff) - zr);  // whole numbers: exact
        ho[e] = (_Float16)t;
        x[j][e] = (float)ho[e];
      }
      if (p.h_out && live && ok) *reinterpret_cast<typename LnVec<V>::Half *>(p.h_out + at * p.ldho + V * v) = ho;
    }
    if (!ok) {
#pragma unroll
      for (int e = 0; e < V; ++e) x[j][e] = 0.0f;
    }
  }
  if (!p.x_q) return;
  const float mean = row_sum<LPR, NV, V, PAIRS>([&](float s, int j, int e) { return s + x[j][e]; }) * p.inv_c;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const bool ok = FULL || lane + LPR * j < nvec;
#pragma unroll
    for (int e = 0; e < V; ++e) x[j][e] = ok ? x[j][e] - mean : 0.0f;
  }
  const float var =
      row_sum<LPR, NV, V, PAIRS>([&](float s, int j, int e) { return __builtin_fmaf(x[j][e], x[j][e], s); }) * p.inv_c;
  const float rstd = __builtin_amdgcn_rsqf(var + p.eps);  // 1 ulp
  const float zf = (float)p.z_x, inv_s = p.inv_s_x;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int v = lane + LPR * j;
    const int vs = (FULL || v < nvec) ? v : 0;
    uint32_t w[V / 4];
#pragma unroll
    for (int q = 0; q < V / 4; ++q) {
      float4 g4, b4;
      if constexpr (kLds) {
        g4 = *reinterpret_cast<const float4 *>(s_gb + 1024 * q + 4 * vs);
        b4 = *reinterpret_cast<const float4 *>(s_gb + 2048 + 1024 * q + 4 * vs);
      } else {
        g4 = gr[j][q], b4 = br[j][q];
      }
      const float g[4] = {g4.x, g4.y, g4.z, g4.w}, b[4] = {b4.x, b4.y, b4.z, b4.w};
      float y[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = __builtin_fmaf(__builtin_fmaf(x[j][4 * q + e] * rstd, g[e], b[e]), inv_s, zf);
      w[q] = pack_codes(y);
    }
    if (live && (FULL || v < nvec)) *reinterpret_cast<typename LnVec<V>::Codes *>(p.x_q + at * p.ldxq + V * v) = LnVec<V>::pack(w);
  }
}

// A wavefront or 256 threads to a workgroup.
template <int LPR, int NV, bool FULL>
void launch_ln_form(const LnParams &p, bool wave, hipStream_t st) {
  if (wave) {
    constexpr int V = LPR == 64 ? 8 : 4, L = LPR * 8 / V;  // (no pairs of lanes for the widest rows)
    residual_ln_quant_kernel<L, NV, V, 64, FULL, V == 4><<<dim3((unsigned)ceil_div(p.m, 64 / L)), 64, 0, st>>>(p);
  } else {
    residual_ln_quant_kernel<LPR, NV, 8, 256, FULL><<<dim3((unsigned)ceil_div(p.m, 256 / LPR)), 256, 0, st>>>(p);
  }
}

// At most kLnMaxRows rows per launch (64 threads each: a grid counts fewer than 2^32 threads).
constexpr int64_t kLnMaxRows = (int64_t)1 << 25;

cwac_status launch_ln(const LnParams &p, hipStream_t st) {
  const int64_t m = p.m;
  const int c = p.c;
  // lanes per row and vectors of 8 channels per lane: the pair with the fewest idle vector slots, ties to the wider group
  const int nvec = c / 8;
  int lpr = 64, nv = (nvec + 63) / 64;
  for (int cand = 32; cand >= 16; cand /= 2) {
    const int cnv = (nvec + cand - 1) / cand;
    if (cnv <= 4 && cnv * cand < nv * lpr) lpr = cand, nv = cnv;
  }
  if (nvec != lpr * nv && c % 256 == 0) {  // no idle lane with V = 4: C = 1280 (12608 rows 17.4 -> 16.4 us) and 1792
    const dim3 grid((unsigned)m);
    if (c == 1280)
      residual_ln_quant_kernel<64, 5, 4, 64, true><<<grid, 64, 0, st>>>(p);
    else
      residual_ln_quant_kernel<64, 7, 4, 64, true><<<grid, 64, 0, st>>>(p);
    return launch_status();
  }
  // One wavefront to a workgroup (microseconds, 256 threads / this): 197 x 384 3.7 / 3.2, 2308 x 768 5.5 / 4.8, 7252 x 768
  // 10.5 / 10.0, 12608 x 768 15.7 / 14.7, 12608 x 384 9.8 / 9.3; level at 7252 x 192 and behind at 25216 x 192 (10.0 / 11.4) and
  // 25216 x 640 (20.9 / 21.5).  Rows of 64 lanes, where a lane keeps its 8 channels: 197 x 512 3.2 / 2.9, 25216 x 512 18.5 / 17.5,
  // 4616 x 1024 9.4 / 8.8, 7252 x 2048 20.7 / 20.4; level at 12608 x 1024 (17.9) and behind at 25216 x 2048 (54.7 / 60.0).
  const bool wave = lpr == 64 ? m <= 8192 || c <= 512 : m <= (c >= 256 ? 16384 : 2304);
#define CWAC_LN_CASE(L, N)                                                                          \
  if (lpr == L && nv == N) {                                                                        \
    if (nvec == L * N)                                                                              \
      launch_ln_form<L, N, true>(p, wave, st);                                                      \
    else                                                                                            \
      launch_ln_form<L, N, false>(p, wave, st);                                                     \
  }
  // clang-format off
  CWAC_LN_CASE(64, 1) else CWAC_LN_CASE(64, 2) else CWAC_LN_CASE(64, 3) else CWAC_LN_CASE(64, 4)
  else CWAC_LN_CASE(32, 1) else CWAC_LN_CASE(32, 2) else CWAC_LN_CASE(32, 3) else CWAC_LN_CASE(32, 4)
  else CWAC_LN_CASE(16, 1) else CWAC_LN_CASE(16, 2) else CWAC_LN_CASE(16, 3) else CWAC_LN_CASE(16, 4)
  else return CWAC_E_SHAPE;
  // clang-format on
#undef CWAC_LN_CASE
  return launch_status();
}

// ------------------------------------------------------------------------------------------
// GELU between fc1 and fc2 on int8 codes: a function of one code, so a 256-entry table.
// ------------------------------------------------------------------------------------------
__global__ void gelu_table_kernel(float s_in, int z_in, float s_out, int z_out, int8_t *table) {
  const int code = (int)threadIdx.x - 128;
  const double x = (double)s_in * (double)(code - z_in);
  const double g = 0.5 * x * (1.0 + erf(x * 0.70710678118654752440));
  double v = rint(g / (double)s_out + (double)z_out);
  v = fmin(fmax(v, -128.0), 127.0);
  table[threadIdx.x] = (int8_t)(int)v;
}

// out[i] = table[in[i] + 128]; 16 codes per lane and pass, the table in LDS (64 words: the lanes
// of a read hit distinct banks or the same word).  HBM bytes per element: 1 + 1.
__global__ __launch_bounds__(256) void table_lookup_kernel(const int8_t *in, int64_t ld_in, const int8_t *table,
                                                           int8_t *out, int64_t ld_out, int64_t m, int n) {
  __shared__ uint8_t s_tab[256];
  s_tab[threadIdx.x] = (uint8_t)table[threadIdx.x];
  __syncthreads();
  const int vec_per_row = n >> 4;
  const int64_t total = m * vec_per_row;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int64_t row = i / vec_per_row;
    const int v = (int)(i - row * vec_per_row);
    const v4i cw = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(in + row * ld_in + 16 * v));
    v4i ow;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t w = (uint32_t)cw[q];
      uint32_t o = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) o |= (uint32_t)s_tab[((w >> (8 * e)) & 0xff) ^ 0x80] << (8 * e);
      ow[q] = (int)o;
    }
    *reinterpret_cast<v4i *>(out + row * ld_out + 16 * v) = ow;
  }
}

// ------------------------------------------------------------------------------------------
// Multi-head self-attention, head width D = 64 or 32.  One wavefront owns 32 queries; K (as (code - z) in
// binary16, row-major, rows of 2 D + 16 bytes) and V (transposed, rows of 64 NT + 16 bytes) of 32 NT keys
// sit in LDS.  S^T = K Q^T: 32 x 32 x 16 MFMA tiles with keys along M, so a lane owns one query (its N
// index) and, with its partner lane ^ 32, all of that query's scores - the softmax is a reduction over the
// lane's own registers plus one exchange.  Registers 8u .. 8u + 7 of score tile t are, in order, the B operand
// of k-step (t, u) of O^T = V^T P^T; they hold keys 32 t + 16 u + 8 (e >> 2) + 4 half + (e & 3), so V^T is
// stored with the four quads of every 16 keys in the order 0, 2, 1, 3 and the A operand is one 16-byte read.
// Scores are exact integers; p is scaled by 1024 before its conversion to binary16 so that no term that
// matters falls into the subnormal range.
//
// What bounds it: the vector ALU - per score one fused multiply-add, one exponential, one addition, half a
// maximum and half a conversion - as long as enough wavefronts are resident to cover the loads of a head and
// the chain scores -> maximum -> exponentials -> second product.  Hence at most 128 registers (two workgroups
// of seven wavefronts to a compute unit), score tiles in pairs, a bias read a pair ahead, and a fill that moves
// 4 keys x D / 8 channels per thread: V is transposed in registers (8-byte LDS writes instead of 2-byte ones).
// Against one workgroup to a compute unit, 2-byte transposing writes and 224-query blocks of long sequences:
// 128 images x 12 heads x 197 tokens 45.5 -> 38.0 us, 8 x 12 x 577 32.1 -> 20.9, 148 x 16 x 49 with a bias
// 9.5 -> 8.5, one image 7.2 -> 6.6; blocks of 224 or 256 queries where attention_form says so.  Chunks of 64 or 192 keys, three,
// five or seven wavefronts and shorter chunks for 197 tokens were 5 to 150 % slower.
// ------------------------------------------------------------------------------------------
constexpr int kHeadDim = 64;     // widest head; 32 is the other width
constexpr int kMaxTokens = 4096; // longest sequence
// bytes per K row in LDS: the head's binary16 values + 16 (conflict-free 16-byte operand reads for both widths)
constexpr int k_stride(int d) { return 2 * d + 16; }
// bytes per V^T row in LDS: 2 * 32 * NT of keys + 16; four times an odd number of words, so the 16-byte operand
// reads of 16 consecutive rows cover all 64 banks once
constexpr int v_stride(int nt) { return 64 * nt + 16; }

struct AttnParams {
  const int8_t *r;
  int64_t ld;
  float s;
  int z;
  int tokens, heads;
  uint32_t pairs;  // batch * heads
  const uint16_t *bias;  // binary16 [heads][tokens][ldb] added to the logits, or NULL
  int64_t ldb;
  float s_a;
  int z_a;
  int8_t *a;
  int64_t lda;
};

// One thread's share of a chunk of keys: units of 4 keys x D / 8 channels, 64 per 32 keys.
template <int NT, int NW, int D>
struct AttnFill {
  static constexpr int kUnits = 64 * NT, kThreads = 64 * NW, kPer = (kUnits + kThreads - 1) / kThreads;
  static constexpr int kWords = D / 32;  // words of codes per key and unit
  uint32_t k[kPer][4][kWords], v[kPer][4][kWords];

  // Keys from key0 on; keys beyond the last token repeat it (their scores are masked, their weights zero).
  __device__ __forceinline__ void load(const int8_t *base, int64_t ld, int c, int key0, int tokens, int tid) {
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int i = tid + j * kThreads;
      if (kUnits % kThreads != 0 && i >= kUnits) break;
      const int quad = i >> 3, col = (i & 7) * (D / 8);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int key = key0 + 4 * quad + r;
        key = key < tokens ? key : tokens - 1;
        const int8_t *at = base + (uint32_t)(key * (int)ld + col);
        if constexpr (kWords == 2) {
          const uint2 kw = *reinterpret_cast<const uint2 *>(at + c), vw = *reinterpret_cast<const uint2 *>(at + 2 * c);
          k[j][r][0] = kw.x, k[j][r][1] = kw.y, v[j][r][0] = vw.x, v[j][r][1] = vw.y;
        } else {
          k[j][r][0] = *reinterpret_cast<const uint32_t *>(at + c);
          v[j][r][0] = *reinterpret_cast<const uint32_t *>(at + 2 * c);
        }
      }
    }
  }

  __device__ __forceinline__ void store(int8_t *s_k, int8_t *s_v, h2 zbias, int tid) const {
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int i = tid + j * kThreads;
      if (kUnits % kThreads != 0 && i >= kUnits) break;
      const int quad = i >> 3, col = (i & 7) * (D / 8);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int8_t *at = s_k + (4 * quad + r) * k_stride(D) + 2 * col;
        if constexpr (kWords == 2) {
          *reinterpret_cast<h8 *>(at) = codes_to_h8(make_uint2(k[j][r][0], k[j][r][1]), zbias);
        } else {
          h2 lo, hi;
          codes_to_h4(k[j][r][0], zbias, lo, hi);
          *reinterpret_cast<h4 *>(at) = h4{lo[0], lo[1], hi[0], hi[1]};
        }
      }
      // quads 0, 1, 2, 3 of 16 keys go to positions 0, 2, 1, 3
      int8_t *vt = s_v + col * v_stride(NT) + (quad >> 2) * 32 + ((quad & 1) << 4) + ((quad & 2) << 2);
#pragma unroll
      for (int w = 0; w < kWords; ++w)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          // channel 4 w + b of keys 0, 1 and of keys 2, 3: the byte under 0x64 with its sign bit flipped is 1024 + (code + 128)
          const uint32_t sel = 0x0c000c00u | ((4u + b) << 16) | (uint32_t)b;
          const uint32_t p01 = __builtin_amdgcn_perm(v[j][1][w], v[j][0][w], sel) ^ 0x64806480u;
          const uint32_t p23 = __builtin_amdgcn_perm(v[j][3][w], v[j][2][w], sel) ^ 0x64806480u;
          const h2 a = __builtin_bit_cast(h2, p01) - zbias, d = __builtin_bit_cast(h2, p23) - zbias;
          *reinterpret_cast<h4 *>(vt + (4 * w + b) * v_stride(NT)) = h4{a[0], a[1], d[0], d[1]};
        }
    }
  }
};

// Running state of one query: maximum of the logits the weights refer to (as the exponent offset
// 10 - max), lane-local sum of the weights and the output accumulators.
template <int D>
struct AttnState {
  float mx, eoff, sum;
  v16f oc[D / 32];
};

// A query's bias for a pair of key tiles, read one pair ahead (so the loads travel under the pair before).
// Rows are padded to whole key tiles; a second tile beyond the last one reads the last one again.
struct AttnBias {
  uint2 w[2][4];
  __device__ __forceinline__ void load(const uint16_t *row, int key0, int tokens, int half) {
    const int last = (tokens - 1) & ~31;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int key = key0 + 32 * t < last ? key0 + 32 * t : last;
#pragma unroll
      for (int g = 0; g < 4; ++g) w[t][g] = *reinterpret_cast<const uint2 *>(row + key + 8 * g + 4 * half);
    }
  }
};

// Scores of CNT key tiles from LDS tile t0 on - with a bias already as logits in the log2 domain -, minus infinity for keys
// beyond the `left` that are left of the sequence, and their maximum (in both lanes of a query).  HALF: only the first
// 16 keys of the (single) tile can be real.
template <int CNT, int D, bool BIAS, bool HALF>
__device__ __forceinline__ float attention_scores(int t0, const int8_t *s_k, const h8 (&fq)[D / 16], const AttnBias &bias, int left,
                                                  float lscale, int l32, int half, v16f (&sc)[CNT]) {
  constexpr int R = HALF ? 8 : 16;  // score registers of a tile that can hold real keys
#pragma unroll
  for (int t = 0; t < CNT; ++t) {
#pragma unroll
    for (int i = 0; i < 16; ++i) sc[t][i] = 0.0f;
#pragma unroll
    for (int s = 0; s < D / 16; ++s) {
      const h8 fk = *reinterpret_cast<const h8 *>(s_k + (32 * (t0 + t) + l32) * k_stride(D) + (2 * s + half) * 16);
      sc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fk, fq[s], sc[t], 0, 0, 0);
    }
  }
  // register 4 g + r of tile t is key 32 t + 8 g + 4 half + r of this lane's query
  if (BIAS) {
    // with a bias the scores become logits in the log2 domain first: x = S * lscale + bias * log2(e)
#pragma unroll
    for (int t = 0; t < CNT; ++t)
#pragma unroll
      for (int g = 0; g < R / 4; ++g) {
        const h2 b01 = __builtin_bit_cast(h2, bias.w[t][g].x), b23 = __builtin_bit_cast(h2, bias.w[t][g].y);
        const float bf[4] = {(float)b01[0], (float)b01[1], (float)b23[0], (float)b23[1]};
#pragma unroll
        for (int r = 0; r < 4; ++r)
          sc[t][4 * g + r] = __builtin_fmaf(bf[r], 1.44269504088896340736f, sc[t][4 * g + r] * lscale);
      }
  }
  float gmx = -1e30f;  // finite, so that a group whose keys are all masked by the bias has zero weights
#pragma unroll
  for (int t = 0; t < CNT; ++t) {
    if (32 * t + 2 * R > left) {  // only the last tile can hold padded keys (uniform branch)
#pragma unroll
      for (int i = 0; i < R; ++i)
        if (8 * (i >> 2) + (i & 3) >= left - 32 * t - 4 * half) sc[t][i] = -INFINITY;
    }
#pragma unroll
    for (int i = 0; i < R; ++i) gmx = fmaxf(gmx, sc[t][i]);
  }
  const uint32_t mine = __builtin_bit_cast(uint32_t, gmx);
  const auto both = __builtin_amdgcn_permlane32_swap(mine, mine, false, false);
  const uint32_t low = both[0], high = both[1];
  return fmaxf(__builtin_bit_cast(float, low), __builtin_bit_cast(float, high));
}

// Scores, softmax weights and the second product for CNT key tiles from LDS tile t0 on, whose first key is
// key0 + 32 t0 of the sequence.
// The weights always refer to the exact running maximum: the largest one is then 1024 and binary16 does not
// round it.  Rescaling only after a rise by more than 2^5 took 1-5 % less time, but its dominant weights are rounded
// while their sum is not: 128 x 197 tokens of peaked scores had 1.8 times the codes off against 64 bits (2.5e-3,
// here 1.4e-3).  STRAIGHT: rescale in every group, by 1 where nothing rose.  With the chunked kernel's free registers
// that is ahead of the branch (4 x 577 tokens 14.1 -> 13.4 us); the whole-sequence forms of 6 and 7 tiles spill for it
// (128 x 197: 39 -> 68 us).
template <int CNT, int D, int VS, bool BIAS, bool STRAIGHT, bool HALF = false>
__device__ __forceinline__ void attention_key_group(int t0, bool first, const int8_t *s_k, const int8_t *s_v,
                                                    const h8 (&fq)[D / 16], const AttnBias &bias, int left,
                                                    float lscale, int l32, int half, AttnState<D> &st) {
  constexpr int R = HALF ? 8 : 16;
  v16f sc[CNT];
  float gmx = attention_scores<CNT, D, BIAS, HALF>(t0, s_k, fq, bias, left, lscale, l32, half, sc);
  const float dscale = BIAS ? 1.0f : lscale;  // what turns a score difference into a log2 difference
  // 1024 p = exp2(S * lscale + (10 - mx * lscale)), one fused multiply-add per exponent
  if (first) {
    st.mx = gmx;
    st.eoff = __builtin_fmaf(-gmx, dscale, 10.0f);
  } else if (STRAIGHT || gmx > st.mx) {  // the same decision in both lanes of a query
    if (STRAIGHT) gmx = fmaxf(gmx, st.mx);
    const float eoff = __builtin_fmaf(-gmx, dscale, 10.0f);
    const float corr = __builtin_amdgcn_exp2f(eoff - st.eoff);  // of the offsets as they are used
    st.sum *= corr;
#pragma unroll
    for (int a = 0; a < D / 32; ++a)
#pragma unroll
      for (int i = 0; i < 16; ++i) st.oc[a][i] *= corr;
    st.mx = gmx;
    st.eoff = eoff;
  }
  const float eoff = st.eoff;
#pragma unroll
  for (int t = 0; t < CNT; ++t)
#pragma unroll
    for (int u = 0; u < R / 8; ++u) {
      h8 fp;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = sc[t][8 * u + e];
        const float w = __builtin_amdgcn_exp2f(BIAS ? x + eoff : __builtin_fmaf(x, lscale, eoff));  // exp2(-inf) = 0
        st.sum += w;
        fp[e] = (_Float16)w;
      }
#pragma unroll
      for (int a = 0; a < D / 32; ++a) {
        const h8 fv = *reinterpret_cast<const h8 *>(s_v + (32 * a + l32) * VS + (32 * (t0 + t) + 16 * u + 8 * half) * 2);
        st.oc[a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fv, fp, st.oc[a], 0, 0, 0);
      }
    }
}

// The NT tiles of a chunk in LDS, in pairs, from key key0 of the sequence on.  A sequence that does not come
// in CHUNKS has more than 32 (NT - 1) keys.  `bias` holds the first pair's on entry and, on exit, the next chunk's.
template <int NT, int D, bool BIAS, bool CHUNKS>
__device__ __forceinline__ void attention_chunk(int key0, int tokens, const int8_t *s_k, const int8_t *s_v,
                                                const h8 (&fq)[D / 16], const uint16_t *bias_row, AttnBias &bias,
                                                float lscale, int l32, int half, AttnState<D> &st) {
  constexpr int VS = v_stride(NT);
#pragma unroll
  for (int t0 = 0; t0 < NT; t0 += 2) {
    const int rest = tokens - key0 - 32 * t0;
    const bool f = key0 == 0 && t0 == 0;
    if (CHUNKS && rest <= 0) break;  // uniform over the wavefront
    const AttnBias now = bias;
    if (BIAS && (CHUNKS || t0 + 2 < NT)) bias.load(bias_row, key0 + 32 * t0 + 64, tokens, half);
    if (t0 + 1 < NT && (!CHUNKS || rest > 32))
      attention_key_group<2, D, VS, BIAS, CHUNKS>(t0, f, s_k, s_v, fq, now, rest, lscale, l32, half, st);
    else if (rest > 16)
      attention_key_group<1, D, VS, BIAS, CHUNKS>(t0, f, s_k, s_v, fq, now, rest, lscale, l32, half, st);
    else
      attention_key_group<1, D, VS, BIAS, CHUNKS, true>(t0, f, s_k, s_v, fq, now, rest, lscale, l32, half, st);
    __builtin_amdgcn_sched_barrier(0);  // one group's score tiles live at a time
  }
}

// Normalizes, quantizes and stores 32 channels of one query's output.  O^T: register 8 g .. of the tile is channel
// 8 g + 4 half + r of this lane's query; `sum` is the sum of its weights.
__device__ __forceinline__ void attention_store_tile(const AttnParams &p, float sum, const v16f &oc, int8_t *orow, int half,
                                                     bool store) {
  // sum and the accumulators both carry the factor 1024; the code is rne(O * s / (sum * s_a) + z_a)
  const float onorm = p.s / (sum * p.s_a), zf = (float)p.z_a;
  uint32_t packed[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    float v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = __builtin_fmaf(oc[4 * g + r], onorm, zf);
    packed[g] = pack_codes(v);
  }
  // lower half-wave holds channels 8g .. 8g+3, upper 8g+4 .. 8g+7: after the two swaps the lower
  // lane owns channels 0 .. 15 of this 32-channel tile and the upper lane 16 .. 31
  const auto s02 = __builtin_amdgcn_permlane32_swap(packed[0], packed[2], false, false);
  const auto s13 = __builtin_amdgcn_permlane32_swap(packed[1], packed[3], false, false);
  const v4i o = {(int)s02[0], (int)s02[1], (int)s13[0], (int)s13[1]};
  if (store) *reinterpret_cast<v4i *>(orow + 16 * half) = o;
}

// G heads per workgroup (short sequences: a head of two wavefronts alone would leave the compute unit to
// workgroup turnover), NW wavefronts (32 queries each) per head; the wavefronts of a head work only on that
// head's slice of LDS.  CHUNKS: the sequence passes through LDS in chunks of 32 NT keys, the next chunk's
// codes travelling in registers; otherwise it fits one.  gridDim.y counts blocks of 32 NW queries.
// Launch bounds: four wavefronts to a SIMD where the form fits 128 registers.  The biased 32-wide form of 6 tiles, like that of 7,
// does not: held to 128 it spilled 10 of them (3 x 16 x 192 tokens 9.0 us, now 7.4; 128 x 16 x 192 60 / 52).
template <int NT, int NW, int D, int G, bool BIAS, bool CHUNKS>
__global__ __launch_bounds__(64 * NW * G, D == 64 && BIAS ? 2 : (CHUNKS || (BIAS && NT > 5) ? 3 : 4)) void attention_int8_kernel(const AttnParams p) {
  constexpr int TP = 32 * NT;
  __shared__ __attribute__((aligned(16))) int8_t s_k_all[G * TP * k_stride(D)];
  __shared__ __attribute__((aligned(16))) int8_t s_v_all[G * D * v_stride(NT)];
  // which of the workgroup's heads: the same for a whole wavefront, so everything derived from it is scalar
  const int slot = G == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / (64 * NW));
  int8_t *s_k = s_k_all + slot * (TP * k_stride(D));
  int8_t *s_v = s_v_all + slot * (D * v_stride(NT));
  const int tid = threadIdx.x - slot * (64 * NW), lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  // (image, head) pairs beyond the last repeat it and store nothing (every wavefront reaches the barrier)
  uint32_t pair = blockIdx.x * G + slot;  // at most 2^31 pairs
  const bool live = pair < p.pairs;
  if (!live) pair = p.pairs - 1;
  const uint32_t image = pair / (uint32_t)p.heads;
  const int head = (int)(pair - image * p.heads);
  const int64_t row0 = (int64_t)image * p.tokens;
  const int c = p.heads * D;
  const int8_t *qbase = p.r + row0 * p.ld + head * D;

  const _Float16 zb = (_Float16)(float)(1152 + p.z);
  const h2 zbias = {zb, zb};
  // all of the thread's loads go out before the first conversion (one round trip to memory)
  AttnFill<NT, NW, D> fill;
  fill.load(qbase, p.ld, c, 0, p.tokens, tid);
  // this lane's query row as B operands (rows beyond the last token repeat it; never stored)
  const int q0 = (int)blockIdx.y * (32 * NW) + wave * 32, q = q0 + l32;
  const int qrow = q < p.tokens ? q : p.tokens - 1;
  const bool wave_live = q0 < p.tokens;  // otherwise it only helps to fill LDS
  // this lane's row of the bias: [head][query][key], rows padded to whole key tiles
  const uint16_t *bias_row = BIAS ? p.bias + ((int64_t)head * p.tokens + qrow) * p.ldb : nullptr;
  AttnBias bias;
  if (BIAS) bias.load(bias_row, 0, p.tokens, half);
  h8 fq[D / 16];
  {
    uint2 qraw[D / 16];
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
      qraw[s] = *reinterpret_cast<const uint2 *>(qbase + (uint32_t)(qrow * (int)p.ld + 16 * s + 8 * half));
    fill.store(s_k, s_v, zbias, tid);
#pragma unroll
    for (int s = 0; s < D / 16; ++s) fq[s] = codes_to_h8(qraw[s], zbias);
  }

  // s^2 / sqrt(D) * log2(e)
  const float lscale = p.s * p.s * (D == 64 ? 0.125f : 0.17677669529663687f) * 1.44269504088896340736f;
  AttnState<D> st;
  st.mx = 0.0f, st.eoff = 0.0f, st.sum = 0.0f;
#pragma unroll
  for (int a = 0; a < D / 32; ++a)
#pragma unroll
    for (int i = 0; i < 16; ++i) st.oc[a][i] = 0.0f;

  __syncthreads();
  if constexpr (!CHUNKS) {
    if (wave_live) attention_chunk<NT, D, BIAS, false>(0, p.tokens, s_k, s_v, fq, bias_row, bias, lscale, l32, half, st);
  } else {
    for (int key0 = 0;; key0 += TP) {
      const bool more = key0 + TP < p.tokens;  // uniform over the workgroup
      if (more) fill.load(qbase, p.ld, c, key0 + TP, p.tokens, tid);
      if (wave_live)
        attention_chunk<NT, D, BIAS, true>(key0, p.tokens, s_k, s_v, fq, bias_row, bias, lscale, l32, half, st);
      if (!more) break;
      __syncthreads();  // every wavefront is done with this chunk
      fill.store(s_k, s_v, zbias, tid);
      __syncthreads();
    }
  }
  if (wave_live) {
    const float sum = st.sum + __shfl_xor(st.sum, 32, 64);
#pragma unroll
    for (int a = 0; a < D / 32; ++a)
      attention_store_tile(p, sum, st.oc[a], p.a + (row0 + qrow) * p.lda + head * D + 32 * a, half, q < p.tokens && live);
  }
}

// Few heads (an image or two): a workgroup per (image, head, block of 32 queries) whose wavefronts split the keys.  What
// takes the time there is the chain of one wavefront through all key tiles on a few compute units; here wavefronts 0 .. 7
// take tiles wave, wave + 8, ... - one at 197 tokens - with K and V of a tile in their own slices of LDS.  The result is
// that of the kernel above bit for bit, so that an image's codes do not depend on how many images are with it:
// the tiles' maxima are exchanged, every weight refers to the running maximum of its pair of tiles as there, and the weights
// go through LDS to one wavefront per 32 channels, which adds the second products up in the order of the keys,
// and to one that adds up the weights.  These three hold a round's operands in registers, so that their chains run under
// the scores of the next round.
// us per call of a replayed graph, the kernel above / eight partial results merged at the end, which another number of images
// does not reproduce / this: one image of 12 heads and 197 tokens 7.5 / 5.4 / 5.7, of 577 tokens 13.4 / 9.0 / 9.2, of 16 heads
// and 257 tokens with a bias 10.2 / 6.9 / 7.3, windows of 16 heads of 32 and 144 tokens with a bias 6.0 / 4.7 / 4.8.  With the chains on
// wavefronts 0 to 2: 5.6, 10.0, 7.7, 4.8; with their operands read tile by tile, too: 6.1, 10.9, 7.9, 5.0.
constexpr int kSplitWaves = 8;
constexpr int split_threads(int d) { return 64 * (kSplitWaves + d / 32 + 1); }
template <int D, bool BIAS>
__global__ __launch_bounds__(split_threads(D)) void attention_split_kernel(const AttnParams p) {
  constexpr int NW = kSplitWaves, NO = D / 32, VS = v_stride(1);
  constexpr int KB = 32 * k_stride(D) > 4096 ? 32 * k_stride(D) : 4096;  // K of a tile, then its weights as summands
  constexpr int SLICE = KB + D * VS;
  __shared__ __attribute__((aligned(16))) int8_t s_mem[NW * SLICE];
  __shared__ __attribute__((aligned(16))) h8 s_p[NW][2][64];  // weights as operands of the second product
  __shared__ float s_max[NW][32], s_sum[32];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const uint32_t pair = blockIdx.x, image = pair / (uint32_t)p.heads;
  const int head = (int)(pair - image * p.heads);
  const int64_t row0 = (int64_t)image * p.tokens;
  const int c = p.heads * D;
  const int q = (int)blockIdx.y * 32 + l32, qrow = q < p.tokens ? q : p.tokens - 1;
  const int tiles = (p.tokens + 31) / 32, rounds = (tiles + NW - 1) / NW;
  const float lscale = p.s * p.s * (D == 64 ? 0.125f : 0.17677669529663687f) * 1.44269504088896340736f;
  const float dscale = BIAS ? 1.0f : lscale;
  float run = 0.0f;  // running maximum
  // exponent offsets of the four pairs of tiles of round i, from the tiles' maxima
  auto offsets = [&](int i, float(&eoff)[NW / 2]) {
#pragma unroll
    for (int g = 0; g < NW / 2; ++g) {
      const float gmx = fmaxf(s_max[2 * g][l32], s_max[2 * g + 1][l32]);
      run = i == 0 && g == 0 ? gmx : fmaxf(run, gmx);
      eoff[g] = __builtin_fmaf(-run, dscale, 10.0f);
    }
  };

  // Three barriers to a round: the maxima (and V) are there; the weights are there; both are read.
  if (wave < NW) {  // ---- scores and weights of a tile
    int8_t *s_k = s_mem + wave * SLICE, *s_v = s_k + KB;
    const int8_t *qbase = p.r + row0 * p.ld + head * D;
    const _Float16 zb = (_Float16)(float)(1152 + p.z);
    const h2 zbias = {zb, zb};
    const uint16_t *bias_row = BIAS ? p.bias + ((int64_t)head * p.tokens + qrow) * p.ldb : nullptr;
    AttnFill<1, 1, D> fill;
    AttnBias bias;
    if (wave < tiles) {
      fill.load(qbase, p.ld, c, 32 * wave, p.tokens, lane);
      if (BIAS) bias.load(bias_row, 32 * wave, p.tokens, half);
    }
    uint2 qraw[D / 16];
    h8 fq[D / 16];
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
      qraw[s] = *reinterpret_cast<const uint2 *>(qbase + (uint32_t)(qrow * (int)p.ld + 16 * s + 8 * half));
#pragma unroll
    for (int s = 0; s < D / 16; ++s) fq[s] = codes_to_h8(qraw[s], zbias);
    for (int i = 0; i < rounds; ++i) {
      const int tile = wave + NW * i;
      const bool mine = tile < tiles;
      v16f sc[1];
      float tmax = -1e30f;
      if (mine) {
        fill.store(s_k, s_v, zbias, lane);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const AttnBias now = bias;
        if (tile + NW < tiles) {
          fill.load(qbase, p.ld, c, 32 * (tile + NW), p.tokens, lane);
          if (BIAS) bias.load(bias_row, 32 * (tile + NW), p.tokens, half);
        }
        tmax = attention_scores<1, D, BIAS, false>(0, s_k, fq, now, p.tokens - 32 * tile, lscale, l32, half, sc);
      }
      if (half == 0) s_max[wave][l32] = tmax;
      __syncthreads();
      float eoff[NW / 2], off = 0.0f;
      offsets(i, eoff);
#pragma unroll
      for (int g = 0; g < NW / 2; ++g)
        if (wave >> 1 == g) off = eoff[g];
      if (mine) {
        v4f *s_w = reinterpret_cast<v4f *>(s_k) + lane;  // K of the tile has been read
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          h8 fp;
          float w[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float x = sc[0][8 * u + e];
            w[e] = __builtin_amdgcn_exp2f(BIAS ? x + off : __builtin_fmaf(x, lscale, off));
            fp[e] = (_Float16)w[e];
          }
          s_p[wave][u][lane] = fp;
          s_w[(2 * u) * 64] = v4f{w[0], w[1], w[2], w[3]};
          s_w[(2 * u + 1) * 64] = v4f{w[4], w[5], w[6], w[7]};
        }
      }
      __syncthreads();
      if (i + 1 < rounds) __syncthreads();
    }
    __syncthreads();
    return;
  }

  // ---- the chains through the tiles, everything that a round needs in registers first (asm: the compiler would move each
  // load down to its use).  Tiles beyond the last are read, whatever is there, and left out.
  float prev = 0.0f;  // exponent offset that the sums refer to
  if (wave < NW + NO) {
    const int a = wave - NW;
    v16f oc;
#pragma unroll
    for (int r = 0; r < 16; ++r) oc[r] = 0.0f;
    for (int i = 0; i < rounds; ++i) {
      const int here = tiles - NW * i < NW ? tiles - NW * i : NW;
      float eoff[NW / 2];
      h8 fv[NW][2], fp[NW][2];
      __syncthreads();
      offsets(i, eoff);
#pragma unroll
      for (int t = 0; t < NW; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u)
          fv[t][u] = *reinterpret_cast<const h8 *>(s_mem + t * SLICE + KB + (32 * a + l32) * VS + (16 * u + 8 * half) * 2);
#pragma unroll
      for (int t = 0; t < NW; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u) asm volatile("" : "+v"(fv[t][u]));
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NW; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u) fp[t][u] = s_p[t][u][lane];
#pragma unroll
      for (int t = 0; t < NW; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u) asm volatile("" : "+v"(fp[t][u]));
      if (i + 1 < rounds) __syncthreads();
#pragma unroll
      for (int t = 0; t < NW; ++t) {
        if (t >= here) break;
        if (t % 2 == 0) {
          const float corr = __builtin_amdgcn_exp2f(eoff[t / 2] - prev);  // of the offsets as they are used
          if (i > 0 || t > 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) oc[r] *= corr;
          }
          prev = eoff[t / 2];
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) oc = __builtin_amdgcn_mfma_f32_32x32x16_f16(fv[t][u], fp[t][u], oc, 0, 0, 0);
      }
    }
    __syncthreads();
    attention_store_tile(p, s_sum[l32], oc, p.a + (row0 + qrow) * p.lda + head * D + 32 * a, half, q < p.tokens);
  } else {
    float sum = 0.0f;
    for (int i = 0; i < rounds; ++i) {
      const int here = tiles - NW * i < NW ? tiles - NW * i : NW;
      float eoff[NW / 2];
      v4f w[NW][4];
      __syncthreads();
      offsets(i, eoff);
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NW; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g) w[t][g] = reinterpret_cast<const v4f *>(s_mem + t * SLICE)[g * 64 + lane];
#pragma unroll
      for (int t = 0; t < NW; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g) asm volatile("" : "+v"(w[t][g]));
      if (i + 1 < rounds) __syncthreads();
#pragma unroll
      for (int t = 0; t < NW; ++t) {
        if (t >= here) break;
        if (t % 2 == 0) {
          const float corr = __builtin_amdgcn_exp2f(eoff[t / 2] - prev);
          if (i > 0 || t > 0) sum *= corr;
          prev = eoff[t / 2];
        }
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
          for (int r = 0; r < 4; ++r) sum += w[t][g][r];
      }
    }
    sum += __shfl_xor(sum, 32, 64);
    if (half == 0) s_sum[l32] = sum;
    __syncthreads();
  }
}

template <int NT, int NW, int D, int G, bool CHUNKS>
cwac_status launch_attention(const AttnParams &p, hipStream_t st) {
  const dim3 grid((unsigned)ceil_div((int64_t)p.pairs, G), (unsigned)ceil_div(p.tokens, 32 * NW));
  if (p.bias)
    attention_int8_kernel<NT, NW, D, G, true, CHUNKS><<<grid, 64 * NW * G, 0, st>>>(p);
  else
    attention_int8_kernel<NT, NW, D, G, false, CHUNKS><<<grid, 64 * NW * G, 0, st>>>(p);
  return launch_status();
}

template <int D>
cwac_status launch_attention_d(const AttnParams &p, hipStream_t st) {
  switch (attention_form(p.tokens, p.pairs, D, p.bias != nullptr)) {
    case kAttnSplit: {
      const dim3 grid(p.pairs, (unsigned)ceil_div(p.tokens, 32));
      if (p.bias)
        attention_split_kernel<D, true><<<grid, split_threads(D), 0, st>>>(p);
      else
        attention_split_kernel<D, false><<<grid, split_threads(D), 0, st>>>(p);
      return launch_status();
    }
    // 256 threads per workgroup for short sequences
    case 1: return launch_attention<1, 1, D, 4, false>(p, st);
    case 2: return launch_attention<2, 2, D, 2, false>(p, st);
    case 3: return launch_attention<3, 3, D, 1, false>(p, st);
    case 4: return launch_attention<4, 4, D, 1, false>(p, st);
    case 5: return launch_attention<5, 5, D, 1, false>(p, st);
    case 6: return launch_attention<6, 6, D, 1, false>(p, st);
    case 7: return launch_attention<7, 7, D, 1, false>(p, st);
    case kAttnChunks: return launch_attention<4, 4, D, 1, true>(p, st);
    default: {  // kAttnChunksWide: without a bias
      constexpr int NW = attention_wide_waves(D);
      const dim3 grid(p.pairs, (unsigned)ceil_div(p.tokens, 32 * NW));
      attention_int8_kernel<4, NW, D, 1, false, true><<<grid, 64 * NW, 0, st>>>(p);
      return launch_status();
    }
  }
}

}  // namespace
}  // namespace cwac

using namespace cwac;

extern "C" {

cwac_status vit_residual_ln_quant(const uint16_t *h, int64_t ldh, const int8_t *r, int64_t ldr, float s_r,
                                  int32_t z_r, uint16_t *h_out, int64_t ldho, const float *gamma,
                                  const float *beta, float eps, float s_x, int32_t z_x, int8_t *x_q,
                                  int64_t ldxq, int64_t m, int32_t c, void *stream) {
  if (!h || (!r && !x_q)) return CWAC_E_NULL;
  if (x_q && (!gamma || !beta)) return CWAC_E_NULL;
  if (h_out && !r) return CWAC_E_MODE;
  if (m < 1 || c < 8 || c % 8 != 0 || c > 2048 || ldh < c || (r && ldr < c) || (h_out && ldho < c) ||
      (x_q && ldxq < c) || m > 0x7fffffff)
    return CWAC_E_SHAPE;
  if (!(s_x > 0.0f) && x_q) return CWAC_E_MODE;
  if (!aligned(h, 16) || ldh % 8 != 0 || (r && (!aligned(r, 8) || ldr % 8 != 0)) ||
      (h_out && (!aligned(h_out, 16) || ldho % 8 != 0)) || (x_q && (!aligned(x_q, 8) || ldxq % 8 != 0)) ||
      (x_q && (!aligned(gamma, 16) || !aligned(beta, 16))))
    return CWAC_E_ALIGN;
  LnParams p;
  p.h = reinterpret_cast<const _Float16 *>(h);
  p.ldh = ldh;
  p.r = r;
  p.ldr = ldr;
  p.s_r = s_r;
  p.z_r = z_r;
  p.h_out = reinterpret_cast<_Float16 *>(h_out);
  p.ldho = ldho;
  p.gamma = gamma;
  p.beta = beta;
  p.eps = eps;
  p.inv_s_x = x_q ? 1.0f / s_x : 1.0f;
  p.inv_c = 1.0f / (float)c;
  p.z_x = z_x;
  p.x_q = x_q;
  p.ldxq = ldxq;
  p.m = m;
  p.c = c;
  for (int64_t row = 0; row < m; row += kLnMaxRows) {
    LnParams q = p;
    q.m = m - row < kLnMaxRows ? m - row : kLnMaxRows;
    q.h += row * ldh;
    if (r) q.r += row * ldr;
    if (h_out) q.h_out += row * ldho;
    if (x_q) q.x_q += row * ldxq;
    const cwac_status st = launch_ln(q, as_stream(stream));
    if (st != CWAC_OK) return st;
  }
  return CWAC_OK;
}

cwac_status vit_gelu_table(float s_in, int32_t z_in, float s_out, int32_t z_out, int8_t *table, void *stream) {
  if (!table) return CWAC_E_NULL;
  if (!(s_in > 0.0f) || !(s_out > 0.0f)) return CWAC_E_MODE;
  gelu_table_kernel<<<1, 256, 0, as_stream(stream)>>>(s_in, z_in, s_out, z_out, table);
  return launch_status();
}

cwac_status vit_table_lookup(const int8_t *in, int64_t ld_in, const int8_t *table, int8_t *out, int64_t ld_out,
                             int64_t m, int32_t n, void *stream) {
  if (!in || !table || !out) return CWAC_E_NULL;
  if (m < 1 || n < 16 || n % 16 != 0 || ld_in < n || ld_out < n) return CWAC_E_SHAPE;
  if (!aligned(in, 16) || !aligned(out, 16) || ld_in % 16 != 0 || ld_out % 16 != 0) return CWAC_E_ALIGN;
  const int64_t vecs = m * (n / 16);
  int64_t blocks = ceil_div(vecs, 256);
  if (blocks > 256 * 16) blocks = 256 * 16;  // grid-stride beyond 16 workgroups per compute unit
  table_lookup_kernel<<<dim3((unsigned)blocks), 256, 0, as_stream(stream)>>>(in, ld_in, table, out, ld_out, m, n);
  return launch_status();
}

cwac_status vit_attention_int8(const int8_t *r_qkv, int64_t ld, float s, int32_t z, int32_t batch, int32_t tokens,
                               int32_t heads, int32_t head_dim, const uint16_t *bias, int64_t ldb, float s_a,
                               int32_t z_a, int8_t *a_q, int64_t lda, void *stream) {
  if (!r_qkv || !a_q) return CWAC_E_NULL;
  if (bias && (ldb < 32 * ((tokens + 31) / 32) || ldb % 4 != 0)) return CWAC_E_SHAPE;
  if (bias && !aligned(bias, 8)) return CWAC_E_ALIGN;
  if (head_dim != 64 && head_dim != 32) return CWAC_E_SHAPE;
  if (batch < 1 || tokens < 1 || tokens > kMaxTokens || heads < 1 || heads > 64) return CWAC_E_SHAPE;
  const int64_t c = (int64_t)heads * head_dim;
  if (ld < 3 * c || lda < c || (int64_t)batch * heads > 0x7fffffff) return CWAC_E_SHAPE;
  if (!(s > 0.0f) || !(s_a > 0.0f) || z < -128 || z > 127) return CWAC_E_MODE;
  if (!aligned(r_qkv, 8) || ld % 8 != 0 || !aligned(a_q, 16) || lda % 16 != 0) return CWAC_E_ALIGN;
  if (tokens * ld > 0x7fffffff) return CWAC_E_SHAPE;  // 32-bit row offsets inside one image
  AttnParams p;
  p.r = r_qkv;
  p.ld = ld;
  p.s = s;
  p.z = z;
  p.tokens = tokens;
  p.heads = heads;
  p.pairs = (uint32_t)batch * (uint32_t)heads;
  p.bias = bias;
  p.ldb = ldb;
  p.s_a = s_a;
  p.z_a = z_a;
  p.a = a_q;
  p.lda = lda;
  hipStream_t st = as_stream(stream);
  return head_dim == 64 ? launch_attention_d<64>(p, st) : launch_attention_d<32>(p, st);
}

size_t vit_block_workspace(int32_t batch, int32_t tokens, int32_t heads, int32_t hidden) {
  if (batch < 1 || tokens < 1 || heads < 1 || hidden < 1) return 0;
  const size_t m = (size_t)batch * (size_t)tokens, c = (size_t)heads * kHeadDim;
  return m * (5 * c + (size_t)hidden);
}

}  // extern "C"

namespace {

cwac_status check_block(const vit_block_params *bp) {
  if (!bp->gelu_table || !bp->ln1_gamma || !bp->ln1_beta || !bp->ln2_gamma || !bp->ln2_beta) return CWAC_E_NULL;
  if (bp->batch < 1 || bp->tokens < 1 || bp->heads < 1 || bp->heads > 64 || bp->hidden < 16 || bp->hidden % 16 != 0)
    return CWAC_E_SHAPE;
  if (bp->head_dim != 0 && bp->head_dim != 64 && bp->head_dim != 32) return CWAC_E_SHAPE;
  for (int i = 0; i < 4; ++i)
    if (!bp->layer[i].w_q || !bp->layer[i].mult || !bp->layer[i].offset) return CWAC_E_NULL;
  return CWAC_OK;
}

// One block.  x1_ready: the workspace already holds x1 = Q(LN1(h)) (the block before produced it with its
// last residual); next: the block that follows, whose LN1 and input quantizer then ride on this block's
// last residual pass.  h_out may be h: every kernel that writes the stream reads, in the same lanes, only
// the elements it writes, and the stream is otherwise read by earlier launches only.
cwac_status run_block(const vit_block_params *bp, bool x1_ready, const vit_block_params *next, const uint16_t *h,
                      uint16_t *h_out, void *workspace, void *stream) {
  const int64_t m = (int64_t)bp->batch * bp->tokens;
  const int32_t hd = bp->head_dim ? bp->head_dim : kHeadDim;
  const int32_t c = bp->heads * hd, hid = bp->hidden;
  int8_t *xq = static_cast<int8_t *>(workspace);  // x1, then the attention output, then x2 (then the next x1)
  int8_t *r_qkv = xq + m * c;
  int8_t *r_c = r_qkv + m * 3 * c;  // proj output, then fc2 output
  int8_t *r_h = r_c + m * c;        // GELU codes (fc1's output through the table)
  const vit_block_layer *L = bp->layer;
  auto params = [&](int i) {
    cwac_qparams qp;
    qp.mode = CWAC_EPI_INT_OFFSET;
    qp.act_per_token = 0;
    qp.s_x = L[i].s_x;
    qp.z_x = L[i].z_x;
    qp.s_r = L[i].s_r;
    qp.z_r = L[i].z_r;
    qp.qmin = -128;
    qp.qmax = 127;
    return qp;
  };
  auto linear = [&](int i, const int8_t *x, int32_t n, int32_t k, int8_t *out) {
    const cwac_qparams qp = params(i);
    return qlinear_cwac_forward(x, k, L[i].w_q, k, m, n, k, &qp, L[i].mult, L[i].offset, nullptr, nullptr, CWAC_OUT_INT8,
                                out, n, stream);
  };
  cwac_status st;
  if (!x1_ready) {
    st = vit_residual_ln_quant(h, c, nullptr, 0, 0.0f, 0, nullptr, 0, bp->ln1_gamma, bp->ln1_beta, bp->eps, L[0].s_x,
                               L[0].z_x, xq, c, m, c, stream);
    if (st != CWAC_OK) return st;
  }
  if ((st = linear(0, xq, 3 * c, c, r_qkv)) != CWAC_OK) return st;
  st = vit_attention_int8(r_qkv, 3 * c, L[0].s_r, L[0].z_r, bp->batch, bp->tokens, bp->heads, hd, bp->attn_bias, bp->attn_bias_ld,
                          L[1].s_x, L[1].z_x, xq, c, stream);
  if (st != CWAC_OK) return st;
  if ((st = linear(1, xq, c, c, r_c)) != CWAC_OK) return st;
  st = vit_residual_ln_quant(h, c, r_c, c, L[1].s_r, L[1].z_r, h_out, c, bp->ln2_gamma, bp->ln2_beta, bp->eps, L[2].s_x,
                             L[2].z_x, xq, c, m, c, stream);
  if (st != CWAC_OK) return st;
  {  // fc1 with the GELU table in its epilogue (large layers) or as a pass in place behind it
    const cwac_qparams qp = params(2);
    st = qlinear_cwac_forward_table(xq, c, L[2].w_q, c, m, hid, c, &qp, L[2].mult, L[2].offset, bp->gelu_table, r_h,
                                    hid, stream);
    if (st != CWAC_OK) return st;
  }
  if ((st = linear(3, r_h, c, hid, r_c)) != CWAC_OK) return st;
  // h2 = RN16(h1 + deq(r4)) in place over h1, with the next block's x1 = Q(LN1(h2)) in the same pass
  if (next)
    return vit_residual_ln_quant(h_out, c, r_c, c, L[3].s_r, L[3].z_r, h_out, c, next->ln1_gamma, next->ln1_beta,
                                 next->eps, next->layer[0].s_x, next->layer[0].z_x, xq, c, m, c, stream);
  return vit_residual_ln_quant(h_out, c, r_c, c, L[3].s_r, L[3].z_r, h_out, c, nullptr, nullptr, 0.0f, 1.0f, 0, nullptr,
                               0, m, c, stream);
}

}  // namespace

extern "C" {

cwac_status vit_block_w8a8_forward(const vit_block_params *bp, const uint16_t *h, uint16_t *h_out, void *workspace,
                                   size_t workspace_bytes, void *stream) {
  return vit_encoder_w8a8_forward(bp, 1, h, h_out, workspace, workspace_bytes, stream);
}

cwac_status vit_encoder_w8a8_forward(const vit_block_params *blocks, int32_t n_blocks, const uint16_t *h,
                                     uint16_t *h_out, void *workspace, size_t workspace_bytes, void *stream) {
  if (!blocks || !h || !h_out || !workspace) return CWAC_E_NULL;
  if (n_blocks < 1) return CWAC_E_SHAPE;
  for (int b = 0; b < n_blocks; ++b) {
    const cwac_status st = check_block(blocks + b);
    if (st != CWAC_OK) return st;
    if (blocks[b].batch != blocks[0].batch || blocks[b].tokens != blocks[0].tokens ||
        blocks[b].heads != blocks[0].heads || blocks[b].hidden != blocks[0].hidden ||
        blocks[b].head_dim != blocks[0].head_dim)  // (each block may bring its own attention bias)
      return CWAC_E_SHAPE;
  }
  if (workspace_bytes < vit_block_workspace(blocks[0].batch, blocks[0].tokens, blocks[0].heads, blocks[0].hidden))
    return CWAC_E_WORKSPACE;
  if (!aligned(workspace, 16)) return CWAC_E_ALIGN;
  for (int b = 0; b < n_blocks; ++b) {
    const cwac_status st = run_block(blocks + b, b > 0, b + 1 < n_blocks ? blocks + b + 1 : nullptr, b == 0 ? h : h_out,
                                     h_out, workspace, stream);
    if (st != CWAC_OK) return st;
  }
  return CWAC_OK;
}

}  // extern "C"
