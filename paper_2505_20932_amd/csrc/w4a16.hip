// Weight-only INT4 linear layer with the CWAC epilogue (LLM setting of Sec. 4.4: group-wise
// asymmetric 4-bit weights, group size 128, binary16 activations; compensation of Sec. 3.3
// folded into the epilogue as in Sec. 3.4), plus its quantizer, weight re-ordering and fold.
//
// Forward kernel: 256 x 256 output tile, eight wavefronts (2 x 4, each 128 tokens x 64 channels =
// 4 x 2 tiles of v_mfma_f32_32x32x16_f16, 128 fp32 accumulators per lane), one workgroup per
// compute unit, two wavefronts per SIMD.  Measured on this device with register-resident operands:
// beside one such MFMA (32 cycles of the matrix pipe) a SIMD issues about five vector ALU
// instructions per wavefront for free when two wavefronts share it, but only about three when one
// wavefront has it alone - and the weight expansion needs five per MFMA.
//   * Activation panels go global -> LDS directly (global_load_lds_dwordx4); one K stage is one
//     quantization group (128 channels = 256 bytes per row, 64 KiB per stage, two stages).  The
//     bank swizzle (16-byte chunk position XOR row & 15) is applied on the global-address side.
//   * Weights never touch LDS: they were re-ordered once into the order in which a wavefront's
//     lanes consume them, so each wavefront streams its own 4-bit codes with contiguous 1 KiB
//     loads straight into registers, one stage ahead, together with the group's scale and
//     zero-point, and expands them to binary16 MFMA operands right before use:
//     (code | 0x6400) is the binary16 number 1024 + code, so (1024 + c) - (1024 + z) and
//     fma(1024 + 16 c, 1/16, -(64 + z)) give c - z exactly with one packed instruction each,
//     and one packed multiply by the scale is the single rounding of RN16(s * (c - z)).
//   * Epilogue in registers: acc * mult[n] + fbias[n] (two fp32 operations), conversion to
//     binary16, transposition through a wave-private LDS slab, whole 128-byte line stores.
// The same kernel with 128-token tiles (two token blocks per wavefront) serves batches whose
// 128-token tiles fit the chip in one round; small batches (a decoding step, and up to several hundred tokens
// while its estimate is the lower one) take the weight-streaming kernel further down.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "qlinear_common.h"
#include "w4_rules.h"

namespace cwac {
namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) u4 GU4;        // in global memory (not a generic address)
typedef __attribute__((address_space(1))) uint32_t GU32;

#define CWAC_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))
#define CWAC_GLOBAL_PTR(p) ((const __attribute__((address_space(1))) void *)(p))

constexpr int wait_imm(int vmcnt, int lgkmcnt) {
  // gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] << 14 ; expcnt = 7 (no wait)
  return (vmcnt & 15) | (7 << 4) | ((lgkmcnt & 15) << 8) | (((vmcnt >> 4) & 3) << 14);
}

constexpr int kGroup = CWAC_W4_GROUP;  // input channels per scale / zero-point = per K stage
constexpr int kThreads = 256;

// ------------------------------------------------------------------------------------------
// Quantizer (Eq. 1-2, b = 4, per group): one wavefront per (output channel, group), two
// weights per lane.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void w4_quantize_kernel(const float *__restrict__ w, int64_t ldw,
                                                               int n, int groups,
                                                               uint8_t *__restrict__ codes,
                                                               uint16_t *__restrict__ scales,
                                                               uint8_t *__restrict__ zeros) {
  const int lane = threadIdx.x & 63;
  const int64_t task = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (task >= (int64_t)n * groups) return;
  const int r = (int)(task / groups), g = (int)(task - (int64_t)r * groups);
  const float2 v = *reinterpret_cast<const float2 *>(w + (int64_t)r * ldw + g * kGroup + 2 * lane);
  const float mn = wave_min(fminf(v.x, v.y)), mx = wave_max(fmaxf(v.x, v.y));
  const _Float16 sh = (_Float16)__fdiv_rn(mx - mn, 15.0f);  // round to nearest even
  uint16_t sb = __builtin_bit_cast(uint16_t, sh);
  if (sb < 0x0400u) sb = 0x0400u;   // zero or subnormal: 2^-14
  if (sb >= 0x7c00u) sb = 0x7bffu;  // never infinite
  const float s = (float)__builtin_bit_cast(_Float16, sb);
  float zf = rintf(__fdiv_rn(-mn, s));
  zf = fminf(fmaxf(zf, 0.0f), 15.0f);
  float c0 = rintf(__fdiv_rn(v.x, s)) + zf, c1 = rintf(__fdiv_rn(v.y, s)) + zf;
  c0 = fminf(fmaxf(c0, 0.0f), 15.0f);
  c1 = fminf(fmaxf(c1, 0.0f), 15.0f);
  const int64_t kk = (int64_t)groups * kGroup;
  *reinterpret_cast<uint16_t *>(codes + (int64_t)r * kk + g * kGroup + 2 * lane) =
      (uint16_t)((uint32_t)c0 | ((uint32_t)c1 << 8));
  if (lane == 0) {
    scales[(int64_t)r * groups + g] = sb;
    zeros[(int64_t)r * groups + g] = (uint8_t)zf;
  }
}

// ------------------------------------------------------------------------------------------
// Re-ordering into the forward kernel's streaming layout: one thread per output dword.
// dword index = (((n / 32) * (k / 64) + kb) * 64 + lane) * 4 + j, lane = 32 * h + n % 32; it
// holds the codes of input channels 64 * kb + 16 * j + 8 * h + e (e = 0..7) at nibble p(e).
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void w4_pack_kernel(const uint8_t *__restrict__ codes, int n, int k,
                                                           uint32_t *__restrict__ packed) {
  const int64_t total = (int64_t)n * (k / 8);
  for (int64_t d = (int64_t)blockIdx.x * kThreads + threadIdx.x; d < total;
       d += (int64_t)gridDim.x * kThreads) {
    const int j = (int)(d & 3), lane = (int)((d >> 2) & 63);
    const int64_t blk = d >> 8;
    const int kb64 = k / 64;
    const int nb = (int)(blk / kb64), kb = (int)(blk - (int64_t)nb * kb64);
    const int row = nb * 32 + (lane & 31), h = lane >> 5;
    const uint8_t *src = codes + (int64_t)row * k + kb * 64 + j * 16 + h * 8;
    const uint2 raw = *reinterpret_cast<const uint2 *>(src);  // 8 codes, 8-byte aligned
    uint32_t word = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t c = ((e < 4 ? raw.x : raw.y) >> (8 * (e & 3))) & 15u;
      const int p = (e >> 1) + 4 * (e & 1);  // (0, 4, 1, 5, 2, 6, 3, 7)
      word |= c << (4 * p);
    }
    packed[d] = word;
  }
}

__global__ __launch_bounds__(kThreads) void w4_pack_sz_kernel(const uint16_t *__restrict__ scales,
                                                              const uint8_t *__restrict__ zeros, int n,
                                                              int groups, uint32_t *__restrict__ sz) {
  const int64_t total = (int64_t)n * groups;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * kThreads) {
    const int g = (int)(i / n), r = (int)(i - (int64_t)g * n);
    sz[i] = (uint32_t)scales[(int64_t)r * groups + g] | ((uint32_t)zeros[(int64_t)r * groups + g] << 16);
  }
}

// Fold (Sec. 3.4 for a layer without requantization): mult = alpha, fbias = alpha * b + beta.
__global__ __launch_bounds__(kThreads) void fold_weight_only_kernel(const float *__restrict__ alpha,
                                                                    const float *__restrict__ beta,
                                                                    const float *__restrict__ bias, int n,
                                                                    float *__restrict__ mult,
                                                                    float *__restrict__ fbias) {
  const int c = blockIdx.x * kThreads + threadIdx.x;
  if (c >= n) return;
  const double a = alpha ? (double)alpha[c] : 1.0;
  const double be = beta ? (double)beta[c] : 0.0;
  const double b = bias ? (double)bias[c] : 0.0;
  mult[c] = (float)a;
  fbias[c] = (float)(__dadd_rn(__dmul_rn(a, b), be));
}

// ------------------------------------------------------------------------------------------
// Forward
// ------------------------------------------------------------------------------------------
struct W4Params {
  const char *x;  // binary16 [m, k]
  int64_t ldx_bytes;
  const u4 *wp;
  const uint32_t *sz;
  int64_t m;
  int n, k;
  const float *mult;
  const float *fbias;
  char *out;
  int64_t ldo;
  int tiles_m, tiles_n;
  int whole;  // tiled kernel: workgroups that take a whole tile
};

constexpr int kFwdThreads = 512;  // 8 wavefronts: 2 per SIMD
constexpr int kTA = 2;            // MFMA row blocks per wavefront: 64 channels
constexpr int kSlabStride = 144;
// Tile of WM x (8 / WM) wavefronts, each TB token blocks x kTA channel blocks of 32: (32 * TB * WM) tokens x
// (512 / WM) channels.  WM = 2: 256 channels x 256 tokens (TB = 4), or 128 tokens (TB = 2) for batches of a few
// hundred tokens, where one row of 256-token tiles would leave most compute units idle.  WM = 1 (TB = 4): 512
// channels x 128 tokens - every wavefront expands weights that no other wavefront of the tile needs (with WM = 2
// the two wavefronts of a channel block expand the same codes), so the tile spends half the vector work per MFMA.
template <int TB, int WM = 2>
struct W4Cfg {
  static_assert(WM == 1 || WM == 2, "wavefronts along the tokens");
  static constexpr int BM = 32 * TB * WM;
  static constexpr int BN = 64 * (8 / WM);
  static constexpr int STAGE_BYTES = BM * 256;  // BM rows x 128 binary16
  static constexpr int RING = 2 * STAGE_BYTES;
  static constexpr int XROWS = BM / 8;          // activation rows one wavefront fetches per stage
  static constexpr int XLOADS = XROWS / 4;      // global_load_lds per wavefront and stage (4 rows x 256 bytes each)
  static constexpr int SLAB_ROWS = 32 * TB;
  static constexpr int SLAB_BYTES = SLAB_ROWS * kSlabStride;
  // epilogue parameters sit behind the ring and the slabs
  static constexpr int PARAMS = 8 * SLAB_BYTES > RING ? 8 * SLAB_BYTES : RING;
  static constexpr int LDS = PARAMS + 2 * BN * 4;
  static_assert(LDS <= 160 * 1024, "LDS budget of one compute unit");
};

__device__ __forceinline__ h2 as_h2(uint32_t u) { return __builtin_bit_cast(h2, u); }

// Scale and zero-point of one weight row in the three forms the expansion needs.
struct GroupConst {
  h2 s, zlo, zhi;  // (s, s), (1024 + z) twice, (64 + z) twice
};
__device__ __forceinline__ GroupConst group_const(uint32_t sz) {
  GroupConst g;
  const uint32_t z = sz >> 16;
  g.s = as_h2((sz & 0xffffu) * 0x00010001u);
  g.zlo = as_h2(0x64006400u + z * 0x00010001u);  // 1024 + z: one unit per mantissa step
  g.zhi = as_h2(0x54005400u + z * 0x00100010u);  // 64 + z: sixteen mantissa steps per unit
  return g;
}

// Eight codes (one dword in the packed order) -> the MFMA operand of 8 consecutive input channels.
__device__ __forceinline__ h8 expand8(uint32_t w, const GroupConst &g) {
  const uint32_t w8 = w >> 8;
  const h2 t0 = as_h2((w & 0x000f000fu) | 0x64006400u);   // 1024 + c      channels 0, 1
  const h2 t1 = as_h2((w & 0x00f000f0u) | 0x64006400u);   // 1024 + 16 c   channels 2, 3
  const h2 t2 = as_h2((w8 & 0x000f000fu) | 0x64006400u);  //               channels 4, 5
  const h2 t3 = as_h2((w8 & 0x00f000f0u) | 0x64006400u);  //               channels 6, 7
  const h2 sixteenth = {(_Float16)0.0625f, (_Float16)0.0625f};
  const h2 d0 = t0 - g.zlo;                                        // c - z, exact
  const h2 d1 = __builtin_elementwise_fma(t1, sixteenth, -g.zhi);  // c - z, exact
  const h2 d2 = t2 - g.zlo;
  const h2 d3 = __builtin_elementwise_fma(t3, sixteenth, -g.zhi);
  const h2 r0 = d0 * g.s, r1 = d1 * g.s, r2 = d2 * g.s, r3 = d3 * g.s;  // the one rounding
  return h8{r0.x, r0.y, r1.x, r1.y, r2.x, r2.y, r3.x, r3.y};
}

// The same with the two masks in scalar registers and the exponent pattern in a vector register,
// which lets the compiler fuse every mask-and-set into one v_and_or_b32 (13 instead of 17
// instructions); pays where the expansion is what bounds the kernel.
struct ExpandConst {
  uint32_t mask_lo, mask_hi;  // wave-uniform
  uint32_t magic;             // per lane (the same value in all)
};
__device__ __forceinline__ ExpandConst expand_const() {
  ExpandConst c;
  c.mask_lo = 0x000f000fu;
  c.mask_hi = 0x00f000f0u;
  c.magic = 0x64006400u;
  asm volatile("" : "+s"(c.mask_lo), "+s"(c.mask_hi));  // opaque: not folded back into literals
  asm volatile("" : "+v"(c.magic));
  return c;
}
__device__ __forceinline__ h8 expand8(uint32_t w, const GroupConst &g, const ExpandConst &c) {
  const uint32_t w8 = w >> 8;
  const h2 t0 = as_h2((w & c.mask_lo) | c.magic);
  const h2 t1 = as_h2((w & c.mask_hi) | c.magic);
  const h2 t2 = as_h2((w8 & c.mask_lo) | c.magic);
  const h2 t3 = as_h2((w8 & c.mask_hi) | c.magic);
  const h2 sixteenth = {(_Float16)0.0625f, (_Float16)0.0625f};
  const h2 d0 = t0 - g.zlo;
  const h2 d1 = __builtin_elementwise_fma(t1, sixteenth, -g.zhi);
  const h2 d2 = t2 - g.zlo;
  const h2 d3 = __builtin_elementwise_fma(t3, sixteenth, -g.zhi);
  const h2 r0 = d0 * g.s, r1 = d1 * g.s, r2 = d2 * g.s, r3 = d3 * g.s;
  return h8{r0.x, r0.y, r1.x, r1.y, r2.x, r2.y, r3.x, r3.y};
}

template <int OUT_KIND, int ROWS>
__device__ __forceinline__ void store_slab(const int8_t *slab, char *gbase, int64_t row_bytes,
                                           int64_t rows_left, int lane) {
  const int rd_row = lane >> 3, rd_chunk = lane & 7;
#pragma unroll
  for (int i = 0; i < ROWS / 8; ++i) {
    const int row = i * 8 + rd_row;
    const u4 v = *reinterpret_cast<const u4 *>(slab + row * kSlabStride + rd_chunk * 16);
    u4 *dst = reinterpret_cast<u4 *>(gbase + row * row_bytes + rd_chunk * 16);
    if (row < rows_left) {
      // fp32 results (the calibration forward's Y_quant) are far larger than the caches and are
      // streamed out; binary16 results stay cacheable for the layer that consumes them
      if (OUT_KIND == CWAC_OUT_FP32)
        __builtin_nontemporal_store(v, dst);
      else
        *dst = v;
    }
  }
}

// Accumulator element 4*g + r of tile (a, b): channel n = bn0 + wave_n*64 + a*32 + 8*g + 4*half + r,
// token m = bm0 + wave_m*32*TB + b*32 + l32.  Each wavefront transposes its 32*TB rows x 128 bytes
// through a private LDS slab (row stride 144 bytes) and writes whole 128-byte lines: binary16
// output = all 64 channels of the wave tile in one slab, fp32 output = one slab per MFMA column.
template <int OUT_KIND, int TB, int WM>
__device__ __forceinline__ void w4_epilogue(const W4Params &p, v16f (&acc)[kTA][TB], int8_t *smem,
                                            const float *s_mult, const float *s_fb, int64_t bm0, int bn0,
                                            int wave_m, int wave_n, int lane) {
  constexpr int ESZ = OUT_KIND == CWAC_OUT_FP16 ? 2 : 4;
  constexpr int APS = OUT_KIND == CWAC_OUT_FP16 ? 2 : 1;  // MFMA columns per 128-byte slab row
  const int l32 = lane & 31, half = lane >> 5;
  const int wave = wave_m + WM * wave_n;
  int8_t *slab = smem + wave * W4Cfg<TB, WM>::SLAB_BYTES;
  const int64_t row_bytes = p.ldo * ESZ;
  const int64_t wrow0 = bm0 + wave_m * 32 * TB;
  char *wbase = p.out + (wrow0 * p.ldo + bn0 + wave_n * 64) * ESZ;
  const int64_t rows_left = p.m - wrow0;
#pragma unroll
  for (int a = 0; a < kTA; ++a) {
    float mu[4][4], fb[4][4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int cl = wave_n * 64 + a * 32 + 8 * g + 4 * half;  // channel inside the tile
      const float4 m4 = *reinterpret_cast<const float4 *>(s_mult + cl);
      mu[g][0] = m4.x; mu[g][1] = m4.y; mu[g][2] = m4.z; mu[g][3] = m4.w;
      const float4 f4 = *reinterpret_cast<const float4 *>(s_fb + cl);
      fb[g][0] = f4.x; fb[g][1] = f4.y; fb[g][2] = f4.z; fb[g][3] = f4.w;
    }
#pragma unroll
    for (int b = 0; b < TB; ++b) {
      const int row = b * 32 + l32;  // row inside the wave tile
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float u[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = acc[a][b][4 * g + r] * mu[g][r];  // mult == NULL: 1
          u[r] = v + fb[g][r];                              // fbias == NULL: +0
        }
        const int col = (a % APS) * 32 + 8 * g + 4 * half;  // channel inside the slab row
        if (OUT_KIND == CWAC_OUT_FP16) {
          const h2 lo = {(_Float16)u[0], (_Float16)u[1]}, hi = {(_Float16)u[2], (_Float16)u[3]};
          *reinterpret_cast<uint2 *>(slab + row * kSlabStride + col * 2) =
              make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi));
        } else {
          *reinterpret_cast<float4 *>(slab + row * kSlabStride + col * 4) = make_float4(u[0], u[1], u[2], u[3]);
        }
      }
    }
    if (a % APS == APS - 1)
      store_slab<OUT_KIND, 32 * TB>(slab, wbase + (a / APS) * 128, row_bytes, rows_left, lane);
  }
}

// One tile: 32 TB WM tokens from bm0 on (bm0 < m) x 512 / WM channels from bn0 on.
template <int OUT_KIND, int TB, int WM>
__device__ __forceinline__ void w4_tile(const W4Params &p, int64_t bm0, int bn0, int8_t *smem) {
  using Cfg = W4Cfg<TB, WM>;
  constexpr int BN = Cfg::BN;
  constexpr int kXLoads = Cfg::XLOADS, kStageBytes = Cfg::STAGE_BYTES, kParams = Cfg::PARAMS;
  float *s_mult = reinterpret_cast<float *>(smem + kParams);
  float *s_fb = reinterpret_cast<float *>(smem + kParams + BN * 4);

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wave_m = wave % WM, wave_n = wave / WM;  // WM x (8 / WM) wavefronts of 32*TB tokens x 64 channels
  const int l32 = lane & 31, half = lane >> 5;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);

  float p_mult = 1.0f, p_fb = 0.0f;
  if (tid < BN) {
    if (p.mult) p_mult = p.mult[bn0 + tid];
    if (p.fbias) p_fb = p.fbias[bn0 + tid];
  }

  // ---- activations, global -> LDS: wavefront `wave` owns XROWS consecutive rows, fetched 4
  // rows per load; lane = (row lr, slot pc) fetches 16-byte chunk pc ^ (row & 15) of its row
  const int lr = lane >> 4, pc = lane & 15;
  uint32_t xvo[kXLoads];
#pragma unroll
  for (int i = 0; i < kXLoads; ++i) {
    const int row = wave * Cfg::XROWS + i * 4 + lr;
    int64_t grow = bm0 + row;
    if (grow > p.m - 1) grow = p.m - 1;
    xvo[i] = (uint32_t)((grow - bm0) * p.ldx_bytes) + (uint32_t)((pc ^ (row & 15)) << 4);
  }
  const char *xtile = p.x + bm0 * p.ldx_bytes;
  // a wave-uniform 64-bit address that the compiler must keep in scalar registers, so that loads
  // take the (scalar base + 32-bit lane offset) form and need no vector address arithmetic
  auto uniform = [](const char *q) {
    const uint64_t v = reinterpret_cast<uint64_t>(q);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const char *>(((uint64_t)hi << 32) | lo);
  };
  auto issue_x = [&](int buf, int stage) {
    int8_t *sx = smem + buf * kStageBytes + wave_s * Cfg::XROWS * 256;
    const char *xk = uniform(xtile + (int64_t)stage * 256);
#pragma unroll
    for (int i = 0; i < kXLoads; ++i)
      __builtin_amdgcn_global_load_lds(CWAC_GLOBAL_PTR(xk + xvo[i]), CWAC_LDS_PTR(sx + i * 1024), 16, 0, 0);
  };

  // ---- weights, global -> registers: per MFMA row block a, 2 x 16 bytes per lane and stage
  const int kb64 = p.k / 64;
  const int n0w = bn0 + wave_s / WM * 64;  // first channel of this wavefront
  const uint32_t w_lane = (uint32_t)lane * 16u, sz_lane = (uint32_t)l32 * 4u;
  struct RawW {
    u4 c[kTA][2];
    uint32_t sz[kTA];
  };
  auto issue_w = [&](RawW &r, int stage) {
#pragma unroll
    for (int a = 0; a < kTA; ++a) {
      const int nb = (n0w + a * 32) >> 5;
      const char *wb = uniform(reinterpret_cast<const char *>(p.wp) +
                               ((int64_t)nb * kb64 + 2 * stage) * 1024);
      r.c[a][0] = *reinterpret_cast<const GU4 *>(CWAC_GLOBAL_PTR(wb + w_lane));
      r.c[a][1] = *reinterpret_cast<const GU4 *>(CWAC_GLOBAL_PTR(wb + 1024 + w_lane));
      const char *sb = uniform(reinterpret_cast<const char *>(p.sz) +
                               ((int64_t)stage * p.n + n0w + a * 32) * 4);
      r.sz[a] = *reinterpret_cast<const GU32 *>(CWAC_GLOBAL_PTR(sb + sz_lane));
    }
  };
  constexpr int kWLoads = 3 * kTA;

  // ---- LDS -> activation operand fragments
  const int x_off = (wave_m * 32 * TB + l32) * 256;
  const int swz_l = l32 & 15;
  auto read_x = [&](int buf, int kk, h8(&fx)[TB]) {
    const int8_t *base = smem + buf * kStageBytes + x_off + (((2 * kk + half) ^ swz_l) << 4);
#pragma unroll
    for (int b = 0; b < TB; ++b) fx[b] = *reinterpret_cast<const h8 *>(base + b * 32 * 256);
  };
  auto expand_w = [&](const RawW &r, const GroupConst (&gc)[kTA], int kk, h8(&fw)[kTA]) {
#pragma unroll
    for (int a = 0; a < kTA; ++a) fw[a] = expand8(r.c[a][kk >> 2][kk & 3], gc[a]);
  };

  v16f acc[kTA][TB];
#pragma unroll
  for (int a = 0; a < kTA; ++a)
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;
  auto mma = [&](const h8(&fw)[kTA], const h8(&fx)[TB]) {
#pragma unroll
    for (int a = 0; a < kTA; ++a)
#pragma unroll
      for (int b = 0; b < TB; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fw[a], fx[b], acc[a][b], 0, 0, 0);
  };
  // Scheduler hint for one k-step: first the LDS reads of the next step's activation fragments,
  // then kTA * TB MFMAs; the expansion of the next step's weight fragments (about
  // 35 vector ALU operations) spread evenly behind all of them; `vmem` loads spread likewise.
  auto interleave = [&](int vmem) {
    __builtin_amdgcn_sched_group_barrier(0x100, TB, 0);  // the next step's LDS reads go first
#pragma unroll
    for (int i = 0; i < kTA * TB; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (i < vmem) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 40 / (kTA * TB), 0);
    }
    __builtin_amdgcn_sched_barrier(0);  // one k-step per scheduling region
  };

  // ---- prologue.  Load order: X(0), W(0), X(1); waiting for all but the last kXLoads leaves X(1) in flight.
  const int stages = p.k / kGroup;
  RawW rawA, rawB;
  GroupConst gc[kTA];
  h8 fxA[TB], fxB[TB], fwA[kTA], fwB[kTA];
  issue_x(0, 0);
  issue_w(rawA, 0);
  if (stages > 1) issue_x(1, 1);
  if (tid < BN) {
    s_mult[tid] = p_mult;
    s_fb[tid] = p_fb;
  }
  if (stages > 1)
    __builtin_amdgcn_s_waitcnt(wait_imm(kXLoads, 0));
  else
    __builtin_amdgcn_s_waitcnt(wait_imm(0, 0));
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int a = 0; a < kTA; ++a) gc[a] = group_const(rawA.sz[a]);
  read_x(0, 0, fxA);
  expand_w(rawA, gc, 0, fwA);

  // One stage = one group.  `cur` holds this stage's codes (landed), `nxt` receives the next
  // stage's during k-step 0.  Every k-step fetches and expands the fragments of the following
  // one while its own MFMAs run.  Before the MFMAs of the last k-step every wavefront has fetched
  // its last fragments of this stage (its buffer is free for stage s + 2) and stage s + 1 has
  // landed; that k-step prepares the first fragments of the next stage.
  auto stage_body = [&](int s, int buf, RawW &cur, RawW &nxt) {
    const bool more = s + 1 < stages;
#pragma unroll
    for (int kk = 0; kk < 7; ++kk) {
      if (kk == 0 && more) issue_w(nxt, s + 1);
      if (kk & 1) {
        read_x(buf, kk + 1, fxA);
        expand_w(cur, gc, kk + 1, fwA);
        mma(fwB, fxB);
      } else {
        read_x(buf, kk + 1, fxB);
        expand_w(cur, gc, kk + 1, fwB);
        mma(fwA, fxA);
      }
      interleave(kk == 0 ? kWLoads : 0);
    }
    __builtin_amdgcn_s_waitcnt(wait_imm(0, 0));  // X(s + 1) and W(s + 1) have landed; fragments read
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (s + 2 < stages) issue_x(buf, s + 2);
    if (more) {
#pragma unroll
      for (int a = 0; a < kTA; ++a) gc[a] = group_const(nxt.sz[a]);  // this stage's are dead by now
      read_x(buf ^ 1, 0, fxA);
      expand_w(nxt, gc, 0, fwA);
    }
    mma(fwB, fxB);  // k-step 7
    interleave(kXLoads);
  };

  int s = 0;
  for (; s + 2 <= stages; s += 2) {
    stage_body(s, 0, rawA, rawB);
    stage_body(s + 1, 1, rawB, rawA);
  }
  if (s < stages) stage_body(s, 0, rawA, rawB);

  // every wavefront is past its last LDS read of the ring (the barrier of the last stage)
  w4_epilogue<OUT_KIND, TB, WM>(p, acc, smem, s_mult, s_fb, bm0, bn0, wave_m, wave_n, lane);
}

// Workgroups below p.whole take a tile each.  The others, PIECES to a tile, take 32 TB WM / PIECES tokens of one each: the
// tiles of a last round that would leave at least half of the compute units idle.  A piece expands the whole tile's
// weights, so it lasts longer than its share: about two thirds (halves) and half (quarters) of a tile.
template <int OUT_KIND, int TB, int WM, int PIECES>
__global__ __launch_bounds__(kFwdThreads) void w4a16_kernel(const W4Params p) {
  extern __shared__ __attribute__((aligned(16))) int8_t smem[];
  constexpr int BM = W4Cfg<TB, WM>::BM, BN = W4Cfg<TB, WM>::BN;
  int id = blockIdx.x, piece = 0;
  if (PIECES > 1 && id >= p.whole) {
    const int rest = p.tiles_m * p.tiles_n - p.whole, j = id - p.whole;
    piece = j / rest;
    id = p.whole + j - piece * rest;
  }
  int tile_m, tile_n;
  tile_of_block(id, p.tiles_m, p.tiles_n, tile_m, tile_n);
  int64_t bm0 = (int64_t)tile_m * BM;  // row edges: clamped loads, predicated stores
  int bn0 = tile_n * BN;
  if (bn0 > p.n - BN) bn0 = p.n - BN;  // channel edge: tile shifted inwards (n % 32 == 0)
  if constexpr (PIECES > 1) {
    if ((int)blockIdx.x >= p.whole) {
      bm0 += piece * (BM / PIECES);
      if (bm0 < p.m) w4_tile<OUT_KIND, TB / PIECES, WM>(p, bm0, bn0, smem);  // the last tile's later pieces can be empty
      return;
    }
  }
  w4_tile<OUT_KIND, TB, WM>(p, bm0, bn0, smem);
}

template <int OUT_KIND, int TB, int WM = 2, int PIECES = 1>
cwac_status launch_w4(W4Params p, hipStream_t st) {
  static const hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void *>(&w4a16_kernel<OUT_KIND, TB, WM, PIECES>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, W4Cfg<TB, WM>::LDS);
  if (attr != hipSuccess) return CWAC_E_LAUNCH;
  const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n, rest = PIECES > 1 ? tiles % 256 : 0;
  const int64_t blocks = tiles + rest * (PIECES - 1);
  if (blocks > 0x7fffffff) return CWAC_E_LAUNCH;
  p.whole = (int)(tiles - rest);
  w4a16_kernel<OUT_KIND, TB, WM, PIECES><<<dim3((unsigned)blocks), kFwdThreads, W4Cfg<TB, WM>::LDS, st>>>(p);
  return launch_status();
}

// ------------------------------------------------------------------------------------------
// Small batches (decoding steps, a few users).  The layer is bound by the stream of 4-bit weights and by the
// activations that every workgroup re-reads from the L2, not by the matrix cores.  A workgroup owns NB blocks of 32
// output channels and up to MP tokens (MB = ceil(MP / 32) MFMA columns) over the whole of K; its NW wavefronts
// split K, each a contiguous share of the units of 64 input channels.  Neither operand passes through registers on its
// way in: every wavefront owns a ring of D slots in LDS - per unit NB KiB of codes, the scale / zero-point words and the
// unit's 128-byte pieces of MP activation rows - that direct-to-LDS loads fill D units ahead of the arithmetic, with
// no barrier before the sums meet.  The activations come eight rows per instruction (whole 128-byte lines; a
// lane-per-row register load would touch a line per lane), the chunk position XORed with bits 1-3 of the row on
// the global side so that the MFMA operand reads are free of bank conflicts.  Rows beyond m lie behind the
// descriptor's extent and cost no memory traffic (their results are not stored).  Codes are expanded in registers, once
// for all MB columns.  The partial tiles are added in wavefront order through LDS (deterministic), by all threads,
// then the epilogue of the tiled kernel.  No workspace, no atomics.
// ------------------------------------------------------------------------------------------
template <int NB_, int MP_, int NW_, int D_>
struct StreamCfg {
  static constexpr int NB = NB_, MP = MP_, NW = NW_, D = D_;
  static constexpr int MB = (MP + 31) / 32;
  static constexpr int SZ_OFF = NB * 1024;              // behind the codes: 64 lanes x 4 bytes of scale words
  static constexpr int X_OFF = SZ_OFF + 256;
  static constexpr int SLOT = X_OFF + MP * 128;
  static constexpr int RING = D * SLOT;                 // of one wavefront; its partial tiles go over it
  static constexpr int L = NB + 1 + MP / 8;             // load instructions per unit
  static constexpr int PART = NB * MB * 4096;
  static constexpr int WAVE_BYTES = RING > PART ? RING : PART;
  static constexpr int LDS = NW * WAVE_BYTES;
  static constexpr bool FITS = LDS <= 160 * 1024 && D * L < 64;
  static_assert(MP % 8 == 0 && (NB == 1 || NB == 2), "whole loads; one scale load per unit");
};

// 64 lanes x 16 bytes from desc + offset (per lane) + k0 to 1 KiB of LDS (outside the kernel template: the host pass drops
// the stub of a template that passes dependent arguments to this builtin)
__device__ __forceinline__ void load_x_to_lds(__amdgpu_buffer_rsrc_t desc, int8_t *dst, int offset, int k0) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(desc, CWAC_LDS_PTR(dst), 16, offset, k0, 0, 0);
}

typedef float v4f __attribute__((ext_vector_type(4)));

// The epilogue of four channels of one token.
template <int OUT_KIND>
__device__ __forceinline__ void w4_store4(const W4Params &p, int64_t row, int ch, const v4f &sum) {
  constexpr int ESZ = OUT_KIND == CWAC_OUT_FP16 ? 2 : 4;
  float u[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float v = sum[r] * (p.mult ? p.mult[ch + r] : 1.0f);
    u[r] = v + (p.fbias ? p.fbias[ch + r] : 0.0f);
  }
  char *o = p.out + (row * p.ldo + ch) * ESZ;
  if (OUT_KIND == CWAC_OUT_FP16) {
    const h2 lo = {(_Float16)u[0], (_Float16)u[1]}, hi = {(_Float16)u[2], (_Float16)u[3]};
    *reinterpret_cast<uint2 *>(o) = make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi));
  } else {
    *reinterpret_cast<float4 *>(o) = make_float4(u[0], u[1], u[2], u[3]);
  }
}

template <int OUT_KIND, class S>
__global__ __launch_bounds__(64 * S::NW) void w4a16_stream_kernel(const W4Params p) {
  constexpr int NB = S::NB, MB = S::MB, MP = S::MP, NW = S::NW, D = S::D;
  extern __shared__ __attribute__((aligned(16))) int8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  int tile_m, tile_n;
  tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, tile_m, tile_n);
  const int64_t bm0 = (int64_t)tile_m * MP;
  const int rows = p.m - bm0 < MP ? (int)(p.m - bm0) : MP;
  int n0 = tile_n * (32 * NB);
  if (n0 > p.n - 32 * NB) n0 = p.n - 32 * NB;  // channel edge: shifted inwards (n % 32 == 0; the same values twice)
  const int kb64 = p.k / 64;
  const int u_begin = wave * kb64 / NW, mine = (wave + 1) * kb64 / NW - u_begin;
  int8_t *ring = smem + wave * S::WAVE_BYTES;

  const char *wrow = reinterpret_cast<const char *>(p.wp) + ((int64_t)(n0 >> 5) * kb64 + u_begin) * 1024 + lane * 16;
  const uint32_t *szp = p.sz + n0 + (NB == 2 ? lane : l32);
  const __amdgpu_buffer_rsrc_t xd = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char *>(p.x + bm0 * p.ldx_bytes), 0, (int)((int64_t)(rows - 1) * p.ldx_bytes + 2 * p.k), 0x00020000);
  const int lr = lane >> 3, pc = lane & 7;
  int xo[MP / 8];
#pragma unroll
  for (int t = 0; t < MP / 8; ++t) xo[t] = (8 * t + lr) * (int)p.ldx_bytes + ((pc ^ (lr >> 1) ^ ((t & 1) << 2)) << 4);
  auto issue = [&](int i, int slot_i) {  // this wavefront's unit i
    int8_t *slot = ring + slot_i * S::SLOT;
#pragma unroll
    for (int a = 0; a < NB; ++a)
      __builtin_amdgcn_global_load_lds(CWAC_GLOBAL_PTR(wrow + ((int64_t)a * kb64 + i) * 1024), CWAC_LDS_PTR(slot + a * 1024),
                                       16, 0, 0);
    __builtin_amdgcn_global_load_lds(CWAC_GLOBAL_PTR(szp + (int64_t)((u_begin + i) >> 1) * p.n),
                                     CWAC_LDS_PTR(slot + S::SZ_OFF), 4, 0, 0);
#pragma unroll
    for (int t = 0; t < MP / 8; ++t) load_x_to_lds(xd, slot + S::X_OFF + t * 1024, xo[t], (u_begin + i) * 128);
  };
  // two accumulators per tile where a wavefront has one tile only: consecutive MFMAs do not wait for each other
  constexpr int ACCS = NB * MB == 1 ? 2 : 1;
  v16f acc[ACCS][NB][MB];
#pragma unroll
  for (int c = 0; c < ACCS; ++c)
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
      for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[c][a][b][i] = 0.0f;
  const ExpandConst ec = expand_const();

  struct Unit {
    u4 c[NB];
    uint32_t sz[NB];
    h8 x[4][MB];
  };
  auto read = [&](int slot_i, Unit &u) {
    const int8_t *slot = ring + slot_i * S::SLOT;
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      u.c[a] = *reinterpret_cast<const u4 *>(slot + a * 1024 + lane * 16);
      u.sz[a] = *reinterpret_cast<const uint32_t *>(slot + S::SZ_OFF + (a * 32 + l32) * 4);
    }
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      const int row = b * 32 + l32 < MP ? b * 32 + l32 : MP - 1;
      const int8_t *base = slot + S::X_OFF + row * 128;
      const int sw = (row >> 1) & 7;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) u.x[kk][b] = *reinterpret_cast<const h8 *>(base + (((2 * kk + half) ^ sw) << 4));
    }
  };
  auto multiply = [&](const Unit &u) {
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      const GroupConst gc = group_const(u.sz[a]);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const h8 w = expand8(u.c[a][kk], gc, ec);
#pragma unroll
        for (int b = 0; b < MB; ++b)
          acc[kk % ACCS][a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w, u.x[kk][b], acc[kk % ACCS][a][b], 0, 0, 0);
      }
    }
  };

  // Memory operations return in order: with r units issued behind a unit, it is complete at r * L outstanding.
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < mine) issue(d, d);
  int slot_i = 0;
#pragma unroll 1
  for (int i = 0; i + D < mine; ++i) {
    __builtin_amdgcn_s_waitcnt(wait_imm((D - 1) * S::L, 15));
    asm volatile("" ::: "memory");  // the slot reads stay below the wait
    __builtin_amdgcn_sched_barrier(0);
    Unit u;
    read(slot_i, u);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_imm(63, 0));  // in registers before the next unit may land in the slot
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    issue(i + D, slot_i);
    multiply(u);
    slot_i = slot_i + 1 == D ? 0 : slot_i + 1;
  }
  auto last = [&](auto tag) {  // the last D units: nothing more to issue
    constexpr int behind = decltype(tag)::value;
    if (behind >= D || behind >= mine) return;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_imm(behind < D ? behind * S::L : 0, 15));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    Unit u;
    read(slot_i, u);
    multiply(u);
    slot_i = slot_i + 1 == D ? 0 : slot_i + 1;
  };
  static_assert(D <= 8, "one call per slot");
  last(std::integral_constant<int, 7>{});
  last(std::integral_constant<int, 6>{});
  last(std::integral_constant<int, 5>{});
  last(std::integral_constant<int, 4>{});
  last(std::integral_constant<int, 3>{});
  last(std::integral_constant<int, 2>{});
  last(std::integral_constant<int, 1>{});
  last(std::integral_constant<int, 0>{});
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  // partial tiles over this wavefront's own ring: [tile][q][lane] x 4 channels (accumulator elements 4q .. 4q + 3)
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        v4f t;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          t[r] = acc[0][a][b][4 * q + r];
          if (ACCS == 2) t[r] += acc[ACCS - 1][a][b][4 * q + r];
        }
        reinterpret_cast<v4f *>(ring)[((a * MB + b) * 4 + q) * 64 + lane] = t;
      }
  __syncthreads();
  // thread -> (token, four channels): consecutive threads take consecutive channels of a token
  constexpr int CG = NB * 8, GROUPS = MB * 32 * CG;
  for (int g = tid; g < GROUPS; g += 64 * NW) {
    const int cg = g % CG, row = g / CG;
    if (row >= rows) break;
    const int tile = (cg >> 3) * MB + (row >> 5);
    const int8_t *part = smem + (((tile * 4 + ((cg & 7) >> 1)) * 64 + (cg & 1) * 32 + (row & 31)) * 16);
    v4f sum = *reinterpret_cast<const v4f *>(part);
#pragma unroll
    for (int w = 1; w < NW; ++w) sum += *reinterpret_cast<const v4f *>(part + w * S::WAVE_BYTES);
    w4_store4<OUT_KIND>(p, bm0 + row, n0 + 4 * cg, sum);
  }
}

// ------------------------------------------------------------------------------------------
// Up to 16 tokens: the same scheme on tiles of 16 output channels.  What bounds a decoding step here is not the
// weight stream but what a compute unit does with it - thirteen vector instructions per eight codes, waits and
// LDS reads, about 0.4 us per unit of a wavefront -, so the channels have to be dealt out evenly: 32-channel tiles
// leave half of the compute units idle at n = 4096 and give 64 channels to some and 32 to others at n = 12288.
// A unit is one quantization group, 128 input channels x 16 output channels = 1 KiB of codes.  Lane (r, q) of the
// 16 x 16 x 32 MFMA takes channel r and, in step t, dword t of the 16 bytes that the packed layout keeps for (channel,
// input channels 64 (q >> 1) + 8 (q & 1) + 16 t ..): one load and one LDS read bring all four steps, and the activation
// operand follows with chunk 8 (q >> 1) + (q & 1) + 2 t of the token's 256-byte piece.  One token, cold weights, us, 32-channel tiles /
// these: 4096 x 4096 6.3 / 4.6, 4096 x 11008 12.0 / 8.1 (2.9 TB/s), 12288 x 4096 9.6 / 8.4 (3.2 TB/s), 2048 x 2048 4.3 / 3.3.  Rings of
// three or four slots and four wavefronts: within 4 % where one workgroup sits on a compute unit, up to 40 % slower
// where three do.
// ------------------------------------------------------------------------------------------
template <int MP_, int NW_, int D_>
struct Stream16Cfg {
  static constexpr int MP = MP_, NW = NW_, D = D_;
  static constexpr int SZ_OFF = 1024, X_OFF = SZ_OFF + 256;
  static constexpr int SLOT = X_OFF + MP * 256;
  static constexpr int RING = D * SLOT;
  static constexpr int L = 2 + MP / 4;  // load instructions per unit
  static constexpr int WAVE_BYTES = RING;
  static constexpr int LDS = NW * WAVE_BYTES;
  static_assert((MP == 8 || MP == 16) && RING >= 1024 && LDS <= 160 * 1024 && D * L < 64, "LDS budget, 6-bit load counter");
};

template <int OUT_KIND, class S>
__global__ __launch_bounds__(64 * S::NW) void w4a16_stream16_kernel(const W4Params p) {
  constexpr int MP = S::MP, NW = S::NW, D = S::D;
  extern __shared__ __attribute__((aligned(16))) int8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, quad = lane >> 4;
  const int n0 = blockIdx.x * 16;  // n % 32 == 0
  const int rows = (int)p.m;
  const int kb64 = p.k / 64, units = p.k / kGroup;
  const int u_begin = wave * units / NW, mine = (wave + 1) * units / NW - u_begin;
  int8_t *ring = smem + wave * S::WAVE_BYTES;

  // quad q of the lanes: 64-channel block q >> 1, half q & 1
  const char *wrow = reinterpret_cast<const char *>(p.wp) + ((int64_t)(n0 >> 5) * kb64 + 2 * u_begin + (quad >> 1)) * 1024 +
                     ((quad & 1) * 32 + (n0 & 16) + l16) * 16;
  const uint32_t *szp = p.sz + n0 + l16;
  const __amdgpu_buffer_rsrc_t xd = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p.x), 0,
                                                                      (int)((int64_t)(rows - 1) * p.ldx_bytes + 2 * p.k), 0x00020000);
  int xo[MP / 4];
#pragma unroll
  for (int t = 0; t < MP / 4; ++t) {  // 4 rows of 256 bytes per load, the chunk position XORed with the row
    const int row = 4 * t + quad;
    xo[t] = row * (int)p.ldx_bytes + ((l16 ^ row) << 4);
  }
  auto issue = [&](int i, int slot_i) {
    int8_t *slot = ring + slot_i * S::SLOT;
    __builtin_amdgcn_global_load_lds(CWAC_GLOBAL_PTR(wrow + (int64_t)i * 2048), CWAC_LDS_PTR(slot), 16, 0, 0);
    __builtin_amdgcn_global_load_lds(CWAC_GLOBAL_PTR(szp + (int64_t)(u_begin + i) * p.n), CWAC_LDS_PTR(slot + S::SZ_OFF), 4, 0, 0);
#pragma unroll
    for (int t = 0; t < MP / 4; ++t) load_x_to_lds(xd, slot + S::X_OFF + t * 1024, xo[t], (u_begin + i) * 256);
  };
  v4f acc[2] = {v4f{0.0f, 0.0f, 0.0f, 0.0f}, v4f{0.0f, 0.0f, 0.0f, 0.0f}};
  const ExpandConst ec = expand_const();
  struct Unit {
    u4 c;
    uint32_t sz;
    h8 x[4];
  };
  const int xrow = l16 < MP ? l16 : MP - 1;
  auto read = [&](int slot_i, Unit &u) {
    const int8_t *slot = ring + slot_i * S::SLOT;
    u.c = *reinterpret_cast<const u4 *>(slot + lane * 16);
    u.sz = *reinterpret_cast<const uint32_t *>(slot + S::SZ_OFF + l16 * 4);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int chunk = 8 * (quad >> 1) + (quad & 1) + 2 * t;
      u.x[t] = *reinterpret_cast<const h8 *>(slot + S::X_OFF + xrow * 256 + ((chunk ^ xrow) << 4));
    }
  };
  auto multiply = [&](const Unit &u) {
    const GroupConst gc = group_const(u.sz);
#pragma unroll
    for (int t = 0; t < 4; ++t)
      acc[t & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(expand8(u.c[t], gc, ec), u.x[t], acc[t & 1], 0, 0, 0);
  };

  // Memory operations return in order: with r units issued behind a unit, it is complete at r * L outstanding.
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < mine) issue(d, d);
  int slot_i = 0;
#pragma unroll 1
  for (int i = 0; i + D < mine; ++i) {
    __builtin_amdgcn_s_waitcnt(wait_imm((D - 1) * S::L, 15));
    asm volatile("" ::: "memory");  // the slot reads stay below the wait
    __builtin_amdgcn_sched_barrier(0);
    Unit u;
    read(slot_i, u);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_imm(63, 0));  // in registers before the next unit may land in the slot
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    issue(i + D, slot_i);
    multiply(u);
    slot_i = slot_i + 1 == D ? 0 : slot_i + 1;
  }
  auto last = [&](auto tag) {  // the last D units: nothing more to issue
    constexpr int behind = decltype(tag)::value;
    if (behind >= D || behind >= mine) return;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_imm(behind < D ? behind * S::L : 0, 15));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    Unit u;
    read(slot_i, u);
    multiply(u);
    slot_i = slot_i + 1 == D ? 0 : slot_i + 1;
  };
  static_assert(D <= 4, "one call per slot");
  last(std::integral_constant<int, 3>{});
  last(std::integral_constant<int, 2>{});
  last(std::integral_constant<int, 1>{});
  last(std::integral_constant<int, 0>{});
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  // partial tile over this wavefront's own ring: slot `lane` holds channels 4 quad .. 4 quad + 3 of token l16
  reinterpret_cast<v4f *>(ring)[lane] = acc[0] + acc[1];
  __syncthreads();
  if (tid < 64) {  // thread -> (token, four channels): consecutive threads take consecutive channels of a token
    const int cg = tid & 3, row = tid >> 2;
    if (row < rows) {
      const int8_t *part = smem + (cg * 16 + row) * 16;
      v4f sum = *reinterpret_cast<const v4f *>(part);
#pragma unroll
      for (int w = 1; w < NW; ++w) sum += *reinterpret_cast<const v4f *>(part + w * S::WAVE_BYTES);
      w4_store4<OUT_KIND>(p, row, n0 + 4 * cg, sum);
    }
  }
}

template <int NB, int MP, int NW, int D>
cwac_status launch_w4_stream_cfg(W4Params p, int out_kind, hipStream_t st) {
  using S = StreamCfg<NB, MP, NW, D>;
  if constexpr (!S::FITS) {  // a depth whose rings do not fit is lowered to one that does
    return launch_w4_stream_cfg<NB, MP, NW, D - 1>(p, out_kind, st);
  } else {
    p.tiles_m = (int)ceil_div(p.m, MP);
    p.tiles_n = (int)ceil_div(p.n, 32 * NB);
    const int64_t blocks = (int64_t)p.tiles_m * p.tiles_n;
    if (blocks > 0x7fffffff) return CWAC_E_LAUNCH;
    const dim3 grid((unsigned)blocks);
    if (out_kind == CWAC_OUT_FP16) {
      static const hipError_t attr = hipFuncSetAttribute(
          reinterpret_cast<const void *>(&w4a16_stream_kernel<CWAC_OUT_FP16, S>), hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS);
      if (attr != hipSuccess) return CWAC_E_LAUNCH;
      w4a16_stream_kernel<CWAC_OUT_FP16, S><<<grid, 64 * NW, S::LDS, st>>>(p);
    } else {
      static const hipError_t attr = hipFuncSetAttribute(
          reinterpret_cast<const void *>(&w4a16_stream_kernel<CWAC_OUT_FP32, S>), hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS);
      if (attr != hipSuccess) return CWAC_E_LAUNCH;
      w4a16_stream_kernel<CWAC_OUT_FP32, S><<<grid, 64 * NW, S::LDS, st>>>(p);
    }
    return launch_status();
  }
}

template <int MP, int NW, int D>
cwac_status launch_w4_stream16(const W4Params &p, int out_kind, hipStream_t st) {
  using S = Stream16Cfg<MP, NW, D>;
  const dim3 grid((unsigned)(p.n / 16));
  if (out_kind == CWAC_OUT_FP16) {
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&w4a16_stream16_kernel<CWAC_OUT_FP16, S>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS);
    if (attr != hipSuccess) return CWAC_E_LAUNCH;
    w4a16_stream16_kernel<CWAC_OUT_FP16, S><<<grid, 64 * NW, S::LDS, st>>>(p);
  } else {
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&w4a16_stream16_kernel<CWAC_OUT_FP32, S>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS);
    if (attr != hipSuccess) return CWAC_E_LAUNCH;
    w4a16_stream16_kernel<CWAC_OUT_FP32, S><<<grid, 64 * NW, S::LDS, st>>>(p);
  }
  return launch_status();
}

// waves / depth: the caller's overrides (cwac_tuning.w4_small_waves / w4_small_depth), which keep to 32 channels and at most
// 32 tokens per workgroup.
template <int NW>
cwac_status launch_w4_stream_forced(const W4Params &p, int depth, int out_kind, hipStream_t st) {
#define CWAC_W4_DEPTH(MP)                                                           \
  return depth == 3   ? launch_w4_stream_cfg<1, MP, NW, 3>(p, out_kind, st)         \
         : depth == 4 ? launch_w4_stream_cfg<1, MP, NW, 4>(p, out_kind, st)         \
                      : launch_w4_stream_cfg<1, MP, NW, 2>(p, out_kind, st)
  if (p.m <= 8) CWAC_W4_DEPTH(8);
  if (p.m <= 16) CWAC_W4_DEPTH(16);
  CWAC_W4_DEPTH(32);
#undef CWAC_W4_DEPTH
}

template <int I>
cwac_status launch_w4_stream_tile(const W4Params &p, int out_kind, hipStream_t st) {
  return launch_w4_stream_cfg<kW4Stream[I].nb, kW4Stream[I].mp, kW4Stream[I].nw, kW4Stream[I].depth>(p, out_kind, st);
}

cwac_status launch_w4_stream(const W4Params &p, int tile, int waves, int depth, int out_kind, hipStream_t st) {
  if (waves || depth)
    return waves == 4 ? launch_w4_stream_forced<4>(p, depth, out_kind, st) : launch_w4_stream_forced<8>(p, depth, out_kind, st);
  if (w4_stream16_pays(p.m, p.n, p.k))
    return p.m <= 8 ? launch_w4_stream16<8, 8, 2>(p, out_kind, st) : launch_w4_stream16<16, 8, 2>(p, out_kind, st);
  switch (tile) {
    case 0: return launch_w4_stream_tile<0>(p, out_kind, st);
    case 1: return launch_w4_stream_tile<1>(p, out_kind, st);
    case 2: return launch_w4_stream_tile<2>(p, out_kind, st);
    case 3: return launch_w4_stream_tile<3>(p, out_kind, st);
    case 4: return launch_w4_stream_tile<4>(p, out_kind, st);
    case 5: return launch_w4_stream_tile<5>(p, out_kind, st);
    case 6: return launch_w4_stream_tile<6>(p, out_kind, st);
    case 7: return launch_w4_stream_tile<7>(p, out_kind, st);
    case 8: return launch_w4_stream_tile<8>(p, out_kind, st);
  }
  static_assert(kW4StreamTiles == 9, "one case per tile");
  return CWAC_E_MODE;
}

int grid_for(int64_t items) {
  const int64_t b = ceil_div(items, kThreads);
  return (int)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

}  // namespace
}  // namespace cwac

using namespace cwac;

extern "C" {

cwac_status cwac_w4_quantize_groupwise(const float *w, int64_t ldw, int32_t n, int32_t k, uint8_t *codes,
                                       uint16_t *scales, uint8_t *zeros, void *stream) {
  if (!w || !codes || !scales || !zeros) return CWAC_E_NULL;
  if (n < 1 || k < kGroup || k % kGroup != 0 || ldw < k) return CWAC_E_SHAPE;
  if (!aligned(w, 8) || ldw % 2 != 0 || !aligned(codes, 2)) return CWAC_E_ALIGN;
  const int groups = k / kGroup;
  const int64_t tasks = (int64_t)n * groups;
  const int64_t blocks = ceil_div(tasks, kThreads / 64);
  if (blocks > 0x7fffffff) return CWAC_E_SHAPE;
  w4_quantize_kernel<<<dim3((unsigned)blocks), kThreads, 0, as_stream(stream)>>>(w, ldw, n, groups, codes,
                                                                                 scales, zeros);
  return launch_status();
}

size_t cwac_w4_packed_w_bytes(int32_t n, int32_t k) {
  if (n < 1 || k < 1) return 0;
  return (size_t)n * (size_t)k / 2;
}

cwac_status cwac_w4_pack(const uint8_t *codes, const uint16_t *scales, const uint8_t *zeros, int32_t n,
                         int32_t k, void *packed_w, uint32_t *packed_sz, void *stream) {
  if (!codes || !scales || !zeros || !packed_w || !packed_sz) return CWAC_E_NULL;
  if (n < 32 || n % 32 != 0 || k < kGroup || k % kGroup != 0) return CWAC_E_SHAPE;
  if (!aligned(codes, 8) || !aligned(packed_w, 16) || !aligned(packed_sz, 4)) return CWAC_E_ALIGN;
  hipStream_t st = as_stream(stream);
  w4_pack_kernel<<<grid_for((int64_t)n * (k / 8)), kThreads, 0, st>>>(codes, n, k,
                                                                      static_cast<uint32_t *>(packed_w));
  if (launch_status() != CWAC_OK) return CWAC_E_LAUNCH;
  w4_pack_sz_kernel<<<grid_for((int64_t)n * (k / kGroup)), kThreads, 0, st>>>(scales, zeros, n, k / kGroup,
                                                                              packed_sz);
  return launch_status();
}

cwac_status cwac_fold_weight_only(const float *alpha, const float *beta, const float *bias, int32_t n_out,
                                  float *mult, float *fbias, void *stream) {
  if (!mult || !fbias) return CWAC_E_NULL;
  if ((alpha == nullptr) != (beta == nullptr)) return CWAC_E_MODE;
  if (n_out < 1) return CWAC_E_SHAPE;
  fold_weight_only_kernel<<<grid_for(n_out), kThreads, 0, as_stream(stream)>>>(alpha, beta, bias, n_out, mult,
                                                                                fbias);
  return launch_status();
}

cwac_status qlinear_w4a16_cwac_forward_ex(const uint16_t *x, int64_t ldx, const void *packed_w,
                                          const uint32_t *packed_sz, int64_t m, int32_t n, int32_t k,
                                          const float *mult, const float *fbias, int32_t out_kind, void *out,
                                          int64_t ldo, const cwac_tuning *tuning, void *stream_handle) {
  if (!x || !packed_w || !packed_sz || !out) return CWAC_E_NULL;
  if (out_kind != CWAC_OUT_FP16 && out_kind != CWAC_OUT_FP32) return CWAC_E_MODE;
  const int w4_tile = tuning ? tuning->w4_tile : 0, small_waves = tuning ? tuning->w4_small_waves : 0;
  const int small_depth = tuning ? tuning->w4_small_depth : 0;
  if ((w4_tile != 0 && w4_tile != 256 && w4_tile != 128 && w4_tile != 512) || (w4_tile == 512 && n < 512) ||
      (small_waves != 0 && small_waves != 4 && small_waves != 8) || (small_depth != 0 && (small_depth < 2 || small_depth > 4)))
    return CWAC_E_MODE;
  if (m < 1 || n < 256 || n % 32 != 0 || k < kGroup || k > 32768 || k % kGroup != 0 || ldx < k || ldo < n)
    return CWAC_E_SHAPE;
  const int64_t esz = out_kind == CWAC_OUT_FP16 ? 2 : 4;
  if (!aligned(x, 16) || ldx % 8 != 0 || !aligned(packed_w, 16) || !aligned(packed_sz, 4) ||
      !aligned(out, 16) || (ldo * esz) % 16 != 0)
    return CWAC_E_ALIGN;
  if (ceil_div(m, 256) > 0x7fffff) return CWAC_E_SHAPE;
  // per-lane activation offsets inside a tile are 32-bit
  if (255 * ldx * 2 + 32768 * 2 > 0xffffffffLL) return CWAC_E_SHAPE;
  W4Params p;
  p.x = reinterpret_cast<const char *>(x);
  p.ldx_bytes = ldx * 2;
  p.wp = static_cast<const u4 *>(packed_w);
  p.sz = packed_sz;
  p.m = m;
  p.n = n;
  p.k = k;
  p.mult = mult;
  p.fbias = fbias;
  p.out = static_cast<char *>(out);
  p.ldo = ldo;
  p.tiles_n = (int)ceil_div(n, 256);
  // The caller's override (results agree to the rounding of the fp32 sums): w4_tile = 256 keeps the
  // 256-token tiles at every batch size, 128 the 128-token tiles.  Otherwise the weight-streaming kernel where it pays.
  const int stream_tile = w4_stream_tile(m, n, k);
  if (w4_tile == 0 && w4_stream_pays(m, n, k, stream_tile))
    return launch_w4_stream(p, stream_tile, small_waves, small_depth, out_kind, as_stream(stream_handle));
  // 128-token tiles while they fit the chip in one round (one tile per compute unit): a half tile
  // takes about two thirds of a full tile's time (the weight expansion is per channel block, not
  // per token, so it spends more vector work per MFMA), which pays exactly while the full tiles
  // would leave compute units idle
  const bool half = w4_tile == 128 || (w4_tile == 0 && ceil_div(m, 128) * p.tiles_n <= kW4HalfTileUpTo);
  if (half) {
    p.tiles_m = (int)ceil_div(m, 128);
    return out_kind == CWAC_OUT_FP16 ? launch_w4<CWAC_OUT_FP16, 2>(p, as_stream(stream_handle))
                                     : launch_w4<CWAC_OUT_FP32, 2>(p, as_stream(stream_handle));
  }
  // large batches: the tile of 512 channels x 128 tokens (no wavefront expands another one's weights)
  if (w4_tile == 512 || (w4_tile == 0 && n >= 512)) {
    p.tiles_m = (int)ceil_div(m, 128);
    p.tiles_n = (int)ceil_div(n, 512);
    const int pieces = w4_pieces((int64_t)p.tiles_m * p.tiles_n);
    if (pieces == 4)
      return out_kind == CWAC_OUT_FP16 ? launch_w4<CWAC_OUT_FP16, 4, 1, 4>(p, as_stream(stream_handle))
                                       : launch_w4<CWAC_OUT_FP32, 4, 1, 4>(p, as_stream(stream_handle));
    if (pieces == 2)
      return out_kind == CWAC_OUT_FP16 ? launch_w4<CWAC_OUT_FP16, 4, 1, 2>(p, as_stream(stream_handle))
                                       : launch_w4<CWAC_OUT_FP32, 4, 1, 2>(p, as_stream(stream_handle));
    return out_kind == CWAC_OUT_FP16 ? launch_w4<CWAC_OUT_FP16, 4, 1>(p, as_stream(stream_handle))
                                     : launch_w4<CWAC_OUT_FP32, 4, 1>(p, as_stream(stream_handle));
  }
  p.tiles_m = (int)ceil_div(m, 256);
  return out_kind == CWAC_OUT_FP16 ? launch_w4<CWAC_OUT_FP16, 4>(p, as_stream(stream_handle))
                                   : launch_w4<CWAC_OUT_FP32, 4>(p, as_stream(stream_handle));
}

cwac_status qlinear_w4a16_cwac_forward(const uint16_t *x, int64_t ldx, const void *packed_w,
                                       const uint32_t *packed_sz, int64_t m, int32_t n, int32_t k,
                                       const float *mult, const float *fbias, int32_t out_kind, void *out,
                                       int64_t ldo, void *stream) {
  return qlinear_w4a16_cwac_forward_ex(x, ldx, packed_w, packed_sz, m, n, k, mult, fbias, out_kind, out, ldo,
                                       nullptr, stream);
}

}  // extern "C"
