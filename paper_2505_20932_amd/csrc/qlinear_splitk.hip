// Small-problem kernel of the quantized linear layer with the CWAC epilogue (Sec. 3.4, Eq. 10): few tokens
// (a decoding step, one image) or few output tiles.
//
// What bounds these layers is not the matrix cores but the time until the operands arrive: a decoding step
// reads every weight once (HBM), a single image's layer is a few microseconds of round trips.  A tile kernel
// that steps through K pays one round trip and two barriers per step and, with 64 x 64 tiles, occupies a
// fraction of the chip.  Here
//   * the tile is small (16 TN channels x 16 TM tokens), so that there are tiles for all compute units;
//   * the W wavefronts of a workgroup split K instead of the tile: every operand byte is fetched by exactly
//     one wavefront of the workgroup, and int32 sums make the split exact;
//   * each wavefront streams its range of K through a ring of D units (128 bytes of K) of its own in LDS, filled by
//     direct-to-LDS buffer loads: no barrier before the sums meet.  LDS is there for the access pattern
//     only: a load covers 8 rows of 128 contiguous bytes.  Fetching the MFMA fragments straight into
//     registers instead (16 rows, 16 bytes per lane, neighbouring lanes in different rows) ran at 16
//     bytes per clock and compute unit, a quarter of the L1's rate: 25 us against 10 at 16 x 12288 x 4096;
//   * rows past the last token or channel lie behind the descriptor's extent: such lanes touch no memory;
//   * the partial tiles meet in LDS once, and the whole epilogue runs on the sums, four consecutive channels
//     per thread.
#include <type_traits>

#include "qlinear_common.h"

namespace cwac {
namespace {

#define CWAC_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

// Partial sums in LDS: 1 KiB per 16 x 16 tile; slot 16 q + t (16 bytes) holds channels 4q .. 4q + 3 of token t, which
// the matrix instruction leaves in that lane.

template <int TN, int TM, int W, int D>
struct SplitCfg {
  static constexpr int BN = 16 * TN, BM = 16 * TM, NT = 64 * W;
  static constexpr int UK = 128;                        // bytes of K per unit
  static constexpr int W_BYTES = BN * UK, UNIT = (BN + BM) * UK;
  static constexpr int LPU = 2 * (TN + TM);             // loads per unit: 8 rows x 128 bytes each
  static constexpr int RING = D * UNIT;                 // of one wavefront
  static constexpr int SLAB = TN * TM * 1024;           // its partial tile, over its own ring
  static constexpr int PARAM = W * RING;                // offset, mult, fbias [BN], row scale [BM], code table [256 bytes]
  static constexpr int LDS_BYTES = PARAM + 12 * BN + 4 * BM + 256;
  static_assert(SLAB <= RING && LDS_BYTES <= 160 * 1024 && D * LPU < 64, "LDS budget, 6-bit load counter");
};

// 64 lanes x 16 bytes from desc + offset (per lane) + k0 to 1 KiB of LDS.  (Outside the kernel template: the host
// pass drops the stub of a template that passes dependent arguments to this builtin.)
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t desc, int8_t *dst, int offset, int k0) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(desc, CWAC_LDS_PTR(dst), 16, offset, k0, 0, 0);
}

template <int N>
__device__ __forceinline__ void wait_loads() {  // at most N loads of this wavefront outstanding
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

template <int TN, int TM, int W, int D, int OUT_KIND, bool INT_ONLY>
__global__ __launch_bounds__(64 * W) void qlinear_splitk_kernel(const FwdParams p) {
  using C = SplitCfg<TN, TM, W, D>;
  extern __shared__ __attribute__((aligned(16))) int8_t smem[];
  int32_t *s_off = reinterpret_cast<int32_t *>(smem + C::PARAM);
  float *s_mult = reinterpret_cast<float *>(s_off + C::BN);
  float *s_fb = s_mult + C::BN;
  float *s_rs = s_fb + C::BN;
  int32_t *s_tab = reinterpret_cast<int32_t *>(s_rs + C::BM);

  int tile_m, tile_n;
  tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, tile_m, tile_n);
  const int64_t bm0 = (int64_t)tile_m * C::BM;
  const int bn0 = tile_n * C::BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, quad = lane >> 4;

  const int rows_m = p.m - bm0 < C::BM ? (int)(p.m - bm0) : C::BM;
  const int rows_n = p.n - bn0 < C::BN ? p.n - bn0 : C::BN;
  const __amdgpu_buffer_rsrc_t xd = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t *>(p.x + bm0 * p.ldx), 0, (int)((int64_t)(rows_m - 1) * p.ldx + p.k), 0x00020000);
  const __amdgpu_buffer_rsrc_t wd = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t *>(p.w + (int64_t)bn0 * p.ldw), 0, (int)((int64_t)(rows_n - 1) * p.ldw + p.k), 0x00020000);
  // ---- global -> LDS: lane = (row lr, 16-byte slot pc) inside a load of 8 rows; the slot of a chunk is XORed with
  // bits 1-3 of the row (on the global side), so that 16 lanes reading one chunk of 16 rows hit distinct banks
  const int lr = lane >> 3, pc = lane & 7;
  int wv[2 * TN], xv[2 * TM];
#pragma unroll
  for (int j = 0; j < 2 * TN; ++j) wv[j] = (j * 8 + lr) * (int)p.ldw + ((pc ^ (lr >> 1) ^ ((j & 1) << 2)) << 4);
#pragma unroll
  for (int j = 0; j < 2 * TM; ++j) xv[j] = (j * 8 + lr) * (int)p.ldx + ((pc ^ (lr >> 1) ^ ((j & 1) << 2)) << 4);
  int8_t *ring = smem + wave * C::RING;
  auto issue = [&](int d, int k0) {
    int8_t *dst = ring + d * C::UNIT;
#pragma unroll
    for (int j = 0; j < 2 * TN; ++j)
      load_to_lds(wd, dst + j * 1024, wv[j], k0);
#pragma unroll
    for (int j = 0; j < 2 * TM; ++j)
      load_to_lds(xd, dst + C::W_BYTES + j * 1024, xv[j], k0);
  };
  // ---- LDS -> fragments of k-step s (64 bytes) of unit d: row l16, chunk 4 s + quad
  const int swz = (l16 >> 1) & 7;
  auto read = [&](int d, int s, v4i(&fw)[TN], v4i(&fx)[TM]) {
    const int8_t *base = ring + d * C::UNIT + l16 * C::UK + (((4 * s + quad) ^ swz) << 4);
#pragma unroll
    for (int a = 0; a < TN; ++a) fw[a] = *reinterpret_cast<const v4i *>(base + a * 16 * C::UK);
#pragma unroll
    for (int b = 0; b < TM; ++b) fx[b] = *reinterpret_cast<const v4i *>(base + C::W_BYTES + b * 16 * C::UK);
  };
  v4i acc[TN][TM];
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) acc[a][b] = v4i{0, 0, 0, 0};
  auto mma = [&](const v4i(&fw)[TN], const v4i(&fx)[TM]) {
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
      for (int b = 0; b < TM; ++b) acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[a], fx[b], acc[a][b], 0, 0, 0);
  };

  // ---- K: a contiguous range of whole units per wavefront, D units in flight
  const int units = p.k / C::UK;
  const int mine = units / W + (wave < units % W ? 1 : 0);
  const int k_first = (wave * (units / W) + (wave < units % W ? wave : units % W)) * C::UK;
  // epilogue parameters: the round trip runs under the K loop
  int r_off = 0, r_tab = 0;
  float r_mult = 0.0f, r_fb = 0.0f, r_rs = 1.0f;
  {
    const int ch = bn0 + (tid < rows_n ? tid : rows_n - 1);
    if (tid < C::BN) {
      if (p.offset) r_off = p.offset[ch];
      if (OUT_KIND == kOutFixed) {  // integer multiplier and shift travel in the two float slots
        r_mult = __int_as_float(p.m0[ch]);
        r_fb = __int_as_float(p.shift[ch]);
      } else if (OUT_KIND != CWAC_OUT_INT32) {
        r_mult = p.mult[ch];
        if (!INT_ONLY && p.fbias) r_fb = p.fbias[ch];
      }
    }
    if (!INT_ONLY && OUT_KIND != CWAC_OUT_INT32 && p.sx_row && tid < rows_m) r_rs = p.sx_row[bm0 + tid];
    if (OUT_KIND == kOutTable && tid < 64) r_tab = reinterpret_cast<const int32_t *>(p.code_table)[tid];
  }
  // (The parameter loads above are older than the panel loads and have landed when a unit has.)  Memory operations
  // return in order: with r units issued behind a unit, it is complete at r * LPU outstanding.
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < mine) issue(d, k_first + d * C::UK);
  int d = 0;
#pragma unroll 1
  for (int i = 0; i + D < mine; ++i) {
    wait_loads<(D - 1) * C::LPU>();
    v4i fw0[TN], fx0[TM], fw1[TN], fx1[TM];
    read(d, 0, fw0, fx0);
    read(d, 1, fw1, fx1);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14));  // lgkmcnt(0): the unit is in registers, its place is free
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    issue(d, k_first + (i + D) * C::UK);
    mma(fw0, fx0);
    mma(fw1, fx1);
    d = d + 1 == D ? 0 : d + 1;
  }
  auto last = [&](auto tag) {  // the last D units: nothing more to issue
    constexpr int behind = decltype(tag)::value;
    if (behind >= D || behind >= mine) return;
    wait_loads<(behind < D ? behind * C::LPU : 0)>();
    v4i fw0[TN], fx0[TM], fw1[TN], fx1[TM];
    read(d, 0, fw0, fx0);
    read(d, 1, fw1, fx1);
    mma(fw0, fx0);
    mma(fw1, fx1);
    d = d + 1 == D ? 0 : d + 1;
  };
  static_assert(D <= 4, "one call per slot");
  last(std::integral_constant<int, 3>{});
  last(std::integral_constant<int, 2>{});
  last(std::integral_constant<int, 1>{});
  last(std::integral_constant<int, 0>{});
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  // the last K % 128 bytes, 64 at a time, straight to registers: lanes whose 16 bytes lie beyond K read past the
  // extent (zeros)
  if (wave == W - 1) {
    for (int k0 = units * C::UK; k0 < p.k; k0 += 64) {
      const bool in_k = k0 + quad * 16 < p.k;
      v4i tw[TN], tx[TM];
#pragma unroll
      for (int a = 0; a < TN; ++a) {
        const int o = (a * 16 + l16) * (int)p.ldw + quad * 16 + k0;
        tw[a] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(wd, in_k ? o : 0x7ffffff0, 0, 0));
      }
#pragma unroll
      for (int b = 0; b < TM; ++b) {
        const int o = (b * 16 + l16) * (int)p.ldx + quad * 16 + k0;
        tx[b] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(xd, in_k ? o : 0x7ffffff0, 0, 0));
      }
      mma(tw, tx);
    }
  }

  // ---- the W partial tiles meet in LDS
  if (tid < C::BN) {
    s_off[tid] = r_off;
    s_mult[tid] = r_mult;
    s_fb[tid] = r_fb;
  }
  if (tid < C::BM) s_rs[tid] = r_rs;
  if (OUT_KIND == kOutTable && tid < 64) s_tab[tid] = r_tab;
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) reinterpret_cast<v4i *>(ring + (a * TM + b) * 1024)[lane] = acc[a][b];
  __syncthreads();
  // thread -> (token, four channels): consecutive threads take consecutive channels of a token
  constexpr int GROUPS = C::BM * C::BN / 4;
#pragma unroll
  for (int g0 = 0; g0 < GROUPS; g0 += C::NT) {
    const int g = g0 + tid;
    if (GROUPS % C::NT != 0 && g >= GROUPS) break;
    const int cg = g % (C::BN / 4), row = g / (C::BN / 4);
    const int tile = (cg >> 2) * TM + (row >> 4), at = (cg & 3) * 16 + (row & 15);
    if (row >= rows_m || 4 * cg >= rows_n) continue;
    const int8_t *part = smem + tile * 1024 + at * 16;
    v4i sum = *reinterpret_cast<const v4i *>(part);
#pragma unroll
    for (int s = 1; s < W; ++s) sum += *reinterpret_cast<const v4i *>(part + s * C::RING);
    const v4i o4 = *reinterpret_cast<const v4i *>(s_off + 4 * cg);
    const float4 m4 = *reinterpret_cast<const float4 *>(s_mult + 4 * cg);
    const float4 f4 = *reinterpret_cast<const float4 *>(s_fb + 4 * cg);
    const int av[4] = {sum[0], sum[1], sum[2], sum[3]}, off[4] = {o4[0], o4[1], o4[2], o4[3]};
    const float mu[4] = {m4.x, m4.y, m4.z, m4.w}, fb[4] = {f4.x, f4.y, f4.z, f4.w};
    if constexpr (OUT_KIND == kOutTable) {
      // n % 16 == 0 and a 16-byte aligned output are this output kind's contract: whole words
      const uint8_t *tab = reinterpret_cast<const uint8_t *>(s_tab);
      uint32_t word = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int code = requant_code((float)(av[r] + off[r]) * mu[r], p.lo, p.hi, p.zr);
        word |= (uint32_t)tab[(code + 128) & 255] << (8 * r);
      }
      *reinterpret_cast<uint32_t *>(static_cast<int8_t *>(p.out) + (bm0 + row) * p.ldo + bn0 + 4 * cg) = word;
    } else {
      Epilogue<OUT_KIND, INT_ONLY>::run(p, bm0 + row, bn0 + 4 * cg, av, mu, off, fb, s_rs[row]);
    }
  }
}

template <int TN, int TM, int W, int D, int OUT_KIND, bool INT_ONLY>
cwac_status launch_splitk_one(const FwdParams &p, dim3 grid, hipStream_t st) {
  constexpr int LDS = SplitCfg<TN, TM, W, D>::LDS_BYTES;
  static const hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void *>(&qlinear_splitk_kernel<TN, TM, W, D, OUT_KIND, INT_ONLY>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
  if (attr != hipSuccess) return CWAC_E_LAUNCH;
  qlinear_splitk_kernel<TN, TM, W, D, OUT_KIND, INT_ONLY><<<grid, 64 * W, LDS, st>>>(p);
  return launch_status();
}

template <int TN, int TM, int W, int D>
cwac_status launch_splitk_cfg(FwdParams p, int out_kind, bool int_only, hipStream_t st) {
  p.tiles_m = (int)ceil_div(p.m, 16 * TM);
  p.tiles_n = (int)ceil_div(p.n, 16 * TN);
  const int64_t blocks = (int64_t)p.tiles_m * p.tiles_n;
  if (blocks > 0x7fffffff) return CWAC_E_SHAPE;
  const dim3 grid((unsigned)blocks);
  if (out_kind == kOutFixed) return launch_splitk_one<TN, TM, W, D, kOutFixed, true>(p, grid, st);
  if (out_kind == kOutTable) return launch_splitk_one<TN, TM, W, D, kOutTable, true>(p, grid, st);
  if (out_kind == CWAC_OUT_INT8)
    return int_only ? launch_splitk_one<TN, TM, W, D, CWAC_OUT_INT8, true>(p, grid, st)
                    : launch_splitk_one<TN, TM, W, D, CWAC_OUT_INT8, false>(p, grid, st);
  if (out_kind == CWAC_OUT_FP32) return launch_splitk_one<TN, TM, W, D, CWAC_OUT_FP32, false>(p, grid, st);
  return launch_splitk_one<TN, TM, W, D, CWAC_OUT_INT32, false>(p, grid, st);
}

template <int I>
cwac_status launch_splitk_tile(const FwdParams &p, int out_kind, bool int_only, hipStream_t st) {
  return launch_splitk_cfg<kSplitk[I].tn, kSplitk[I].tm, kSplitk[I].w, kSplitk[I].d>(p, out_kind, int_only, st);
}

}  // namespace

cwac_status launch_splitk(const FwdParams &p, int out_kind, bool int_only, hipStream_t st) {
  const int tile = splitk_tile(p.m, p.n, p.k);
  switch (tile ? tile : 3) {  // forced where the rule leaves the layer to the tile kernels: 32 x 32 tiles
    case 1: return launch_splitk_tile<1>(p, out_kind, int_only, st);
    case 2: return launch_splitk_tile<2>(p, out_kind, int_only, st);
    case 3: return launch_splitk_tile<3>(p, out_kind, int_only, st);
    case 4: return launch_splitk_tile<4>(p, out_kind, int_only, st);
  }
  return CWAC_E_SHAPE;
}

}  // namespace cwac
