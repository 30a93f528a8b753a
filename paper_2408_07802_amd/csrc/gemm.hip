// Dispatch of the batched GEMMs (plan_gemm) and the kernel for a few rows.
#include "gemm_common.hpp"

namespace kraken {
namespace {

// ----------------------------------------------------------------------------- few rows
//
// GEMM for a few rows of A (M <= 64: the tokens of a decode step).  Then every weight
// element is used at most 64 times and the kernel is bound by streaming B (the weights)
// from HBM once, so the tiling is chosen for parallelism: a workgroup owns TW blocks of
// 16 output columns of one batch entry and all M rows, and its 4 waves split the
// (kgroups x K) reduction into 4 contiguous ranges, merged through LDS at the end.  Each
// step of 32 k is one v_mfma_f32_16x16x32 per (16-row block of A, column block): lane l
// supplies B column l % 16 and A row l % 16, k = 8 (l / 16) .. + 7 (one 16-byte load
// each), and gets D rows 4 (l / 16) .. + 3 of column l % 16.  A rows past M load row
// M - 1 and are masked to zero (whole 16-byte loads without branches: per-lane
// conditional loads compile to four 4-byte loads each and halved the throughput at 8
// rows); B columns past N load a clamped row and are not stored.
template <typename S>
__device__ __forceinline__ f32x4 mfma16(uint4 a, uint4 b, f32x4 c) {
  if constexpr (__is_same(S, bf16)) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  } else {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                  __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
}

constexpr int SK_UNROLL = 8;   // steps of 32 k whose loads are issued together

// 16-byte weight load (plain: non-temporal loads measured the same, within 3%, on weight
// streams that do not fit the last-level cache).
__device__ __forceinline__ uint4 load_w16(const void* ptr) {
  return *reinterpret_cast<const uint4*>(ptr);
}

template <typename S, int MB, int TW, int EPI>
__global__ __launch_bounds__(256) void gemm_skinny_kernel(GemmParams p) {
  __shared__ float red[4][MB * TW][256];
  using OutT = std::conditional_t<epi_f32<EPI>, float, S>;
  const int z = blockIdx.y;
  const int n0 = blockIdx.x * 16 * TW;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, kq = lane >> 4;
  const S* Bz[TW];
#pragma unroll
  for (int w = 0; w < TW; ++w)
    Bz[w] = static_cast<const S*>(p.B) + z * p.sB +
            (int64_t)min(n0 + w * 16 + col, p.N - 1) * p.ldb + kq * 8;
  // A rows past M load row M - 1 (whole 16-byte loads, no branches) and are masked to 0
  const S* Az[MB];
  uint32_t amask[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int m = mb * 16 + col;
    amask[mb] = m < p.M ? 0xffffffffu : 0u;
    Az[mb] = static_cast<const S*>(p.A) + z * p.sA + (int64_t)min(m, p.M - 1) * p.lda + kq * 8;
  }
  auto load_a = [&](int mb, int64_t off) {
    uint4 v = *reinterpret_cast<const uint4*>(Az[mb] + off);
    v.x &= amask[mb]; v.y &= amask[mb]; v.z &= amask[mb]; v.w &= amask[mb];
    return v;
  };
  const int steps_per_group = p.K / 32;
  const int steps = steps_per_group * p.kgroups;
  const int t0 = (int)((int64_t)steps * wave / 4), t1 = (int)((int64_t)steps * (wave + 1) / 4);
  f32x4 acc[MB * TW];
#pragma unroll
  for (int q = 0; q < MB * TW; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
  // step t covers k = 32 (t mod steps_per_group) .. + 31 of group g = t / steps_per_group;
  // (g, kk) is tracked incrementally from this wave's first step
  int g = t0 / steps_per_group, kk = (t0 - g * steps_per_group) * 32;
  int gb = g % p.gBmod;
  auto advance = [&]() {
    kk += 32;
    if (kk == p.K) {
      kk = 0;
      ++g;
      if (++gb == p.gBmod) gb = 0;
    }
  };
  int t = t0;
  for (; t + SK_UNROLL <= t1; t += SK_UNROLL) {
    uint4 bv[SK_UNROLL][TW], av[SK_UNROLL][MB];
    int64_t ao[SK_UNROLL], bo[SK_UNROLL];
#pragma unroll
    for (int u = 0; u < SK_UNROLL; ++u) {
      ao[u] = g * p.gA + kk;
      bo[u] = gb * p.gB + kk;
      advance();
    }
#pragma unroll
    for (int u = 0; u < SK_UNROLL; ++u)
#pragma unroll
      for (int w = 0; w < TW; ++w) bv[u][w] = load_w16(Bz[w] + bo[u]);
#pragma unroll
    for (int u = 0; u < SK_UNROLL; ++u)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
        av[u][mb] = load_a(mb, ao[u]);
#pragma unroll
    for (int u = 0; u < SK_UNROLL; ++u)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int w = 0; w < TW; ++w)
          acc[mb * TW + w] = mfma16<S>(av[u][mb], bv[u][w], acc[mb * TW + w]);
  }
  for (; t < t1; ++t) {
    uint4 bv[TW];
#pragma unroll
    for (int w = 0; w < TW; ++w) bv[w] = load_w16(Bz[w] + gb * p.gB + kk);
    const int64_t ao = g * p.gA + kk;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const uint4 av = load_a(mb, ao);
#pragma unroll
      for (int w = 0; w < TW; ++w) acc[mb * TW + w] = mfma16<S>(av, bv[w], acc[mb * TW + w]);
    }
    advance();
  }
  // D row 4 kq + j, column col of each 16-row block -> red[wave][mb][row * 16 + col]
#pragma unroll
  for (int q = 0; q < MB * TW; ++q)
#pragma unroll
    for (int j = 0; j < 4; ++j) red[wave][q][(kq * 4 + j) * 16 + col] = acc[q][j];
  __syncthreads();
  const int tid = threadIdx.x;
  const float* biasz = p.bias ? p.bias + z * p.sBias : nullptr;
  float amax = 0.f;
#pragma unroll
  for (int w = 0; w < TW; ++w) {
    const int n = n0 + w * 16 + (tid & 15);
    if (n >= p.N) continue;
    const float bn = biasz ? biasz[n] : 0.f;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int m = mb * 16 + (tid >> 4);
      if (m >= p.M) break;
      const int q = mb * TW + w;
      float v = (red[0][q][tid] + red[1][q][tid]) + (red[2][q][tid] + red[3][q][tid]) + bn;
      if constexpr (EPI == EPI_BIAS_N_GELU) v = gelu_erf(v);
      if constexpr (epi_res<EPI>) {
        if (p.R) v += p.R[z * p.sR + (int64_t)m * p.ldc + n];
      }
      track4<OutT>(amax, make_float4(v, 0.f, 0.f, 0.f));
      OutT* dst = static_cast<OutT*>(p.C) + z * p.sC + (int64_t)m * p.ldc + n;
      store_val<OutT>(dst, v);
      if constexpr (EPI == EPI_BIAS_N_HILO) store_val<OutT>(dst + p.sPlane, v - (float)(S)v);
    }
  }
  flag_overflow<OutT>(amax, p.ovf);
}

template <typename S, int MB, int TW>
hipError_t launch_skinny(const GemmDesc& g, hipStream_t s) {
  GemmParams p = gemm_params(g);
  p.tiles_n = (g.N + 16 * TW - 1) / (16 * TW);
  dim3 grid((unsigned)p.tiles_n, (unsigned)g.batch), block(256);
  switch (g.epi) {
    case EPI_BIAS_N:
      hipLaunchKernelGGL((gemm_skinny_kernel<S, MB, TW, EPI_BIAS_N>), grid, block, 0, s, p);
      break;
    case EPI_BIAS_N_GELU:
      hipLaunchKernelGGL((gemm_skinny_kernel<S, MB, TW, EPI_BIAS_N_GELU>), grid, block, 0, s, p);
      break;
    case EPI_BIAS_N_RES:
      hipLaunchKernelGGL((gemm_skinny_kernel<S, MB, TW, EPI_BIAS_N_RES>), grid, block, 0, s, p);
      break;
    case EPI_BIAS_N_HILO:
      hipLaunchKernelGGL((gemm_skinny_kernel<S, MB, TW, EPI_BIAS_N_HILO>), grid, block, 0, s, p);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Two 16-column blocks per wave (each A fragment feeds two MFMAs, halving the A loads per
// weight byte) for several rows and reductions up to 4096; one block (twice the
// workgroups) otherwise.  Measured on the N=8, d=2048 decode projections with weights
// streamed from HBM: one row, one block 5-18% faster for every projection (FFN down 54
// against 66 us); eight rows, two blocks 4-5% faster at K = 2048, one block 5% faster at
// K = 8192.
template <typename S, int MB>
hipError_t launch_skinny_tw(const GemmDesc& g, hipStream_t s) {
  if (g.M > 1 && (int64_t)g.K * g.kgroups <= 4096) return launch_skinny<S, MB, 2>(g, s);
  return launch_skinny<S, MB, 1>(g, s);
}

template <typename S>
hipError_t launch_skinny_rows(const GemmDesc& g, hipStream_t s) {
  if (g.M <= 16) return launch_skinny_tw<S, 1>(g, s);
  if (g.M <= 32) return launch_skinny_tw<S, 2>(g, s);
  return launch_skinny_tw<S, 4>(g, s);
}

}  // namespace

namespace {

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Modelled time (us) of a GEMM of `tiles` workgroups whose reduction is `slices` 128-byte
// slices long: launch + rounds of workgroups x (prologue and epilogue + slices).  The
// constants are a fit to measured times (5 to 500 us kernels; fp16 / bf16: 2638 runs over 65
// to 17228 rows, widths 256 to 16384, 1 to 8 K splits; fp32: 772 runs): the plan with the
// least modelled time is on average 3% (fp32 2%) slower than the fastest of all plans.
struct TileCost {
  double launch, round, slice, slice_half, slice_nb;
};
constexpr TileCost COST16_256{0.0, 7.6, 1.28, 0, 0}, COST16_128{1.7, 1.3, 1.13, 0.72, 0},
    COST16_MID{2.4, 1.25, 0.17, 0, 0.106};
constexpr TileCost COST32_256{3.7, 6.9, 7.07, 0, 0}, COST32_128{4.1, 0.1, 3.74, 1.98, 0},
    COST32_MID{2.8, 1.4, 0.105, 0, 0.466};
// The GELU epilogue per round of 256 x 256 and 128 x 128 tiles (768 -> 3072 columns, 4 x 2048
// rows: 384 tiles of 256 x 256 65 us, 1536 of 128 x 128 55 us).
constexpr double GELU_256 = 5.0, GELU_128 = 1.2;
// The streaming kernel is considered up to this many rows of activations, and beyond them only
// where 128 x 128 tiles would leave CUs without a workgroup: it reads its A tile from LDS once
// per 32 MFMAs of a wave, and with more rows and enough tiles was never the fastest measured
// 16-bit plan (512 rows: 27 us against 32 us for 2048 -> 8192 columns; 2048 rows, 768 -> 768
// columns of four sub-layers, 384 tiles: 25 us against 18 us).
constexpr int MID_MAX_ROWS = 512;

double cost_256(const TileCost& c, int64_t tiles, int64_t slices, double epi) {
  return c.launch + (double)ceil_div(tiles, 256) * (c.round + epi + (double)slices * c.slice);
}
// two workgroups per CU; a last round that leaves every CU at most one of them runs its
// slices faster (slice_half)
double cost_128(const TileCost& c, int64_t tiles, int64_t slices, double epi) {
  const int64_t full = tiles / 512, rem = tiles % 512;
  double t = c.launch + (double)full * (c.round + epi + (double)slices * c.slice);
  if (rem > 0) t += c.round + epi + (double)slices * (rem > 256 ? c.slice : c.slice_half);
  return t;
}
double cost_mid(const TileCost& c, int64_t tiles, int64_t slices, int nb) {
  return c.launch + (double)ceil_div(tiles, 256) *
                        (c.round + (double)slices * (c.slice + c.slice_nb * nb));
}

}  // namespace

GemmPlan plan_gemm(DType dt, int epi, int M, int N, int K, int kgroups, int batch,
                   int64_t part_elems, bool own_sum) {
  // a few rows of 16-bit operands (a decode step): weight streaming
  if (M <= 64 && epi != EPI_BIAS_M && dt != DType::F32) return {GemmKind::SKINNY, 0, 1};
  const bool f32 = dt == DType::F32;
  const int64_t slices = (int64_t)K / (f32 ? 32 : 64) * kgroups;
  const int64_t t256 = ceil_div(M, 256) * ceil_div(N, 256) * batch;
  const int64_t t128 = ceil_div(M, 128) * ceil_div(N, 128) * batch;
  GemmPlan best{GemmKind::TILE256, 0, 1};
  double best_t = 1e30;
  auto consider = [&](GemmKind kind, int nb, int splits, double t) {
    if (t < best_t) {
      best_t = t;
      best = {kind, nb, splits};
    }
  };
  const int64_t plane = (int64_t)M * N * batch;
  for (int sp = 1; sp <= 8; ++sp) {
    // Splits keep at least 8 slices each (2 of the four times longer fp32 ones; a shorter
    // reduction gains under 0.3 us per split); their planes must fit.  A plane costs about
    // 0.1 us per MB to write and 0.2 us per MB to read in the kernel that sums them, which
    // without a split would read one as well, unless it is launched for the sum alone (4 us,
    // and its result and residual pass through it too).
    if (sp > 1 && (sp * plane > part_elems || slices < (f32 ? 2 : 8) * sp)) break;
    const double mb = (double)plane * 4e-6;
    double extra = 0.0;
    if (sp > 1) extra = 0.1 * mb * sp + 0.2 * mb * (sp - 1) + (own_sum ? 4.0 + 0.4 * mb : 0.0);
    const int64_t sl = ceil_div(slices, sp);
    consider(GemmKind::TILE256, 0, sp,
             extra + cost_256(f32 ? COST32_256 : COST16_256, t256 * sp, sl,
                              epi == EPI_BIAS_N_GELU ? GELU_256 : 0.0));
    consider(GemmKind::TILE128, 0, sp,
             extra + cost_128(f32 ? COST32_128 : COST16_128, t128 * sp, sl,
                              epi == EPI_BIAS_N_GELU ? GELU_128 : 0.0));
    if ((epi == EPI_BIAS_M ? N : M) > MID_MAX_ROWS && t128 * sp >= 256) continue;
    for (int nb = 1; nb <= MID_MAX_NB; ++nb)
      consider(GemmKind::MID, nb, sp,
               extra + cost_mid(f32 ? COST32_MID : COST16_MID,
                                ceil_div(M, MID_BM) * ceil_div(N, 32 * nb) * batch * sp, sl, nb));
  }
  return best;
}

hipError_t launch_gemm_planned(const GemmDesc& g, const GemmPlan& plan, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0 || g.kgroups <= 0) return hipSuccess;
  const int bk = g.dt == DType::F32 ? 32 : 64;
  if (g.K <= 0 || g.K % bk != 0 || g.gBmod <= 0) return hipErrorInvalidValue;
  if (g.splits > 1 && (g.epi != EPI_PART || g.splits > (int64_t)g.K / bk * g.kgroups))
    return hipErrorInvalidValue;
  // the kernels address operand rows of one batch entry / K group with 32-bit byte offsets
  const int64_t es = (int64_t)dtype_size(g.dt);
  if ((int64_t)g.M * g.lda * es >= (1ll << 31) || (int64_t)g.N * g.ldb * es >= (1ll << 31))
    return hipErrorInvalidValue;
  switch (plan.kind) {
    case GemmKind::SKINNY:
      return g.dt == DType::BF16 ? launch_skinny_rows<bf16>(g, s)
             : g.dt == DType::F16 ? launch_skinny_rows<f16>(g, s) : hipErrorInvalidValue;
    case GemmKind::MID:
      return g.dt == DType::BF16 ? launch_gemm_mid<bf16>(g, plan.nb, s)
             : g.dt == DType::F16 ? launch_gemm_mid<f16>(g, plan.nb, s)
                                  : launch_gemm_mid<float>(g, plan.nb, s);
    default:
      return g.dt == DType::BF16 ? launch_gemm_tile<bf16>(g, plan.kind == GemmKind::TILE256, s)
             : g.dt == DType::F16
                 ? launch_gemm_tile<f16>(g, plan.kind == GemmKind::TILE256, s)
                 : launch_gemm_tile<float>(g, plan.kind == GemmKind::TILE256, s);
  }
}

hipError_t launch_gemm(const GemmDesc& g, hipStream_t s) {
  return launch_gemm_planned(
      g, plan_gemm(g.dt, g.epi, g.M, g.N, g.K, g.kgroups, g.batch, 0, false), s);
}

}  // namespace kraken
