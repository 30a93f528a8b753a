// Dispatch of the batched GEMMs (plan_gemm) and the kernel for a few rows.
#include "gemm_common.hpp"

namespace kraken {
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
constexpr double GELU_256 = 7.0, GELU_128 = 1.2;
// The streaming kernel is considered up to MID_ROWS rows of activations, and up to
// MID_ROWS_NARROW where 128 x 128 tiles would leave CUs without a workgroup: it reads its A tile
// from LDS once per 32 MFMAs of a wave, and beyond that was never clearly the fastest measured
// 16-bit plan (512 rows, 2048 -> 8192 columns: 27 us, tiles 32; 1500 rows, 768 -> 1536: 10.3 and
// 11.8; 3000 rows: 16.1 and 13.9; four sub-layers of 2048 rows, 768 -> 768, 384 tiles: 25 and 18).
constexpr int MID_ROWS = 512, MID_ROWS_NARROW = 1536;

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

// A few rows (a decode step): whether the kernel for them is the faster one, and its form.
// Measured with weights from HBM, fp16 (us; 16 columns x 4 waves per workgroup before):
//   1 row     2048 -> 4096  7.6 -> 6.8 with 8 waves, 8192 -> 2048 19.9 -> 14.8, eight sub-layers
//             of 8192 -> 2048 56.0 -> 50.1; 1280 -> 51200 27.9 (8 waves: 34.3)
//   8 rows    eight of 2048 -> 8192 59.4, with two column blocks per workgroup 57.8; one
//             2048 -> 2048 6.5, two blocks 8.7
//   24 rows   2048 -> 2048 8.4, the streaming kernel 10.7; 2048 -> 6144 13.1 and 12.5; eight of
//             8192 -> 2048 81 and 65; past 32 rows the streaming kernel is the faster one
//             everywhere (64 rows, eight of 2048 -> 8192: 119 and 80)
//   fp32      four of 4096 -> 1024 at 1 row 24.1 with 8 waves, 19.0 with 16; at 64 rows 48.5, the
//             streaming kernel 70
bool skinny_wins(bool f32, int M, int N, int64_t Kall, int batch, int64_t part_elems) {
  if (M > 64) return false;
  if (M <= 16 || f32) return true;
  // 17 to 32 rows: few columns and a reduction that is short or cannot be split
  return M <= 32 && (int64_t)N * batch <= 4096 && (Kall <= 2048 || part_elems == 0);
}

GemmPlan skinny_plan(bool f32, int M, int N, int64_t Kall, int batch) {
  const int64_t blocks = ceil_div(N, 16) * batch;   // workgroups of one column block
  GemmPlan p{GemmKind::SKINNY, 1, 1, 4};
  if (f32 && M <= 16) p.waves = 16;
  else if (f32 || Kall >= 2048 || blocks <= 512) p.waves = 8;
  // two column blocks (each A fragment feeds two MFMAs) once they still fill the chip
  if (!f32 && M > 1 && blocks >= 1024 && Kall >= 2048) p.nb = 2;
  return p;
}

}  // namespace

GemmPlan plan_gemm(DType dt, int epi, int M, int N, int K, int kgroups, int batch,
                   int64_t part_elems, bool own_sum) {
  const bool f32 = dt == DType::F32;
  const int64_t Kall = (int64_t)K * kgroups;
  if (epi != EPI_BIAS_M && epi != EPI_PART && skinny_wins(f32, M, N, Kall, batch, part_elems))
    return skinny_plan(f32, M, N, Kall, batch);
  const int64_t slices = (int64_t)K / (f32 ? 32 : 64) * kgroups;
  const int64_t t256 = ceil_div(M, 256) * ceil_div(N, 256) * batch;
  const int64_t t128 = ceil_div(M, 128) * ceil_div(N, 128) * batch;
  GemmPlan best{GemmKind::TILE256, 0, 1, 0};
  double best_t = 1e30;
  auto consider = [&](GemmKind kind, int nb, int splits, double t) {
    if (t < best_t) {
      best_t = t;
      best = {kind, nb, splits, 0};
    }
  };
  const int64_t plane = (int64_t)M * N * batch;
  const int rows = epi == EPI_BIAS_M ? N : M;
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
    if (rows > (t128 * sp < 256 ? MID_ROWS_NARROW : MID_ROWS)) continue;
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
  if (g.gA2 != 0 && (plan.kind != GemmKind::SKINNY || g.epi != EPI_BIAS_N_RES))
    return hipErrorInvalidValue;
  if (plan.kind == GemmKind::SKINNY && (g.M > 64 || g.epi == EPI_BIAS_M || g.epi == EPI_PART))
    return hipErrorInvalidValue;
  if (g.epi == EPI_QKV &&
      (!g.qkv || (plan.kind != GemmKind::SKINNY && plan.kind != GemmKind::MID) ||
       (g.qkv->cache && g.M > 256)))
    return hipErrorInvalidValue;
  switch (plan.kind) {
    case GemmKind::SKINNY:
      return g.dt == DType::BF16 ? launch_gemm_skinny<bf16>(g, plan.nb, plan.waves, s)
             : g.dt == DType::F16 ? launch_gemm_skinny<f16>(g, plan.nb, plan.waves, s)
                                  : launch_gemm_skinny<float>(g, plan.nb, plan.waves, s);
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
