// Dispatch of the batched GEMMs (plan_gemm): which kernel, tile and number of K splits.
#include <algorithm>

#include "gemm_common.hpp"

namespace kraken {
namespace {

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Modelled time (us) of a GEMM of `tiles` workgroups, `slots` of them at a time, whose
// reduction is `slices` 128-byte slices long: launch + rounds x (prologue and epilogue +
// slices), a slice taking longer the fuller the round is (operand traffic, clock).  The
// constants are a fit to measured times over 65 to 17228 rows, widths 256 to 16384, 1 to 8 K
// splits.  On a sample of its own (random shapes, every plan timed; profiles/gemm_plans.md) the
// plan with the least modelled time is on average 2.0% (480 shapes, fp16) and 3.6% (160, fp32)
// slower than the fastest of all plans, half of them are the fastest; the worst are fp32 at 600 to
// 1600 rows, where 128 x 128 tiles of a last round that is partly empty take up to 1.7 times.
// A launch takes at least as long as its weights do at the rate the kernel streams them into LDS
// (128 rows, weights from HBM, 4 x 4992 -> 9984 and 4992 columns: 3.5 TB/s in 128 x 128 tiles, 5.0
// through the streaming kernel's tiles of 5 blocks of columns, 2.8 to 3.4 through 1 or 2; the same
// 5.0 where two terms stream the weights twice, a W_concat of 4 x 4992 -> 4992 in 80 us); a little
// of the modelled time then breaks ties.
struct TileCost {
  double launch, round, slice, slice_nb, load, gelu, stream;   // stream: TB/s
  double us(int64_t tiles, int64_t slots, int64_t slices, int nb, bool with_gelu,
            double weight_mb) const {
    auto per_round = [&](double full) {
      return round + (with_gelu ? gelu : 0.0) +
             (double)slices * (slice + slice_nb * nb) * (1.0 + load * full);
    };
    double t = launch + (double)(tiles / slots) * per_round(1.0);
    if (tiles % slots) t += per_round((double)(tiles % slots) / (double)slots);
    const double rate = nb > 0 ? std::min(2.2 + 0.6 * nb, stream) : stream;
    const double floor = launch + weight_mb / rate;
    return t > floor ? t : floor + 0.03 * t;
  }
};
constexpr TileCost COST16_256{0.0, 9.5, 1.0, 0, 0.63, 6.0, 4.0},
    COST16_128{2.4, 0.9, 0.61, 0, 0.78, 3.1, 3.5},
    COST16_64{2.4, 0.6, 0.42, 0, 0.6, 1.6, 3.5},   // 128 x 64 tiles
    COST16_MID{2.8, 1.3, 0.09, 0.093, 0.56, 1.9, 5.0};
constexpr TileCost COST32_256{3.2, 7.4, 7.04, 0, 0.01, 2.0, 4.0},
    COST32_128{0.0, 4.7, 1.71, 0, 1.05, 2.0, 3.5},
    COST32_MID{3.1, 1.3, 0.083, 0.453, 0.08, 1.0, 5.0};
// The streaming kernel is considered up to MID_ROWS rows of activations, and past them where
// 128 x 128 tiles would leave CUs without a workgroup: up to MID_ROWS_NARROW rows (with a
// reduction of at most MID_SHORT slices, or at most half of the CUs taken: up to MID_ROWS_LAST).  It
// reads its A tile from LDS once per 32 MFMAs of a wave, and beyond that was never clearly the
// fastest measured 16-bit plan (512 rows, 2048 -> 8192 columns: 27 us, tiles 32; 1500 rows,
// 768 -> 1536: 10.3 and 11.8; 1800 rows, 3072 -> 768: 21.3 and 30.5; 3000 rows, 768 -> 1536: 16.1
// and 13.9).  Past MID_ROWS_LAST rows 128 x 64 tiles, two workgroups per CU, take its place there (4713
// rows, 1536 -> 384: 16.4 us, streaming 17.1, 128 x 128 19.6; 384 -> 384: 7.2, 7.7 and 9.8; 4059
// rows, 768 -> 768: 11.8, 15.0 and 12.8; 2563 rows, 3072 -> 768: 26.0, 26.7 and 29.8).  fp32
// is bound by its MFMAs and takes the streaming kernel at any number of rows (4059 rows,
// 768 -> 768: 47.1 us, 128 x 128 56.1).
constexpr int MID_ROWS = 512, MID_ROWS_NARROW = 1536, MID_ROWS_LAST = 2560, MID_SHORT = 8;

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
bool skinny_wins(bool f32, int M, int N, int64_t Kall, int terms, int batch,
                 int64_t part_elems) {
  if (M > 64 || batch > 65535) return false;        // (the batch is a grid dimension)
  if (M <= 16 || f32) return true;
  // 17 to 32 rows: few columns and a reduction that is short (counting the loads of A, which
  // two terms double) or cannot be split
  return M <= 32 && (int64_t)N * batch <= 4096 && (Kall * terms <= 2048 || part_elems == 0);
}

GemmPlan skinny_plan(bool f32, int M, int N, int64_t Kall, int terms, int batch,
                     int64_t part_elems, bool own_sum) {
  const int64_t blocks = ceil_div(N, 16) * batch;   // workgroups of one column block
  GemmPlan p{GemmKind::SKINNY, 1, 1, 4};
  if (f32 && M <= 16) p.waves = 16;
  else if (f32 || Kall * terms >= 2048 || blocks <= 512) p.waves = 8;
  // two column blocks (each A fragment feeds two MFMAs) once they still fill the chip
  if (!f32 && M > 1 && blocks >= 1024 && Kall * terms >= 2048) p.nb = 2;
  // Few column blocks and a long reduction: K splits, as long as every wave keeps a whole batch
  // of 8 loads of A: 8 steps, or 4 steps of two terms.  A batch less per wave saves about 3 us; a
  // launch for the sum costs 4.  (Two terms, 1 row, with the sum's launch, us in 1 / 2 / 4 / 8
  // splits: 4 x 1024 -> 1024, 16 steps a wave whole, 11.3 / 9.3 / 7.3 / 7.2; 4 x 768 -> 768, 12
  // steps, 7.4 / 6.8 / 5.9 / 6.4; 4 x 256 -> 256, 4 steps, 3.4 / 4.6 / 4.4.)
  const int64_t batches = Kall * terms / (f32 ? 16 : 32) / (8 * p.waves);
  const int64_t sp = std::min<int64_t>(
      {8, 512 / blocks, batches, part_elems / ((int64_t)M * N * batch)});
  if (sp > 1 && (!own_sum || 3 * (batches - batches / sp) > 6)) p.splits = (int)sp;
  return p;
}

}  // namespace

GemmPlan plan_gemm(DType dt, int epi, int M, int N, int K, int kgroups, int terms, int batch,
                   int64_t part_elems, bool own_sum) {
  const bool f32 = dt == DType::F32;
  const int64_t Kall = (int64_t)K * kgroups;
  if (epi != EPI_BIAS_M && skinny_wins(f32, M, N, Kall, terms, batch, part_elems))
    return skinny_plan(f32, M, N, Kall, terms, batch, part_elems, own_sum);
  // The other kernels walk the groups once per term, and load every weight each time: slices and
  // streamed bytes count per term.
  const int64_t slices = (int64_t)K / (f32 ? 32 : 64) * kgroups * terms;
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
  const double wmb = (double)(epi == EPI_BIAS_M ? M : N) * (double)(Kall * terms) * batch *
                     (f32 ? 4e-6 : 2e-6);
  for (int sp = 1; sp <= 8; ++sp) {
    // Splits keep at least 8 slices each (2 of the four times longer fp32 ones; a shorter
    // reduction gains under 0.3 us per split); their planes must fit.  A plane costs about
    // 0.1 us per MB to write and 0.2 us per MB to read in the kernel that sums them, which
    // without a split would read one as well, unless it is launched for the sum alone (4 us,
    // and its result and residual pass through it too).  A sum with a launch of its own (W_concat,
    // the last FFN-down) stays whole from 512 tiles of 128 x 128 on: W_concat from 3969 rows at
    // width 2048, 6529 at 1280, 8065 at 1024.  That is not for speed (17228 rows of four sub-layers
    // of width 1280: 457 us whole, 383 in two planes) but keeps the outputs of the widest long
    // prompts in one order: rows 0 .. 4095 of 8192 are those of a 4096-token prompt to the last
    // bits at width 2048.  It is no rule for every shape: below the limit, and for the other
    // projections at any number of rows (GPT-like, width 2048, FFN-down: two planes at 8193 to 12288
    // rows), the order of a sum, and so its last bits, depend on the number of rows.
    if (sp > 1 && (sp * plane > part_elems || slices < (f32 ? 2 : 8) * sp ||
                   (own_sum && t128 >= 512)))
      break;
    const double mb = (double)plane * 4e-6;
    double extra = 0.0;
    if (sp > 1) extra = 0.1 * mb * sp + 0.2 * mb * (sp - 1) + (own_sum ? 4.0 + 0.4 * mb : 0.0);
    const int64_t sl = ceil_div(slices, sp);
    const bool gelu = epi == EPI_BIAS_N_GELU;
    consider(GemmKind::TILE256, 0, sp,
             extra + (f32 ? COST32_256 : COST16_256).us(t256 * sp, 256, sl, 0, gelu, wmb));
    // (two 128 x 128 workgroups per CU)
    consider(GemmKind::TILE128, 0, sp,
             extra + (f32 ? COST32_128 : COST16_128).us(t128 * sp, 512, sl, 0, gelu, wmb));
    const bool narrow = t128 * sp < 256;
    if (!f32 && narrow && rows > MID_ROWS_LAST)
      consider(GemmKind::TILE128, 2, sp,
               extra + COST16_64.us(ceil_div(M, 128) * ceil_div(N, 64) * batch * sp, 512, sl, 0,
                                    gelu, wmb));
    const bool mid = rows <= MID_ROWS ||
                     (narrow && (f32 || rows <= MID_ROWS_NARROW ||
                                 (rows <= MID_ROWS_LAST &&
                                  (t128 * sp <= 128 || slices <= MID_SHORT))));
    if (!mid) continue;
    for (int nb = 1; nb <= MID_MAX_NB; ++nb)
      consider(GemmKind::MID, nb, sp,
               extra + (f32 ? COST32_MID : COST16_MID)
                           .us(ceil_div(M, MID_BM) * ceil_div(N, 32 * nb) * batch * sp, 256, sl, nb,
                               gelu, wmb));
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
  if (g.gA2 != 0 && (plan.kind != GemmKind::SKINNY ||
                     (g.epi != EPI_BIAS_N_RES && g.epi != EPI_PART)))
    return hipErrorInvalidValue;
  if (plan.kind == GemmKind::SKINNY && (g.M > 64 || g.epi == EPI_BIAS_M))
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
    default: {
      const int cols = plan.kind == GemmKind::TILE256 ? 256 : plan.nb == 2 ? 64 : 128;
      return g.dt == DType::BF16 ? launch_gemm_tile<bf16>(g, cols, s)
             : g.dt == DType::F16 ? launch_gemm_tile<f16>(g, cols, s)
                                  : launch_gemm_tile<float>(g, cols, s);
    }
  }
}

hipError_t launch_gemm(const GemmDesc& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0 || g.kgroups <= 0) return hipSuccess;   // no plan
  return launch_gemm_planned(
      g, plan_gemm(g.dt, g.epi, g.M, g.N, g.K, g.kgroups, 1, g.batch, 0, false), s);
}

}  // namespace kraken
