// Batched MFMA GEMM for at most 64 rows of A: the tokens of a decode step, or a very short
// prompt.  C[z] = epi(A[z] B[z]^T).
//
// Every weight element is used at most 64 times and the kernel is bound by streaming B (the
// weights) from HBM once, so the tiling is chosen for loads in flight: a workgroup owns TW
// blocks of 16 output columns of one batch entry and all M rows, and its NW waves split the
// (kgroups x K) reduction into NW contiguous ranges, merged through LDS at the end.  Each step
// of 64 bytes of k is one v_mfma_f32_16x16x32 (16-bit operands; four 16x16x4 for fp32) per
// (16-row block of A, column block): lane l supplies B column l % 16 and A row l % 16, 16 bytes
// of k from 16 (l / 16) on, and gets D rows 4 (l / 16) .. + 3 of column l % 16.  A rows past M
// load row M - 1 and are masked to zero (whole 16-byte loads without branches: per-lane
// conditional loads compile to four 4-byte loads each and halved the throughput at 8 rows); B
// columns past N load a clamped row and are not stored.
//
// NW: a launch with few column blocks needs its loads in flight from more waves per block
// (skinny_plan has the measured rule).
//
// Compiled once per operand type (KRAKEN_T).
#include "gemm_common.hpp"

namespace kraken {
namespace {

// acc += one 64-byte step of k: a and b are the lane's 16 bytes of its row and column.
template <typename S>
__device__ __forceinline__ f32x4 mfma16(uint4 a, uint4 b, f32x4 c) {
  if constexpr (__is_same(S, bf16)) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  } else if constexpr (__is_same(S, f16)) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                  __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  } else {
    // MFMA q takes element q of every lane's chunk: k = 4 (l / 16) + q, for A and B alike
    const f32x4 a4 = __builtin_bit_cast(f32x4, a), b4 = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int q = 0; q < 4; ++q) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[q], b4[q], c, 0, 0, 0);
    return c;
  }
}

constexpr int SK_UNROLL = 8;   // steps whose loads are issued together

// DUAL: A holds two terms (the second p.gA2 elements behind the first), both multiplied with
// the same B fragment: W_concat's hi + lo operand reads its weights once instead of twice.
template <typename S, int MB, int TW, int NW, int EPI, bool DUAL>
__global__ __launch_bounds__(64 * NW) void gemm_skinny_kernel(GemmParams p, QkvArg<EPI> kv) {
  constexpr int EPC = 16 / sizeof(S), KS = 4 * EPC;   // elements per chunk and per step
  constexpr int NA = DUAL ? 2 : 1;
  __shared__ float red[NW][MB * TW][256];
  using OutT = std::conditional_t<epi_f32<EPI>, float, S>;
  const int z = blockIdx.y;
  const int n0 = blockIdx.x * 16 * TW;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, kq = lane >> 4;
  const S* Bz[TW];
#pragma unroll
  for (int w = 0; w < TW; ++w)
    Bz[w] = static_cast<const S*>(p.B) + z * p.sB +
            (int64_t)min(n0 + w * 16 + col, p.N - 1) * p.ldb + kq * EPC;
  // A rows past M load row M - 1 (whole 16-byte loads, no branches) and are masked to 0
  const S* Az[MB];
  uint32_t amask[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int m = mb * 16 + col;
    amask[mb] = m < p.M ? 0xffffffffu : 0u;
    Az[mb] = static_cast<const S*>(p.A) + z * p.sA + (int64_t)min(m, p.M - 1) * p.lda + kq * EPC;
  }
  auto load_a = [&](int mb, int64_t off) {
    uint4 v = *reinterpret_cast<const uint4*>(Az[mb] + off);
    v.x &= amask[mb]; v.y &= amask[mb]; v.z &= amask[mb]; v.w &= amask[mb];
    return v;
  };
  auto load_b = [&](int w, int64_t off) { return *reinterpret_cast<const uint4*>(Bz[w] + off); };
  // this wave's steps: the workgroup's K split (EPI_PART: p.splits of them), then its waves
  const int steps_per_group = p.K / KS;
  const int64_t steps = (int64_t)steps_per_group * p.kgroups;
  const int sp = EPI == EPI_PART ? blockIdx.z : 0, parts = NW * (EPI == EPI_PART ? p.splits : 1);
  const int t0 = (int)(steps * (sp * NW + wave) / parts);
  const int t1 = (int)(steps * (sp * NW + wave + 1) / parts);
  f32x4 acc[MB * TW];
#pragma unroll
  for (int q = 0; q < MB * TW; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
  // step t covers k = KS (t mod steps_per_group) .. of group g = t / steps_per_group; (g, kk)
  // is tracked incrementally from this wave's first step
  int g = t0 / steps_per_group, kk = (t0 - g * steps_per_group) * KS;
  int gb = g % p.gBmod;
  auto advance = [&]() {
    kk += KS;
    if (kk == p.K) {
      kk = 0;
      ++g;
      if (++gb == p.gBmod) gb = 0;
    }
  };
  // n steps, all their loads issued together
  auto batch = [&](auto Nc) {
    constexpr int U = decltype(Nc)::value;
    uint4 bv[U][TW], av[U][MB * NA];
    int64_t ao[U], bo[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      ao[u] = g * p.gA + kk;
      bo[u] = gb * p.gB + kk;
      advance();
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int w = 0; w < TW; ++w) bv[u][w] = load_b(w, bo[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int q = 0; q < NA; ++q) av[u][mb * NA + q] = load_a(mb, ao[u] + q * p.gA2);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < NA; ++q)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int w = 0; w < TW; ++w)
            acc[mb * TW + w] = mfma16<S>(av[u][mb * NA + q], bv[u][w], acc[mb * TW + w]);
  };
  int t = t0;
  for (; t + SK_UNROLL <= t1; t += SK_UNROLL) batch(I<SK_UNROLL>{});
  // the remainder in batches of 4, 2 and 1 (step by step, a wave with 7 steps waits 7 times)
  if ((t1 - t) & 4) batch(I<4>{});
  if ((t1 - t) & 2) batch(I<2>{});
  if ((t1 - t) & 1) batch(I<1>{});
  // D row 4 kq + j, column col of each 16-row block -> red[wave][mb][row * 16 + col]
#pragma unroll
  for (int q = 0; q < MB * TW; ++q)
#pragma unroll
    for (int j = 0; j < 4; ++j) red[wave][q][(kq * 4 + j) * 16 + col] = acc[q][j];
  __syncthreads();
  const float* biasz = p.bias ? p.bias + z * p.sBias : nullptr;
  float amax = 0.f;
  for (int idx = threadIdx.x; idx < MB * TW * 256; idx += 64 * NW) {
    const int q = idx >> 8, e = idx & 255;               // block q, element e
    const int mb = q / TW, w = q - mb * TW;
    const int n = n0 + w * 16 + (e & 15), m = mb * 16 + (e >> 4);
    if (n >= p.N || m >= p.M) continue;
    float part[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) part[k] = red[k][q][e];
#pragma unroll
    for (int d = 1; d < NW; d <<= 1)
#pragma unroll
      for (int k = 0; k + d < NW; k += 2 * d) part[k] += part[k + d];
    float v = part[0] + (EPI != EPI_PART && biasz ? biasz[n] : 0.f);
    if constexpr (EPI == EPI_BIAS_N_GELU) v = gelu_erf(v);
    if constexpr (epi_res<EPI>) {
      if (p.R) v += p.R[z * p.sR + (int64_t)m * p.ldc + n];
    }
    track4<OutT>(amax, make_float4(v, 0.f, 0.f, 0.f));
    if constexpr (EPI == EPI_QKV) {
      if (kv.cache && n >= kv.dq) {
        store_val<S>(static_cast<S*>(kv.cache) + kv_place(kv, z, m, n - kv.dq), v);
        continue;
      }
      if (!kv.cache && n >= kv.dq + kv.dkv) {
        store_val<S>(static_cast<S*>(kv.vt) + z * kv.svt +
                         (int64_t)(n - kv.dq - kv.dkv) * kv.ldv + m, v);
        continue;
      }
    }
    OutT* dst = static_cast<OutT*>(p.C) + z * p.sC + (int64_t)m * p.ldc + n +
                (EPI == EPI_PART ? sp * p.sPlane : 0);
    store_val<OutT>(dst, v);
    if constexpr (EPI == EPI_BIAS_N_HILO) store_val<OutT>(dst + p.sPlane, v - (float)(S)v);
  }
  flag_overflow<OutT>(amax, p.ovf);
}

template <typename S, int MB, int TW, int NW>
hipError_t launch_skinny(const GemmDesc& g, hipStream_t s) {
  GemmParams p = gemm_params(g);
  p.tiles_n = (g.N + 16 * TW - 1) / (16 * TW);
  const dim3 grid((unsigned)p.tiles_n, (unsigned)g.batch, (unsigned)p.splits), block(64 * NW);
  switch (g.epi) {
    case EPI_BIAS_N:
      hipLaunchKernelGGL((gemm_skinny_kernel<S, MB, TW, NW, EPI_BIAS_N, false>), grid, block, 0,
                         s, p, qkv_arg<EPI_BIAS_N>(g));
      break;
    case EPI_BIAS_N_GELU:
      hipLaunchKernelGGL((gemm_skinny_kernel<S, MB, TW, NW, EPI_BIAS_N_GELU, false>), grid, block,
                         0, s, p, qkv_arg<EPI_BIAS_N_GELU>(g));
      break;
    case EPI_BIAS_N_RES:
      if constexpr (sizeof(S) == 2) {
        if (g.gA2 != 0) {
          hipLaunchKernelGGL((gemm_skinny_kernel<S, MB, TW, NW, EPI_BIAS_N_RES, true>), grid,
                             block, 0, s, p, qkv_arg<EPI_BIAS_N_RES>(g));
          break;
        }
      }
      hipLaunchKernelGGL((gemm_skinny_kernel<S, MB, TW, NW, EPI_BIAS_N_RES, false>), grid, block,
                         0, s, p, qkv_arg<EPI_BIAS_N_RES>(g));
      break;
    case EPI_BIAS_N_HILO:
      if constexpr (sizeof(S) == 2) {
        hipLaunchKernelGGL((gemm_skinny_kernel<S, MB, TW, NW, EPI_BIAS_N_HILO, false>), grid,
                           block, 0, s, p, qkv_arg<EPI_BIAS_N_HILO>(g));
        break;
      }
      return hipErrorInvalidValue;
    case EPI_PART:
      if constexpr (sizeof(S) == 2) {
        if (g.gA2 != 0) {
          hipLaunchKernelGGL((gemm_skinny_kernel<S, MB, TW, NW, EPI_PART, true>), grid, block, 0, s,
                             p, qkv_arg<EPI_PART>(g));
          break;
        }
      }
      hipLaunchKernelGGL((gemm_skinny_kernel<S, MB, TW, NW, EPI_PART, false>), grid, block, 0, s, p,
                         qkv_arg<EPI_PART>(g));
      break;
    case EPI_QKV:
      hipLaunchKernelGGL((gemm_skinny_kernel<S, MB, TW, NW, EPI_QKV, false>), grid, block, 0, s, p,
                         qkv_arg<EPI_QKV>(g));
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

// The forms that skinny_plan chooses, no others: 16-bit operands up to 32 rows, fp32 up to 64.
template <>
hipError_t launch_gemm_skinny<KRAKEN_T>(const GemmDesc& g, int tw, int nw, hipStream_t s) {
  using S = KRAKEN_T;
  if constexpr (sizeof(S) == 2) {
    if (g.M <= 16 && tw == 1 && nw == 4) return launch_skinny<S, 1, 1, 4>(g, s);
    if (g.M <= 16 && tw == 1 && nw == 8) return launch_skinny<S, 1, 1, 8>(g, s);
    if (g.M <= 16 && tw == 2 && nw == 8) return launch_skinny<S, 1, 2, 8>(g, s);
    if (g.M > 16 && g.M <= 32 && tw == 1 && nw == 8) return launch_skinny<S, 2, 1, 8>(g, s);
  } else {
    if (g.M <= 16 && tw == 1 && nw == 16) return launch_skinny<S, 1, 1, 16>(g, s);
    if (g.M > 16 && g.M <= 32 && tw == 1 && nw == 8) return launch_skinny<S, 2, 1, 8>(g, s);
    if (g.M > 32 && g.M <= 64 && tw == 1 && nw == 8) return launch_skinny<S, 4, 1, 8>(g, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace kraken
