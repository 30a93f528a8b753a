// Batched MFMA GEMM for 65 to a few hundred rows: C[z] = epi(A[z] B[z]^T), the shape of a
// short prompt's or a large decode batch's projections.
//
// Every weight (B) element is used M times only, so the launch is bound by streaming the
// weights, and what matters is how many weight bytes are in flight.  The tiled kernel keeps
// one B slice per workgroup in flight and needs a full memory latency (about 1.5 us under
// load) per 64-element slice: 3.3 TB/s with 312 workgroups.  Here one workgroup per CU owns
// 128 rows x 32 NB columns and a ring of NST slices of both operands that fills the LDS, so
// NST - 1 slices (48 to 64 KB of weights per CU) are always on their way.
//
// Measured with weights from HBM, 128 rows, fp16 (before: the 128 x 128 tiled kernel): 4 x
// 4992 -> 9984 columns 115 -> 80 us (5.0 TB/s), 4 x 1280 -> 3072 21 -> 16 us; with K splits,
// 4 x 4992 -> 4992 73 -> 47 us, 4 x 2496 -> 1280 36 -> 12 us, a W_concat of 39936 -> 4992
// 491 -> 80 us.  Per 64-element slice and CU it takes about 0.16 + 0.12 NB us.
//
// 4 waves; wave w owns rows 32 w .. + 31 of all the tile's columns (1 x NB blocks of 32 x 32
// MFMAs; its A rows are loaded by itself).  The (kgroups x K) reduction may be split over
// `splits` workgroups; then each writes its fp32 partial plane and the reader of the result
// (a LayerNorm kernel, or launch_finish) adds the planes, the bias and the residual.
//
// Compiled once per operand type (KRAKEN_T).
#include "gemm_common.hpp"

namespace kraken {
namespace {

template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <typename S, int NB, int NST, int EPI>
__global__ __launch_bounds__(256, 1) void gemm_mid_kernel(GemmParams p) {
  constexpr int BM = MID_BM, BN = 32 * NB;
  constexpr int CH = 8;                        // 16-byte chunks per 128-byte row
  constexpr int EPC = 16 / sizeof(S);
  constexpr int BK = CH * EPC;                 // K elements per slice
  constexpr int AI = 4, PER = AI + NB;         // DMA instructions per wave per slice
  constexpr int STAGE = (BM + BN) * CH;        // uint4 per ring stage
  static_assert(NST >= 2 && (NST - 1) * PER <= 63, "vmcnt is a 6-bit count");
  static_assert(NST * STAGE * 16 <= 160 * 1024, "ring exceeds LDS");
  __shared__ uint4 lds[NST * STAGE];

  // XCD-aware order: workgroup b runs on XCD b % 8; each XCD takes a contiguous range of
  // tiles (rows fastest, then columns, K splits, batch entries), so that the workgroups of
  // one L2 read the same activation rows.
  const int total = p.tiles_m * p.tiles_n * p.splits * p.batch;
  int pid;
  {
    const int x = blockIdx.x & 7, l = blockIdx.x >> 3, q = total >> 3, r = total & 7;
    pid = x * q + min(x, r) + l;
  }
  pid = __builtin_amdgcn_readfirstlane(pid);
  const int tm = pid % p.tiles_m;
  int t = pid / p.tiles_m;
  const int tn = t % p.tiles_n;
  t /= p.tiles_n;
  const int sp = t % p.splits, z = t / p.splits;
  const int m0 = tm * BM, n0 = tn * BN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane & 31, lhalf = lane >> 5;

  // column bias of the lane's NB columns, loaded ahead of the main loop
  constexpr bool COL_BIAS = EPI != EPI_BIAS_M && EPI != EPI_PART;
  float bnj[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int n = n0 + j * 32 + lrow;
    bnj[j] = COL_BIAS && p.bias && n < p.N ? p.bias[z * p.sBias + n] : 0.f;
  }

  const S* Az = static_cast<const S*>(p.A) + z * p.sA;
  const S* Bz = static_cast<const S*>(p.B) + z * p.sB;
  // DMA instruction u of an operand covers 8 tile rows; a lane fetches the logical chunk that
  // the swizzle puts at its place.  Rows past M (N) load a clamped row and feed only outputs
  // that are never stored.
  uint32_t aoff[AI], boff[NB];
#pragma unroll
  for (int u = 0; u < AI; ++u) {
    const int rl = wave * 32 + u * 8 + (lane >> 3);
    const int m = min(m0 + rl, p.M - 1);
    aoff[u] = ((uint32_t)m * (uint32_t)p.lda + (uint32_t)(((lane & 7) ^ swz_key(rl)) * EPC)) *
              (uint32_t)sizeof(S);
  }
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int rl = wave * (BN / 4) + u * 8 + (lane >> 3);
    const int n = min(n0 + rl, p.N - 1);
    boff[u] = ((uint32_t)n * (uint32_t)p.ldb + (uint32_t)(((lane & 7) ^ swz_key(rl)) * EPC)) *
              (uint32_t)sizeof(S);
  }
  const uint32_t lds_base =
      __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_ptr)lds);
  const uint32_t a_dst = lds_base + (uint32_t)(wave * 32) * 128u;
  const uint32_t b_dst = lds_base + (uint32_t)(BM + wave * (BN / 4)) * 128u;

  // this workgroup's slices [s0, s1) of the kgroups * K / BK of the reduction
  const int ksl = p.K / BK, slices = ksl * p.kgroups;
  const int s0 = (int)((int64_t)slices * sp / p.splits);
  const int nsl = (int)((int64_t)slices * (sp + 1) / p.splits) - s0;
  int ld_g = s0 / ksl, ld_k = s0 - ld_g * ksl, ld_bg = ld_g % p.gBmod;
  const char* a_src = reinterpret_cast<const char*>(Az + ld_g * p.gA + (int64_t)ld_k * BK);
  const char* b_src = reinterpret_cast<const char*>(Bz + ld_bg * p.gB + (int64_t)ld_k * BK);
  // loads the next slice into ring stage st
  auto issue = [&](int st) {
    const uint32_t off = __builtin_amdgcn_readfirstlane((uint32_t)(st * STAGE) * 16u);
    const char *a = uniform_ptr(a_src), *b = uniform_ptr(b_src);
#pragma unroll
    for (int u = 0; u < NB; ++u) dma16(b_dst + off + u * 1024u, b, boff[u]);
#pragma unroll
    for (int u = 0; u < AI; ++u) dma16(a_dst + off + u * 1024u, a, aoff[u]);
    if (++ld_k < ksl) {
      a_src += BK * sizeof(S);
      b_src += BK * sizeof(S);
    } else {
      ld_k = 0;
      ++ld_g;
      if (++ld_bg == p.gBmod) ld_bg = 0;
      a_src = reinterpret_cast<const char*>(Az + ld_g * p.gA);
      b_src = reinterpret_cast<const char*>(Bz + ld_bg * p.gB);
    }
  };

  f32x16 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;

  // Fragment reads.  Rows base + 32 i + lrow hold logical chunk k at k ^ swz_key(lrow) ^ 4 (i & 1);
  // choff[c] is that place of the lane's part of K chunk c in an even block (in an odd block
  // it is choff[c ^ 2]).
  const int arow = (wave * 32 + lrow) * CH, brow = (BM + lrow) * CH;
  const int apar = wave & 1;
  int choff[CH / 2];
#pragma unroll
  for (int c = 0; c < CH / 2; ++c) choff[c] = (2 * c + lhalf) ^ swz_key(lrow);
  uint4 af[2], bf[2][NB];
  auto read_chunk = [&](int st, auto Cc) {
    constexpr int c = decltype(Cc)::value;
    const uint4* base = lds + st * STAGE;
    af[c & 1] = base[arow + (apar ? choff[c ^ 2] : choff[c])];
#pragma unroll
    for (int j = 0; j < NB; ++j)
      bf[c & 1][j] = base[brow + j * 32 * CH + choff[(j & 1) ? c ^ 2 : c]];
  };
  // The reads of chunk c + 1 go out before the MFMAs of chunk c (the scheduling fences keep
  // the compiler from moving them back behind one register set, which made every read's
  // latency visible).
  auto compute = [&](int st) {
    static_for<0, CH / 2>([&](auto Cc) {
      constexpr int c = decltype(Cc)::value;
      if constexpr (c + 1 < CH / 2) read_chunk(st, I<c + 1>{});
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[j] = mfma_chunk<S>(af[c & 1], bf[c & 1][j], acc[j]);
      __builtin_amdgcn_sched_barrier(0);
    });
  };

#pragma unroll
  for (int s = 0; s < NST - 1; ++s)
    if (s < nsl) issue(s);
  int st = 0;
  int s = 0;
  // Slice s is complete once at most the NST - 2 later slices are outstanding; after the
  // barrier nobody reads stage s - 1 any more, and slice s + NST - 1 goes there.
  for (; s + NST - 1 < nsl; ++s) {
    wait_vm<(NST - 2) * PER>();
    __syncthreads();
    read_chunk(st, I<0>{});
    __builtin_amdgcn_sched_barrier(0);
    issue(st == 0 ? NST - 1 : st - 1);
    compute(st);
    st = st + 1 == NST ? 0 : st + 1;
  }
  for (; s < nsl; ++s) {                       // the last NST - 1 slices: nothing to load
    const int later = nsl - 1 - s;
    static_for<0, NST - 1>([&](auto K) {
      if (later == decltype(K)::value) wait_vm<decltype(K)::value * PER>();
    });
    __syncthreads();
    read_chunk(st, I<0>{});
    compute(st);
    st = st + 1 == NST ? 0 : st + 1;
  }
  __syncthreads();

  // ---- epilogue: each wave writes its 32 x BN block to LDS (MFMA layout: lane = column, 16
  // rows per lane) and reads it back four consecutive columns per lane.
  using OutT = typename std::conditional<epi_f32<EPI>, float, S>::type;
  constexpr int RS = BN + 4;
  static_assert(4 * 32 * RS * 4 <= NST * STAGE * 16, "epilogue staging exceeds the ring");
  float* stage = reinterpret_cast<float*>(lds) + wave * 32 * RS;
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int ml = (r >> 2) * 8 + lhalf * 4 + (r & 3);
      float v = acc[j][r] + bnj[j];
      if constexpr (EPI == EPI_BIAS_N_GELU) v = gelu_erf(v);
      stage[ml * RS + j * 32 + lrow] = v;
    }
  __builtin_amdgcn_s_waitcnt(0xc07f);          // lgkmcnt(0): this wave's LDS writes are done
  __builtin_amdgcn_wave_barrier();
  OutT* Cz = static_cast<OutT*>(p.C) + z * p.sC + (EPI == EPI_PART ? sp * p.sPlane : 0);
  const float* Rz = epi_res<EPI> && p.R ? p.R + z * p.sR : nullptr;
  const bool vec_ok = (p.ldc & 3) == 0;
  float amax = 0.f;
#pragma unroll 4
  for (int q = 0; q < 4 * NB; ++q) {
    const int idx = q * 64 + lane, ml = idx / (BN / 4), nl = (idx % (BN / 4)) * 4;
    const int m = m0 + wave * 32 + ml, n = n0 + nl;
    if (m >= p.M || n >= p.N) continue;
    float4 v = *reinterpret_cast<const float4*>(stage + ml * RS + nl);
    if constexpr (EPI == EPI_BIAS_M) {
      const float bm = p.bias ? p.bias[z * p.sBias + m] : 0.f;
      v.x += bm; v.y += bm; v.z += bm; v.w += bm;
    }
    const int64_t at = (int64_t)m * p.ldc + n;
    if (vec_ok && n + 3 < p.N) {
      if (Rz) {
        const float4 rr = *reinterpret_cast<const float4*>(Rz + at);
        v.x += rr.x; v.y += rr.y; v.z += rr.z; v.w += rr.w;
      }
      track4<OutT>(amax, v);
      store4<OutT>(Cz + at, v);
      if constexpr (EPI == EPI_BIAS_N_HILO) store4<OutT>(Cz + p.sPlane + at, split_lo<S>(v));
    } else {
      const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (n + k >= p.N) break;
        float o = vv[k];
        if (Rz) o += Rz[at + k];
        track4<OutT>(amax, make_float4(o, 0.f, 0.f, 0.f));
        store_val<OutT>(Cz + at + k, o);
        if constexpr (EPI == EPI_BIAS_N_HILO)
          store_val<OutT>(Cz + p.sPlane + at + k, o - (float)(S)o);
      }
    }
  }
  flag_overflow<OutT>(amax, p.ovf);
}

// Ring stages that fit the LDS (at most 6).
template <int NB>
constexpr int mid_stages() {
  constexpr int n = 160 * 1024 / ((MID_BM + 32 * NB) * 128);
  return n < 6 ? n : 6;
}

template <typename S, int NB>
hipError_t launch_nb(const GemmDesc& g, hipStream_t s) {
  constexpr int NST = mid_stages<NB>();
  GemmParams p = gemm_params(g);
  p.tiles_m = (g.M + MID_BM - 1) / MID_BM;
  p.tiles_n = (g.N + 32 * NB - 1) / (32 * NB);
  const dim3 grid((unsigned)((int64_t)p.tiles_m * p.tiles_n * p.splits * p.batch)), block(256);
  switch (g.epi) {
    case EPI_BIAS_N:
      hipLaunchKernelGGL((gemm_mid_kernel<S, NB, NST, EPI_BIAS_N>), grid, block, 0, s, p);
      break;
    case EPI_BIAS_N_GELU:
      hipLaunchKernelGGL((gemm_mid_kernel<S, NB, NST, EPI_BIAS_N_GELU>), grid, block, 0, s, p);
      break;
    case EPI_BIAS_N_RES:
      hipLaunchKernelGGL((gemm_mid_kernel<S, NB, NST, EPI_BIAS_N_RES>), grid, block, 0, s, p);
      break;
    case EPI_BIAS_M:
      hipLaunchKernelGGL((gemm_mid_kernel<S, NB, NST, EPI_BIAS_M>), grid, block, 0, s, p);
      break;
    case EPI_PART:
      hipLaunchKernelGGL((gemm_mid_kernel<S, NB, NST, EPI_PART>), grid, block, 0, s, p);
      break;
    case EPI_BIAS_N_HILO:
      if constexpr (sizeof(S) == 2) {
        hipLaunchKernelGGL((gemm_mid_kernel<S, NB, NST, EPI_BIAS_N_HILO>), grid, block, 0, s, p);
        break;
      }
      return hipErrorInvalidValue;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename S>
hipError_t launch_typed(const GemmDesc& g, int nb, hipStream_t s) {
  switch (nb) {
    case 1: return launch_nb<S, 1>(g, s);
    case 2: return launch_nb<S, 2>(g, s);
    case 3: return launch_nb<S, 3>(g, s);
    case 4: return launch_nb<S, 4>(g, s);
    case 5: return launch_nb<S, 5>(g, s);
    case 6: return launch_nb<S, 6>(g, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

template <>
hipError_t launch_gemm_mid<KRAKEN_T>(const GemmDesc& g, int nb, hipStream_t s) {
  return launch_typed<KRAKEN_T>(g, nb, s);
}

}  // namespace kraken
