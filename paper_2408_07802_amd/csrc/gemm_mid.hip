// Batched MFMA GEMM for some tens to a few hundred rows: C[z] = epi(A[z] B[z]^T), the shape of a
// short prompt's or a large decode batch's projections.  (plan_gemm takes it from 17 rows on, or
// where the few-row kernel ends, up to 512, up to 2560 where 128 x 128 tiles would leave CUs
// idle; fp32 there at any number of rows.)
//
// Every weight (B) element is used M times only, so the launch is bound by streaming the
// weights, and what matters is how many weight bytes are in flight.  The tiled kernel keeps
// one B slice per workgroup in flight and needs a full memory latency (about 1.5 us under
// load) per 64-element slice: 3.3 TB/s with 312 workgroups.  Here one workgroup per CU owns
// 128 rows x 32 NB columns and keeps a ring of slices of each operand in LDS: 3 or 4 slices of
// A (activations: L2 hits) and as many of B as fill the rest (64 to 100 KB per CU), all of
// them but the one being multiplied on their way.
//
// Measured with weights from HBM, 128 rows, fp16 (before: the 128 x 128 tiled kernel): 4 x
// 4992 -> 9984 columns 115 -> 78 us (5.1 TB/s), 4 x 1280 -> 3072 21 -> 14 us; with K splits,
// 4 x 4992 -> 4992 73 -> 46 us, 4 x 2496 -> 1280 36 -> 11 us, a W_concat of 39936 -> 4992
// 491 -> 80 us (two terms of 19968: its 199 MB of weights come twice, 2.5 TB/s of them once).
// Within a layer (counters and times in profiles/short_prompt_kernels.md) the first of these reads
// 417 MB in 97 us.  With every wave loading and multiplying, one ring for both operands and five
// slices on their way: 4 x 1280 -> 3072 16 us, a W_concat of 10240 -> 1280 13.9 (now 12.8) us.
//
// 8 waves, two per SIMD: 4 loaders only issue the direct-to-LDS loads (two waves for each
// operand: the counter of outstanding loads is in issue order, so in one wave a wait for a
// near A slice would wait for far B slices too), 4 consumers only read
// fragments and multiply (wave w owns rows 32 w .. + 31 of all the tile's columns, NB blocks
// of 32 x 32 MFMAs).  A CU takes 64 bytes of such loads per cycle, 320 to 640 cycles per
// slice during which the issuing wave stalls; with one wave per SIMD doing both, that time
// came on top of the multiplication's.  The (kgroups x K) reduction may be split over
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

// Ring stages: 4 slices of A (3 beside wide B tiles), then as many of B as fit the LDS and
// the 6-bit load counter.
template <int NB>
struct MidRing {
  static constexpr int A = NB <= 4 ? 4 : 3;
  static constexpr int LDS_FIT = (160 * 1024 - A * MID_BM * 128) / (32 * NB * 128);
  static constexpr int COUNT_FIT = 63 / (2 * NB);
  static constexpr int CAP = LDS_FIT < COUNT_FIT ? LDS_FIT : COUNT_FIT;
  static constexpr int B = CAP < 16 ? CAP : 16;
};

// One loader wave's part of an operand: NI instructions of 8 rows per slice into a ring of NST
// stages.  next() returns the current slice's source and moves on to the next one.
template <int NI, int NST, class Next>
__device__ __forceinline__ void mid_load(uint32_t dst, uint32_t stage_bytes, const uint32_t* off,
                                         int nsl, Next&& next) {
  uint32_t st = 0;                             // byte offset of the next stage to fill
  auto issue = [&]() {
    const char* src = uniform_ptr(next());
    const uint32_t d = __builtin_amdgcn_readfirstlane(dst + st);
#pragma unroll
    for (int u = 0; u < NI; ++u) dma16(d + u * 1024u, src, off[u]);
    st = st + stage_bytes == NST * stage_bytes ? 0 : st + stage_bytes;
  };
  // waits until at most the last `later` issued slices are in flight (loads complete in issue
  // order)
  auto wait_later = [&](int later) {
    static_for<0, NST>([&](auto K) {
      if (later == decltype(K)::value) wait_vm<decltype(K)::value * NI>();
    });
  };
  for (int s = 0; s < NST && s < nsl; ++s) issue();
  wait_later(min(nsl, NST) - 1);
  __syncthreads();
  int s = 0;
  for (; s + NST < nsl; ++s) {                 // slices s + 2 .. s + NST - 1 may be in flight
    wait_vm<(NST - 2) * NI>();
    __syncthreads();
    issue();
  }
  for (; s < nsl; ++s) {                       // nothing left to issue
    if (s + 1 < nsl) wait_later(nsl - s - 2);
    __syncthreads();
  }
}

template <typename S, int NB, int EPI>
__global__ __launch_bounds__(512, 1) void gemm_mid_kernel(GemmParams p, QkvArg<EPI> kv) {
  constexpr int BM = MID_BM, BN = 32 * NB;
  constexpr int CH = 8;                        // 16-byte chunks per 128-byte row
  constexpr int EPC = 16 / sizeof(S);
  constexpr int BK = CH * EPC;                 // K elements per slice
  constexpr int NA = MidRing<NB>::A, NSB = MidRing<NB>::B;
  constexpr int AT = BM * CH, BT = BN * CH;    // uint4 per stage of A and of B
  constexpr int LDS4 = NA * AT + NSB * BT;
  static_assert(NA >= 2 && NSB >= 2 && NA * 8 <= 63 && NSB * 2 * NB <= 63, "vmcnt is 6 bits");
  static_assert(LDS4 * 16 <= 160 * 1024, "rings exceed LDS");
  __shared__ uint4 lds[LDS4];

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
  const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave = wave8 & 3;                  // consumers: block of 32 rows
  const int lrow = lane & 31, lhalf = lane >> 5;

  // this workgroup's slices [s0, s0 + nsl) of the kgroups * K / BK of the reduction
  const int ksl = p.K / BK, slices = ksl * p.kgroups;
  const int s0 = (int)((int64_t)slices * sp / p.splits);
  const int nsl = (int)((int64_t)slices * (sp + 1) / p.splits) - s0;

  constexpr int RS = BN + 4;                   // epilogue: staged row stride (floats)
  static_assert(BM * RS * 4 <= LDS4 * 16, "epilogue staging exceeds the ring");
  float* const stage = reinterpret_cast<float*>(lds);

  // Barriers: one once slice 0 is in LDS, then one per slice s, after which slice s + 1 is in
  // LDS and nobody reads slice s any more (its stage takes slice s + NST).
  if (wave8 >= 4) {
    // DMA instruction u of an operand covers 8 tile rows; a lane fetches the logical chunk
    // that the swizzle puts at its place.  Rows past M (N) load a clamped row and feed only
    // outputs that are never stored.
    const bool is_b = wave8 >= 6;
    const int half = wave8 & 1;
    const uint32_t lds_base =
        __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_ptr)lds);
    const int g0 = s0 / ksl;
    int k = s0 - g0 * ksl;
    if (!is_b) {
      uint32_t off[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int rl = half * 64 + u * 8 + (lane >> 3);
        const int m = min(m0 + rl, p.M - 1);
        off[u] = ((uint32_t)m * (uint32_t)p.lda + (uint32_t)(((lane & 7) ^ swz_key(rl)) * EPC)) *
                 (uint32_t)sizeof(S);
      }
      const S* src = static_cast<const S*>(p.A) + z * p.sA + g0 * p.gA;
      mid_load<8, NA>(lds_base + half * 8192u, AT * 16u, off, nsl, [&]() {
        const char* now = reinterpret_cast<const char*>(src + (int64_t)k * BK);
        if (++k == ksl) {
          k = 0;
          src += p.gA;
        }
        return now;
      });
    } else {
      uint32_t off[2 * NB];
#pragma unroll
      for (int u = 0; u < 2 * NB; ++u) {
        const int rl = half * (BN / 2) + u * 8 + (lane >> 3);
        const int n = min(n0 + rl, p.N - 1);
        off[u] = ((uint32_t)n * (uint32_t)p.ldb + (uint32_t)(((lane & 7) ^ swz_key(rl)) * EPC)) *
                 (uint32_t)sizeof(S);
      }
      const S* const Bz = static_cast<const S*>(p.B) + z * p.sB;
      int bg = g0 % p.gBmod;
      mid_load<2 * NB, NSB>(
          lds_base + NA * AT * 16u + half * (BN / 2) * 128u, BT * 16u, off, nsl, [&]() {
            const char* now = reinterpret_cast<const char*>(Bz + bg * p.gB + (int64_t)k * BK);
            if (++k == ksl) {
              k = 0;
              if (++bg == p.gBmod) bg = 0;
            }
            return now;
          });
    }
  } else {
    // column bias of the lane's NB columns, loaded ahead of the main loop
    constexpr bool COL_BIAS = EPI != EPI_BIAS_M && EPI != EPI_PART;
    float bnj[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int n = n0 + j * 32 + lrow;
      bnj[j] = COL_BIAS && p.bias && n < p.N ? p.bias[z * p.sBias + n] : 0.f;
    }
    f32x16 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
    // Fragment reads.  Rows base + 32 i + lrow hold logical chunk k at
    // k ^ swz_key(lrow) ^ 4 (i & 1); choff[c] is that place of the lane's part of K chunk c in
    // an even block (in an odd block it is choff[c ^ 2]).
    const int arow = (wave * 32 + lrow) * CH, brow = NA * AT + lrow * CH;
    const int apar = (wave & 1) * 2;
    int choff[CH / 2], aoff[CH / 2];
#pragma unroll
    for (int c = 0; c < CH / 2; ++c) {
      choff[c] = (2 * c + lhalf) ^ swz_key(lrow);
      aoff[c] = arow + ((2 * (c ^ apar) + lhalf) ^ swz_key(lrow));
    }
    // A half slice (two K chunks) is read one half ahead of its MFMAs; the scheduling fences
    // keep the reads there.
    uint4 af[2][2], bf[2][2][NB];
    auto read_half = [&](int sa, int sb, auto H) {   // stages of A and of B
      constexpr int h = decltype(H)::value;
      const uint4 *a = lds + sa * AT, *b = lds + sb * BT;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int c = 2 * h + k;
        af[h][k] = a[aoff[c]];
#pragma unroll
        for (int j = 0; j < NB; ++j)
          bf[h][k][j] = b[brow + j * 32 * CH + choff[(j & 1) ? c ^ 2 : c]];
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto mul_half = [&](auto H) {
      constexpr int h = decltype(H)::value;
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[j] = mfma_chunk<S>(af[h][k], bf[h][k][j], acc[j]);
      __builtin_amdgcn_sched_barrier(0);
    };
    __syncthreads();
    read_half(0, 0, I<0>{});
    int sa = 0, sb = 0;
    for (int s = 0; s < nsl; ++s) {
      read_half(sa, sb, I<1>{});
      mul_half(I<0>{});
      sa = sa + 1 == NA ? 0 : sa + 1;
      sb = sb + 1 == NSB ? 0 : sb + 1;
      __syncthreads();
      if (s + 1 < nsl) read_half(sa, sb, I<0>{});
      mul_half(I<1>{});
    }
    // (past the last barrier nobody reads the ring)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int ml = wave * 32 + (r >> 2) * 8 + lhalf * 4 + (r & 3);
        stage[ml * RS + j * 32 + lrow] = acc[j][r] + bnj[j];
      }
  }
  __syncthreads();

  // ---- epilogue: the tile is in LDS as fp32 rows; all 8 waves store it, four consecutive
  // columns per lane.
  using OutT = typename std::conditional<epi_f32<EPI>, float, S>::type;
  OutT* Cz = static_cast<OutT*>(p.C) + z * p.sC + (EPI == EPI_PART ? sp * p.sPlane : 0);
  const float* Rz = epi_res<EPI> && p.R ? p.R + z * p.sR : nullptr;
  // (results and residuals of callers, such as logits, need not be aligned to four elements)
  const bool vec_ok = (p.ldc & 3) == 0 &&
                      (reinterpret_cast<uintptr_t>(Cz) & (4 * sizeof(OutT) - 1)) == 0 &&
                      (reinterpret_cast<uintptr_t>(Rz) & 15) == 0;
  float amax = 0.f;
#pragma unroll 4
  for (int q = 0; q < 2 * NB; ++q) {
    const int idx = q * 512 + tid, ml = idx / (BN / 4), nl = (idx % (BN / 4)) * 4;
    const int m = m0 + ml, n = n0 + nl;
    if (m >= p.M || n >= p.N) continue;
    float4 v = *reinterpret_cast<const float4*>(stage + ml * RS + nl);
    if constexpr (EPI == EPI_BIAS_N_GELU)
      v = make_float4(gelu_erf(v.x), gelu_erf(v.y), gelu_erf(v.z), gelu_erf(v.w));
    if constexpr (EPI == EPI_BIAS_M) {
      const float bm = p.bias ? p.bias[z * p.sBias + m] : 0.f;
      v.x += bm; v.y += bm; v.z += bm; v.w += bm;
    }
    const int64_t at = (int64_t)m * p.ldc + n;
    if constexpr (EPI == EPI_QKV) {            // (segments of 4 columns stay in one head)
      if (kv.cache && n >= kv.dq) {
        track4<OutT>(amax, v);
        store4<S>(static_cast<S*>(kv.cache) + kv_place(kv, z, m, n - kv.dq), v);
        continue;
      }
      if (!kv.cache && n >= kv.dq + kv.dkv) continue;      // V^T: below
    }
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
  if constexpr (EPI == EPI_QKV) {
    // V transposed: lanes take consecutive features, each eight tokens of one
    const int dqk = kv.dq + kv.dkv;
    if (!kv.cache && n0 + BN > dqk) {
      for (int idx = tid; idx < BN * (BM / 8); idx += 512) {
        const int f = idx % BN, mg = idx / BN, n = n0 + f, m = m0 + mg * 8;
        if (n < dqk || n >= p.N || m >= p.M) continue;
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = stage[(mg * 8 + k) * RS + f];
        S* dst = static_cast<S*>(kv.vt) + z * kv.svt + (int64_t)(n - dqk) * kv.ldv + m;
        if (m + 8 <= p.M) {
          track4<OutT>(amax, make_float4(v[0], v[1], v[2], v[3]));
          track4<OutT>(amax, make_float4(v[4], v[5], v[6], v[7]));
          store4<S>(dst, make_float4(v[0], v[1], v[2], v[3]));
          store4<S>(dst + 4, make_float4(v[4], v[5], v[6], v[7]));
        } else {
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            if (m + k >= p.M) break;
            track4<OutT>(amax, make_float4(v[k], 0.f, 0.f, 0.f));
            store_val<S>(dst + k, v[k]);
          }
        }
      }
    }
  }
  flag_overflow<OutT>(amax, p.ovf);
}

template <typename S, int NB>
hipError_t launch_nb(const GemmDesc& g, hipStream_t s) {
  GemmParams p = gemm_params(g);
  p.tiles_m = (g.M + MID_BM - 1) / MID_BM;
  p.tiles_n = (g.N + 32 * NB - 1) / (32 * NB);
  const dim3 grid((unsigned)((int64_t)p.tiles_m * p.tiles_n * p.splits * p.batch)), block(512);
  switch (g.epi) {
    case EPI_BIAS_N:
      hipLaunchKernelGGL((gemm_mid_kernel<S, NB, EPI_BIAS_N>), grid, block, 0, s, p,
                         qkv_arg<EPI_BIAS_N>(g));
      break;
    case EPI_BIAS_N_GELU:
      hipLaunchKernelGGL((gemm_mid_kernel<S, NB, EPI_BIAS_N_GELU>), grid, block, 0, s, p,
                         qkv_arg<EPI_BIAS_N_GELU>(g));
      break;
    case EPI_BIAS_N_RES:
      hipLaunchKernelGGL((gemm_mid_kernel<S, NB, EPI_BIAS_N_RES>), grid, block, 0, s, p,
                         qkv_arg<EPI_BIAS_N_RES>(g));
      break;
    case EPI_BIAS_M:
      hipLaunchKernelGGL((gemm_mid_kernel<S, NB, EPI_BIAS_M>), grid, block, 0, s, p,
                         qkv_arg<EPI_BIAS_M>(g));
      break;
    case EPI_QKV:
      hipLaunchKernelGGL((gemm_mid_kernel<S, NB, EPI_QKV>), grid, block, 0, s, p,
                         qkv_arg<EPI_QKV>(g));
      break;
    case EPI_PART:
      hipLaunchKernelGGL((gemm_mid_kernel<S, NB, EPI_PART>), grid, block, 0, s, p,
                         qkv_arg<EPI_PART>(g));
      break;
    case EPI_BIAS_N_HILO:
      if constexpr (sizeof(S) == 2) {
        hipLaunchKernelGGL((gemm_mid_kernel<S, NB, EPI_BIAS_N_HILO>), grid, block, 0, s, p,
                         qkv_arg<EPI_BIAS_N_HILO>(g));
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
