// Device helpers shared by the GEMM kernels: parameters, the GELU epilogue, output stores,
// the LDS swizzle and the direct-to-LDS loads.
#pragma once

#include <type_traits>

#include "kraken_internal.hpp"

namespace kraken {
namespace {

struct GemmParams {
  const void* A;
  const void* B;
  void* C;
  const float* bias;
  const float* R;
  int M, N, K;
  int lda, ldb, ldc;
  int64_t sA, sB, sC, sR, sBias;
  int kgroups;
  int64_t gA, gB;
  int gBmod;
  int tiles_m, tiles_n, batch;
  int xshare;              // XCDs that work through the same tile groups together (1, 2, 4, 8)
  int splits;              // workgroups that share one tile's reduction (EPI_PART: planes)
  int64_t sPlane;          // elements between partial planes (EPI_PART) or from hi to lo
  int64_t gA2;             // elements from the first to the second term of A (0: one term)
  int* ovf;                // fp16 outputs: overflow flag (NULL: not checked)
};

inline GemmParams gemm_params(const GemmDesc& g) {
  GemmParams p;
  p.A = g.A; p.B = g.B; p.C = g.C; p.bias = g.bias; p.R = g.R;
  p.M = g.M; p.N = g.N; p.K = g.K;
  p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc;
  p.sA = g.sA; p.sB = g.sB; p.sC = g.sC; p.sR = g.sR; p.sBias = g.sBias;
  p.kgroups = g.kgroups; p.gA = g.gA; p.gB = g.gB; p.gBmod = g.gBmod;
  p.tiles_m = p.tiles_n = 1;
  p.batch = g.batch;
  p.xshare = 1;
  p.splits = g.splits > 0 ? g.splits : 1;
  p.sPlane = g.sPlane;
  p.gA2 = g.gA2;
  p.ovf = g.ovf;
  return p;
}

// Epilogues that write fp32, and those that add the residual R.
template <int EPI>
constexpr bool epi_f32 = EPI == EPI_BIAS_N_RES || EPI == EPI_PART;
template <int EPI>
constexpr bool epi_res = EPI == EPI_BIAS_N_RES || EPI == EPI_BIAS_N_HILO;

// GELU(v) = v Phi(v) with Phi the standard normal CDF.  With h = Phi(-|v|) this is
// max(v, 0) - |v| h for either sign of v (v >= 0: v (1 - h); v < 0: v h).  h =
// erfc(x) / 2 at x = |v| / sqrt 2, from Abramowitz & Stegun, Handbook of Mathematical
// Functions, formula 7.1.26: for x >= 0,
//   erfc(x) = (a1 t + a2 t^2 + a3 t^3 + a4 t^4 + a5 t^5) exp(-x^2),  t = 1 / (1 + p x),
// within 1.5e-7 absolute, so the GELU error is below 1e-7 |v|.  The halving is folded
// into the coefficients and exp(-x^2) = exp2(-v^2 log2(e) / 2): eleven VALU operations
// and two transcendentals per value.
__device__ __forceinline__ float gelu_erf(float v) {
  const float a = fabsf(v);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, a, 1.0f));
  float poly = 0.5f * 1.061405429f;
  poly = fmaf(poly, t, 0.5f * -1.453152027f);
  poly = fmaf(poly, t, 0.5f * 1.421413741f);
  poly = fmaf(poly, t, 0.5f * -0.284496736f);
  poly = fmaf(poly, t, 0.5f * 0.254829592f);
  poly *= t;
  const float e = __builtin_amdgcn_exp2f(v * (v * -0.72134752044448170f));
  return fmaf(-a, poly * e, fmaxf(v, 0.0f));
}

template <typename S>
__device__ __forceinline__ void store_val(S* p, float v) {
  *p = static_cast<S>(v);
}

// fp16 overflow check of the epilogues: a value of magnitude >= 65520 rounds (to nearest
// even) to an fp16 infinity.  amax tracks the largest magnitude a thread stores; at the end
// one lane of each wave that saw an overflow sets the flag with a vector store.
constexpr float F16_OVERFLOW = 65520.0f;
template <typename OutT>
__device__ __forceinline__ void track4(float& amax, float4 v) {
  if constexpr (__is_same(OutT, f16))
    amax = fmaxf(amax, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
}
template <typename OutT>
__device__ __forceinline__ void flag_overflow(float amax, int* ovf) {
  if constexpr (__is_same(OutT, f16)) {
    if (ovf && __ballot(!(amax < F16_OVERFLOW)) && (threadIdx.x & 63) == 0) *ovf = 1;
  }
}

// Four consecutive outputs of a row segment, stored non-temporally: a tile's outputs are
// written once and read by a later kernel, and streaming stores keep the burst of every
// workgroup's epilogue from evicting the operands the other tiles are still reading
// (measured: Q,K projection -8%, output projection -6% of kernel time).
typedef float f32v4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32v2 __attribute__((ext_vector_type(2)));
template <typename S>
__device__ __forceinline__ void store4(S* p, float4 v);
template <>
__device__ __forceinline__ void store4<float>(float* p, float4 v) {
  const f32v4 w = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(w, reinterpret_cast<f32v4*>(p));
}
template <>
__device__ __forceinline__ void store4<bf16>(bf16* p, float4 v) {
  bf16x4 o;
  o[0] = (bf16)v.x; o[1] = (bf16)v.y; o[2] = (bf16)v.z; o[3] = (bf16)v.w;
  __builtin_nontemporal_store(__builtin_bit_cast(u32v2, o), reinterpret_cast<u32v2*>(p));
}
template <>
__device__ __forceinline__ void store4<f16>(f16* p, float4 v) {
  f16x4 o;
  o[0] = (f16)v.x; o[1] = (f16)v.y; o[2] = (f16)v.z; o[3] = (f16)v.w;
  __builtin_nontemporal_store(__builtin_bit_cast(u32v2, o), reinterpret_cast<u32v2*>(p));
}

// Swizzle of 16-byte chunks inside a 128-byte tile row: logical chunk k of row r sits at
// physical chunk k ^ swz_key(r).  The key mixes bit 3 of the row into bits 0-2 so that the
// 16 rows one ds_read_b128 serves per LDS cycle cover all 64 banks exactly once (rows r and
// r + 8 would collide under the plain r & 7).
__device__ __forceinline__ int swz_key(int row) { return (row ^ (row >> 3)) & 7; }

template <int N>
using I = std::integral_constant<int, N>;

// Compile-time loop: f(I<B>{}), f(I<B+1>{}), ..., f(I<E-1>{}).
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(I<B>{});
    static_for<B + 1, E>(f);
  }
}

// MFMA slot (in [lo, hi)) that item k of n evenly spread items issues after.
__host__ __device__ constexpr int spread_slot(int k, int n, int lo, int hi) {
  return lo + (k * (hi - lo)) / n;
}

typedef __attribute__((address_space(3))) void* lds_void_ptr;

// One 16-byte-per-lane DMA from global memory into LDS: global_load_lds_dwordx4 with a
// wave-uniform base address (SGPR pair), a per-lane 32-bit byte offset, and the
// wave-uniform LDS destination in M0; lane i's 16 bytes land at M0 + 16 i.  It is issued
// from inline assembly so that the compiler does not order later LDS reads of *other*
// ring slots behind it; the kernel orders it explicitly (s_waitcnt vmcnt + barrier before
// the slot is read).
__device__ __forceinline__ void dma16(uint32_t lds_addr, const void* base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds_addr), "v"(off), "s"(base) : "memory", "m0");
}

// hi = S(v), lo = v - hi (rounded to S when stored): the two-term operand of W_concat.
template <typename S>
__device__ __forceinline__ float4 split_lo(float4 v) {
  return make_float4(v.x - (float)(S)v.x, v.y - (float)(S)v.y, v.z - (float)(S)v.z,
                     v.w - (float)(S)v.w);
}

// The QkvOut kernel argument of EPI_QKV kernels (nothing for the others).
struct NoQkv {};
template <int EPI>
using QkvArg = std::conditional_t<EPI == EPI_QKV, QkvOut, NoQkv>;
template <int EPI>
QkvArg<EPI> qkv_arg(const GemmDesc& g) {
  if constexpr (EPI == EPI_QKV) return *g.qkv;
  else return {};
}

// Element of the layer's KV cache that column c >= 0 of K | V (batch entry z, row m) goes to.
__device__ __forceinline__ int64_t kv_place(const QkvOut& o, int z, int m, int c) {
  const int kv = c >= o.dkv ? 1 : 0;
  c -= kv * o.dkv;
  const int h = c / o.hd, e = c - h * o.hd;
  return (((((int64_t)z * 2 + kv) * o.max_seqs + m) * o.Hkv + h) * (int64_t)o.cap + o.lens[m]) *
             o.hd + e;
}

constexpr int MID_BM = 128;    // rows of a gemm_mid_kernel tile
constexpr int MID_MAX_NB = 6;  // its widest tile: 6 blocks of 32 columns

}  // namespace
}  // namespace kraken
