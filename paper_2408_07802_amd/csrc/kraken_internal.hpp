// Internal declarations shared by the Kraken HIP kernels and the runtime.
// Target: gfx950 (CDNA4), 64-lane wavefronts, MFMA matrix cores.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kraken {

typedef __bf16 bf16;
typedef _Float16 f16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Element types.  For a model, the storage type is what the caller's weight blob and
// input use; the compute type is the MFMA operand type of every GEMM and of attention.
enum class DType : int { F32 = 0, BF16 = 1, F16 = 2 };

// A pointer that is the same for every lane, moved to scalar registers.  (readfirstlane
// returns a signed int: each half is taken as unsigned before widening, or a low half with
// bit 31 set would sign-extend over the high half.)
template <typename T>
__device__ __forceinline__ const T* uniform_ptr(const T* ptr) {
  const uint64_t v = reinterpret_cast<uint64_t>(ptr);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v);
  return reinterpret_cast<const T*>(((uint64_t)hi << 32) | (uint64_t)lo);
}

inline size_t dtype_size(DType t) { return t == DType::F32 ? 4 : 2; }

template <typename S>
struct IsHalfWidth {
  static constexpr bool value = sizeof(S) == 2;
};

// One 16-byte operand chunk per lane into a 32x32 MFMA block.
// 16-bit types: the chunk is 8 consecutive k of the lane's row (k = 8*half + j), one
//   v_mfma_f32_32x32x16_{bf16,f16}.
// fp32: the chunk is 4 consecutive k; MFMA q (0..3) takes element q of both halves, so
//   lane half h supplies k = 4*h + q, the same permutation of k for A and B.
template <typename S>
__device__ __forceinline__ f32x16 mfma_chunk(uint4 a, uint4 b, f32x16 c) {
  if constexpr (__is_same(S, bf16)) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  } else if constexpr (__is_same(S, f16)) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                  __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  } else {
    const f32x4 a4 = __builtin_bit_cast(f32x4, a), b4 = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int q = 0; q < 4; ++q) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[q], b4[q], c, 0, 0, 0);
    return c;
  }
}

// Epilogues of the batched GEMM C = epi(A B^T).
enum GemmEpi : int {
  EPI_BIAS_N = 0,       // C (storage type) = acc + bias[n]
  EPI_BIAS_N_GELU = 1,  // C (storage type) = GELU(acc + bias[n]), exact erf form
  EPI_BIAS_N_RES = 2,   // C (float32)      = acc + bias[n] + R[m][n]   (bias, R optional)
  EPI_BIAS_M = 3,       // C (storage type) = acc + bias[m]
  EPI_BIAS_N_HILO = 4,  // v = acc + bias[n] + R[m][n] as two 16-bit terms: C = S(v), and
                        // S(v - S(v)) sPlane elements further
  EPI_QKV = 6,          // columns Q | K | V of one projection, each to its place (QkvOut)
  EPI_PART = 5          // C (float32)      = acc of one K split, plane sp at C + sp * sPlane
};

// Where the columns of a merged Q | K | V projection (dq + 2 dkv of them) go.  Decode step
// (cache != NULL): the Q columns to C (row stride ldc), K and V straight into the layer's KV
// cache (see launch_kv_store) at position lens[m] of slot m.  Prefill: Q | K to C, V transposed
// to vt[z][feature][ldv].
struct QkvOut {
  void* vt;
  int64_t svt;              // elements between the batch entries of vt
  void* cache;
  int ldv, dq, dkv, hd, Hkv, max_seqs, cap;
  int lens[256];            // KRAKEN_MAX_SEQS
};

// C[z][m][n] = epi( sum_g sum_k A[z][g][m][k] * B[z][g mod gBmod][n][k] )
// A element (z,g,m,k) at A + z*sA + g*gA + m*lda + k; B likewise with ldb/sB/gB;
// C element at C + z*sC + m*ldc + n; R at R + z*sR + m*ldc + n; bias at bias + z*sBias.
struct GemmDesc {
  DType dt;
  int epi;
  const void* A;
  const void* B;
  void* C;
  const float* bias;
  const float* R;
  int M, N, K;  // K per group, multiple of 64 (bf16) / 32 (fp32)
  int lda, ldb, ldc;
  int64_t sA, sB, sC, sR, sBias;
  int batch;
  int kgroups;
  int64_t gA, gB;
  int gBmod;
  // EPI_PART: number of K splits and the elements between their planes; EPI_BIAS_N_HILO:
  // elements from the high to the low terms
  int splits;
  int64_t sPlane;
  // SKINNY with EPI_BIAS_N_RES or EPI_PART: != 0 adds a second term of A, gA2 elements behind the first,
  // multiplied by the same B
  int64_t gA2;
  const QkvOut* qkv;        // EPI_QKV (host memory, read by the launch)
  // fp16 outputs only: set to 1 (vector store) when a finite fp32 result rounds to an
  // fp16 infinity (|v| >= 65520); NULL: no check
  int* ovf;
};

hipError_t launch_gemm(const GemmDesc& g, hipStream_t s);

// Kernel and tile of a GEMM.
enum class GemmKind : int { TILE256, TILE128, MID, SKINNY };
struct GemmPlan {
  GemmKind kind;
  int nb;       // MID: 32-column blocks per tile; SKINNY: 16-column blocks per workgroup (1, 2);
                // TILE128: 2 for tiles of 64 columns (16-bit operands), else 0
  int splits;   // K splits
  int waves;    // SKINNY: waves that share a workgroup's reduction (fp32 up to 16 rows: 16, else
                // 8, or 4 with 16-bit operands)
};
// Plan of a GEMM of type dt.  terms: 2 for a two-term operand A (hi and lo: W_concat of 16-bit
// operands) over kgroups K groups of weights; SKINNY multiplies both terms with one load of a
// weight (kgroups groups, gA2 != 0), the others walk terms x kgroups groups (gBmod = kgroups).
// part_elems: fp32 elements available for K-split partial planes
// (0: no split; only EPI_BIAS_N_RES results can be split).
// Only results that the caller sums itself (see PartSum) may be given part_elems > 0; own_sum:
// the sum takes a launch of its own.
GemmPlan plan_gemm(DType dt, int epi, int M, int N, int K, int kgroups, int terms, int batch,
                   int64_t part_elems, bool own_sum);
hipError_t launch_gemm_planned(const GemmDesc& g, const GemmPlan& plan, hipStream_t s);
// The kernels of the plans TILE256 / TILE128, MID and SKINNY (one object file per operand type).
template <typename S>
hipError_t launch_gemm_tile(const GemmDesc& g, int cols, hipStream_t s);
template <typename S>
hipError_t launch_gemm_mid(const GemmDesc& g, int nb, hipStream_t s);
template <typename S>
hipError_t launch_gemm_skinny(const GemmDesc& g, int tw, int nw, hipStream_t s);
template <> hipError_t launch_gemm_skinny<bf16>(const GemmDesc&, int, int, hipStream_t);
template <> hipError_t launch_gemm_skinny<f16>(const GemmDesc&, int, int, hipStream_t);
template <> hipError_t launch_gemm_skinny<float>(const GemmDesc&, int, int, hipStream_t);
template <> hipError_t launch_gemm_tile<bf16>(const GemmDesc&, int, hipStream_t);
template <> hipError_t launch_gemm_tile<f16>(const GemmDesc&, int, hipStream_t);
template <> hipError_t launch_gemm_tile<float>(const GemmDesc&, int, hipStream_t);
template <> hipError_t launch_gemm_mid<bf16>(const GemmDesc&, int, hipStream_t);
template <> hipError_t launch_gemm_mid<f16>(const GemmDesc&, int, hipStream_t);
template <> hipError_t launch_gemm_mid<float>(const GemmDesc&, int, hipStream_t);

// Causal flash attention over packed sequences; n_kv_heads key/value heads (query head
// h reads head h / (n_heads / n_kv_heads)), dkv = n_kv_heads * hd.
struct AttnDesc {
  DType dt;
  const void* qk;   // [n][T][d + dkv]   (Q | K per row)
  const void* vt;   // [n][dkv][ldv]     (V transposed)
  void* out;        // [n][T][d]
  int n, T, d, n_heads, n_kv_heads;
  const int32_t* cu_host;  // host cu_seqlens [num_seqs + 1]
  int num_seqs;
  int q_prescaled;          // the Q columns already carry log2(e) / sqrt(hd)
};

hipError_t launch_attention(const AttnDesc& a, hipStream_t s);

// Row stride (elements) of the transposed V buffer for T tokens: a multiple of 64,
// so that every 8-token group of a row starts on a 16-byte boundary.
inline int vt_ld(int T) { return (T + 63) & ~63; }

// Sets columns [c0, c1) of `rows` rows (row stride ld elements) to zero.
hipError_t launch_zero_cols(DType dt, void* base, int64_t rows, int64_t ld, int c0, int c1,
                            hipStream_t s);

// A GEMM result left as partial planes, to be summed by the kernel that reads it:
// v[i][t][c] = sum_s part[s * plane + (i T + t) d + c] + bias[i d + c] + bias2[i d + c]
//              + res[i * res_stride + t d + c]     (s < splits; bias, bias2, res may be NULL)
// splits = 0: nothing to sum.  out (if not NULL) receives v, [n][T][d] fp32.
struct PartSum {
  const float* part = nullptr;
  int splits = 0;
  int64_t plane = 0;
  const float* bias = nullptr;
  const float* bias2 = nullptr;
  const float* res = nullptr;
  int64_t res_stride = 0;
  float* out = nullptr;
};

// LayerNorm of n rows-sets: out[i][t] = LN(x[i*xs + t*d]) with per-i gamma/beta.  Rows are
// d wide (the stored width); the statistics cover the first dl (logical width, a multiple
// of 4; padding columns past it hold zeros and have gamma = beta = 0).
// ovf (fp16 outputs; may be NULL): set to 1 when an output overflows the fp16 range.
// ps.splits > 0: the rows are ps's sum (and go to ps.out) instead of x.
hipError_t launch_layernorm(DType dt, const float* x, int64_t x_batch_stride, const float* gamma,
                            const float* beta, void* out, int n, int T, int d, int dl, float eps,
                            int* ovf, hipStream_t s, const PartSum& ps = PartSum());

// out[i][t] = LN(h[i][t] + y[t]); y = shared[t] or sum_k x[k][t].  d, dl, ovf as for LN1.
// ps.splits > 0: h is ps's sum (and goes to ps.out).
hipError_t launch_combine_ln2(DType dt, const float* x, const float* shared, const float* h,
                              const float* gamma, const float* beta, void* out, int n, int T,
                              int d, int dl, float eps, int* ovf, hipStream_t s,
                              const PartSum& ps = PartSum());

// v = ps's sum (with splits = 0: bias and res alone) over n x T rows of d elements, written as
// fp32 to ps.out with row stride out_ld (NULL: not), and as the two 16-bit terms hi = S(v) at
// hilo and lo = S(v - hi) at hilo + n T d (NULL: not; dt then names S).  ovf as for LN1 (a hi
// term that overflows fp16).
hipError_t launch_finish(DType dt, const PartSum& ps, int n, int T, int d, int64_t out_ld,
                         void* hilo, int* ovf, hipStream_t s);

// dst[r * dst_ld + pad(c)] = float(src[r * src_ld + c]) for r < R, c < C, with
// pad(c) = (c / g) * gp + c % g (logical element c of group c / g, placed in a group of gp
// slots; g = gp: no padding).  Untouched destination elements keep their values.
hipError_t launch_to_f32_2d(DType st, const void* src, int64_t src_ld, float* dst,
                            int64_t dst_ld, int R, int C, int g, int gp, hipStream_t s);

// dst[r * dst_ld + c] = float(src[r * src_ld + c]) for c < C, 0 for C <= c < dst_ld, r < R, where
// rows_to_f32_ok: C and the strides multiples of 4, src aligned to four elements.
bool rows_to_f32_ok(DType st, const void* src, int64_t src_ld, int64_t dst_ld, int C);
hipError_t launch_rows_to_f32(DType st, const void* src, int64_t src_ld, float* dst, int64_t dst_ld,
                              int64_t R, int C, hipStream_t s);

// dst[r * dst_ld + c] = Dst(src[r * src_ld + c]) for r < R, c < C; *overflow as for
// launch_transpose.
hipError_t launch_convert_2d(DType src_t, const void* src, int64_t src_ld, DType dst_t, void* dst,
                             int64_t dst_ld, int R, int C, int* overflow, hipStream_t s);

// X[t][c] = tok[ids[t]][c] + pos[pos_ids[t]][c] for c < dp (device ids and positions).
hipError_t launch_embed(DType dt, const int* ids, const int* pos_ids, const void* tok,
                        const float* pos, float* X, int T, int dp, hipStream_t s);

// dst[b][:] = src[rows[b]][:], fp32 rows of dp elements (device rows).
hipError_t launch_gather_rows(const float* src, const int* rows, float* dst, int B, int dp,
                              hipStream_t s);

// dst[k] = float(src[k]) for k < count.
hipError_t launch_to_f32(DType dt, const void* src, float* dst, int64_t count, hipStream_t s);

// dst[pad_c(c)][pad_r(r)] = Dst(src[r*src_ld + c]) for r < R, c < C, dst row stride dst_ld,
// with pad_r(r) = (r / gr) * grp + r % gr and pad_c likewise with (gc, gcp) (see
// launch_to_f32_2d; gr = grp and gc = gcp: a plain transpose).  When the destination is
// fp16 and a finite source value does not fit, *overflow is set to 1.
hipError_t launch_transpose(DType src_t, const void* src, int64_t src_ld, DType dst_t, void* dst,
                            int64_t dst_ld, int R, int C, int* overflow, hipStream_t s,
                            int gr = 1, int grp = 1, int gc = 1, int gcp = 1);

// KV cache of one layer: [n][2 (K, V)][max_seqs][n_kv_heads][capacity][hd], compute
// type; dkv = n_kv_heads * hd.  Prefill: K from columns d .. d+dkv-1 of qk [n][T][d + dkv],
// V from vt [n][dkv][vt_ld(T)]; token t of sequence b (cu_host[b] <= t < cu_host[b+1])
// goes to position t - cu_host[b] of slot b.
hipError_t launch_kv_store(DType dt, const void* qk, const void* vt, void* cache_layer, int n,
                           int T, int d, int n_heads, int n_kv_heads, const int32_t* cu_host,
                           int num_seqs, int max_seqs, int capacity, hipStream_t s);

// Decode: the K columns of qk [n][B][d + dkv] and v [n][B][dkv] at position lens_host[b]
// of slot b.
hipError_t launch_kv_append(DType dt, const void* qk, const void* v, void* cache_layer, int n,
                            int B, int d, int n_heads, int n_kv_heads, const int32_t* lens_host,
                            int max_seqs, int capacity, hipStream_t s);

// fp32 elements of the decode-attention partials for `splits` key chunks.
int64_t decode_partial_floats(int n, int B, int n_heads, int hd, int splits);

// out [n][B][d] = attention of the Q columns of qk [n][B][d + dkv] over keys
// 0..lens_host[b] of slot b (the new token's own included, already appended).  part: fp32
// scratch of part_floats elements; the key range is split into as many chunks as it holds.
// q_prescaled: the Q columns already carry log2(e) / sqrt(hd).
hipError_t launch_decode_attention(DType dt, const void* qk, const void* cache_layer,
                                   float* part, int64_t part_floats, void* out, int n, int B,
                                   int d, int n_heads, int n_kv_heads, const int32_t* lens_host,
                                   int max_seqs, int capacity, int q_prescaled, hipStream_t s);

// p[k] *= c for k < count (operand type dt).
hipError_t launch_scale(DType dt, void* p, int64_t count, float c, hipStream_t s);

}  // namespace kraken
