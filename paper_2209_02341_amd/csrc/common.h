// Shared device helpers and the launch functions each kernel file exports.
// gfx950 only: 64-lane wavefronts, bf16 MFMA, hardware bf16 conversion.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace energon {

typedef __bf16 bf16_t;
typedef _Float16 f16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
template <typename E> using vec8 = E __attribute__((ext_vector_type(8)));   // one MFMA operand fragment
template <typename E> using vec4 = E __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kWave = 64;
constexpr int kXcds = 8;
constexpr int kGroupM = 8;        // row tiles per band

// XCD-aware tile order; false if this workgroup is one of the (< 8) padding ids.
template <int BM, int BN>
__device__ __forceinline__ bool tile_origin(int32_t tiles_m, int32_t tiles_n, int64_t& m0, int32_t& n0) {
  const int32_t total = tiles_m * tiles_n;
  const int32_t per_xcd = (total + kXcds - 1) / kXcds;
  const int32_t idx = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  if (idx >= total) return false;
  const int32_t band = idx / (kGroupM * tiles_n);
  const int32_t first_m = band * kGroupM;
  const int32_t band_m = min(kGroupM, tiles_m - first_m);
  const int32_t r = idx - band * kGroupM * tiles_n;
  m0 = (int64_t)(first_m + r % band_m) * BM;
  n0 = (r / band_m) * BN;
  return true;
}

// Element traits: VEC elements make one 16-byte vector.
template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int VEC = 4;
  __device__ static inline float to_f32(float v) { return v; }
  __device__ static inline float from_f32(float v) { return v; }
};
template <> struct Elem<bf16_t> {
  static constexpr int VEC = 8;
  __device__ static inline float to_f32(bf16_t v) { return static_cast<float>(v); }
  __device__ static inline bf16_t from_f32(float v) { return static_cast<bf16_t>(v); }  // RNE
};

template <> struct Elem<f16_t> {
  static constexpr int VEC = 8;
  __device__ static inline float to_f32(f16_t v) { return static_cast<float>(v); }
  __device__ static inline f16_t from_f32(float v) { return static_cast<f16_t>(v); }  // RNE
};

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Transposed LDS read (ds_read_b64_tr_b16).  In each group of 16 lanes, lane i gives the address of four consecutive
// 16-bit elements, columns 4 (i % 4) .. + 3 of row i / 4 of a 4 x 16 block, and receives column i of the block.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ inline s16x4 lds_read_tr16(lds_ptr_t base, uint32_t off) {
  typedef __attribute__((address_space(3))) s16x4* p;
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((p)((__attribute__((address_space(3))) char*)base + off));
}

// The two 16-bit MFMA forms of gfx950 for an element type (bf16 or fp16), fp32 accumulation.
template <typename E> struct Mfma;
template <> struct Mfma<bf16_t> {
  __device__ static inline f32x16 m32x32x16(vec8<bf16_t> a, vec8<bf16_t> b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  __device__ static inline f32x4 m16x16x32(vec8<bf16_t> a, vec8<bf16_t> b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
  __device__ static inline vec4<bf16_t> read_tr(lds_ptr_t base, uint32_t off) {
    return __builtin_bit_cast(vec4<bf16_t>, lds_read_tr16(base, off));
  }
};
template <> struct Mfma<f16_t> {
  __device__ static inline f32x16 m32x32x16(vec8<f16_t> a, vec8<f16_t> b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
  __device__ static inline f32x4 m16x16x32(vec8<f16_t> a, vec8<f16_t> b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
  __device__ static inline vec4<f16_t> read_tr(lds_ptr_t base, uint32_t off) {
    return __builtin_bit_cast(vec4<f16_t>, lds_read_tr16(base, off));
  }
};

constexpr float kLowest = -3.402823466e+38f;   // the lowest finite float: where a running max starts

template <typename T> struct alignas(16) Vec16 { T v[Elem<T>::VEC]; };

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// LDS rows of 128 bytes read as 16-row MFMA operands (lane l: row l % 16, chunk 4 h + l / 16 of 16 bytes): chunk c of row r
// lies in slot c ^ swz16(r), row bits 1, 2, 3 going to slot bits 0, 2, 1; such a read then meets no bank conflict (measured).
__device__ __forceinline__ int swz16(int row) {
  return ((row >> 1) & 1) | (((row >> 2) & 1) << 2) | (((row >> 3) & 1) << 1);
}

// LDS of a workgroup whose WK wavefronts cut K: each has a ring of kDepth slabs of 128 bytes of 16 TN rows of W and 16 TM of x,
// in whose place the fp32 sums of all of them meet at the end.
template <int TM, int TN, int WK, int kDepth> struct WaveRings {
  static constexpr int kSlotVecs = (TM + TN) * 16 * 8;   // 16-byte vectors per slab: W rows, then x rows
  static constexpr size_t kRing = (size_t)WK * kDepth * kSlotVecs * 16;
  static constexpr size_t kRed = (size_t)WK * TN * TM * 1024;
  static constexpr size_t kLds = kRing > kRed ? kRing : kRed;
};

// GeLU in its erf form, z * Phi(z) = 0.5 z (1 + erf(z / sqrt 2)), in fp32, written without the
// cancellation of 1 + erf for negative z:
//   GeLU(z) = max(z, 0) - 0.5 |z| erfc(|z| / sqrt 2),
// with erfc(|z| / sqrt 2) = 2^P(|z|), P a degree-7 polynomial without constant term.  Its
// coefficients are a weighted least-squares fit (reweighted towards the minimax solution) of
// log2 erfc on 0 <= |z| <= 7.35, weighted by the error the term leaves on GeLU, with the leading
// coefficient held negative so that P -> -inf and 2^P -> 0 beyond the fitted range.  Absolute
// error on GeLU <= 1.3e-7 before the final fp32 rounding (a host-side test re-evaluates these
// constants against a library erf); one transcendental instruction and ten multiply-adds per
// element, branch-free, |z| taken as an operand modifier.
constexpr float kGeluErfcPoly[7] = {-1.1511532068252563f,    -0.4588780403137207f,   -0.05332031473517418f,
                                    0.008061456494033337f,   -0.0007832530536688864f, 4.081824226886965e-05f,
                                    -1.0515688018131186e-06f};
__device__ inline float gelu_erf(float z) {
  const float a = fabsf(z);
  float p = fmaf(kGeluErfcPoly[6], a, kGeluErfcPoly[5]);
  p = fmaf(p, a, kGeluErfcPoly[4]);
  p = fmaf(p, a, kGeluErfcPoly[3]);
  p = fmaf(p, a, kGeluErfcPoly[2]);
  p = fmaf(p, a, kGeluErfcPoly[1]);
  p = fmaf(p, a, kGeluErfcPoly[0]);
  const float e = __builtin_amdgcn_exp2f(p * a);   // erfc(|z| / sqrt 2)
  return fmaf(-0.5f * a, e, fmaxf(z, 0.f));
}

// Kernels that use more dynamic LDS than the default limit must be told so once per device (the
// attribute belongs to the kernel on a device).  One flag per device; a race between host threads
// only repeats the call.
struct LdsAttrOnce { bool done[32] = {}; };
inline hipError_t ensure_dynamic_lds(const void* kern, size_t bytes, LdsAttrOnce& once) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool tracked = dev >= 0 && dev < 32;
  if (tracked && once.done[dev]) return hipSuccess;
  e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess && tracked) once.done[dev] = true;
  return e;
}

// A launch holds fewer than 2^32 threads along a dimension of its grid; HIP does not report more, it drops the high bits.
constexpr int64_t kMaxGridThreads = 0xFFFFFFFFll;

enum Epilogue { EPI_BIAS = 0, EPI_BIAS_GELU = 1, EPI_BIAS_RESIDUAL = 2, EPI_LNFOLD = 3, EPI_LNFOLD_GELU = 4 };

// LayerNorm folded into a 16-bit linear (the fusion of Sec. 5.5's comparison system, in algebraic
// form): with mean mu and r = 1/sqrt(var + eps) of an x row,
//   LayerNorm(x) W^T + b = r (x Wf^T - mu c) + bf,   Wf = W gamma,  c = row sums of Wf,  bf = b + W beta.
// EPI_LNFOLD / EPI_LNFOLD_GELU read stats, colsum and bias (fp32); the E-typed bias is unused.
// With EPI_BIAS_RESIDUAL, a non-null `partial` receives, per output row and 128-column segment,
// (sum, sum of squared deviations from the segment mean) of the ROUNDED outputs: the next
// LayerNorm's statistics without another pass over the row.  Null members = feature unused.
constexpr int kStatSeg = 128;  // columns per partial
struct LnFold {
  const float* stats = nullptr;   // [M][2] mu, r
  const float* colsum = nullptr;  // [N]
  const float* bias = nullptr;    // [N]
  float* partial = nullptr;       // [M][N / kStatSeg][2]
};

// ---- launchers (each returns the hipError_t of its launch) --------------------------------
// pack.hip
// Up to kLensArgMax sequence lengths travel by value in the gather kernel's argument block (the
// block is limited to 4 KiB), which then builds cu_seqlens itself: one launch, no copy.
constexpr int kLensArgMax = 896;
struct LensArg { int32_t v[kLensArgMax]; };
hipError_t launch_pack_scan_rows(const void* x_padded, void* x_packed, const int32_t* lengths_host, int32_t* cu,
                                 int32_t* token_idx, int32_t B, int32_t S, int64_t row_bytes, int64_t T,
                                 hipStream_t s);
// cu_seqlens[0..B] from lengths on the host, any B, in launches that carry 896 lengths each in their argument block
hipError_t launch_scan_lengths_host(const int32_t* lengths_host, int32_t* cu_seqlens, int32_t B, hipStream_t s);
hipError_t launch_pack_rows(const void* x_padded, void* x_packed, const int32_t* cu, int32_t* token_idx,
                            int32_t B, int32_t S, int64_t row_bytes, int64_t T, hipStream_t s);
hipError_t launch_unpack_rows(const void* y_packed, void* y_padded, const int32_t* cu, int32_t B, int32_t S,
                              int64_t row_bytes, hipStream_t s);
// layernorm.hip
// dtype: 0 fp32, 1 bf16, 2 fp16 (the values of energon_dtype)
// zero (optional): n_zero words that the launch sets to zero beside its own work
hipError_t launch_layernorm(const void* x, const void* gamma, const void* beta, void* y, int64_t T, int32_t H,
                            float eps, int dtype, hipStream_t s, int32_t* zero = nullptr, int32_t n_zero = 0);
// gemm_f32.hip / gemm_mfma.hip (16-bit element types on the matrix cores)
hipError_t launch_gemm_f32(const float* x, const float* w, const float* bias, const float* res, float* y,
                           int64_t M, int32_t N, int32_t K, int epi, hipStream_t s);
// u = LayerNorm(x) and y = epilogue(u W^T + b) in one launch, for the shapes that gemm_f32_takes_ln says (EPI_BIAS, EPI_BIAS_GELU)
bool gemm_f32_takes_ln(int64_t M, int32_t N, int32_t K);
hipError_t launch_gemm_f32_ln(const float* x, const float* gamma, const float* beta, float eps, float* u, const float* w,
                              const float* bias, float* y, int64_t M, int32_t N, int32_t K, int epi, hipStream_t s);
// true if the launch for this shape can fill LnFold::partial (else the caller takes the statistics itself)
bool gemm_emits_row_partials(int64_t M, int32_t N, int32_t K, bool res_aliases_y);
// scratch (optional, 256-byte aligned): room for fp32 sums where K is cut over workgroups.  What is used of it is
// decided by the shape and its size; gemm_scratch_bytes is what the best plan for a shape would take.
size_t gemm_scratch_bytes(int64_t M, int32_t N, int32_t K);
// the same for the shapes of whole rounds of the persistent 256x256 kernel, 0 for others (and where it would not
// cut tiles along K): room for two pieces of 256x256 fp32 accumulators per workgroup
size_t gemm_sched_scratch_bytes(int64_t M, int32_t N, int32_t K);
// the 256x256 kernel takes the shape in whole rounds of tiles
bool gemm_takes_whole_rounds(int64_t M, int32_t N, int32_t K);
// host-side replay of that kernel's work decomposition for one shape: 0 = every tile and slab covered once
int gemm_sched_selfcheck(int64_t M, int32_t N, int32_t K, int32_t wgs, int32_t can_split, int32_t* pieces_out);
// how a 16-bit linear runs: whose kernel, the output tile of a workgroup, parts or pieces that K is cut into
struct LinearPlan {
  enum Kernel { kFewRows, kWaves, kTiles, kPersistent };   // gemm_skinny, gemm_ksplit, gemm_ring, gemm_mfma_sched
  int32_t kernel, tile_rows, tile_columns, parts;
};
LinearPlan gemm_plan(int64_t M, int32_t N, int32_t K, int epi, bool res_aliases_y, size_t scratch_bytes);
hipError_t launch_gemm_bf16(const bf16_t* x, const bf16_t* w, const bf16_t* bias, const bf16_t* res, bf16_t* y,
                            int64_t M, int32_t N, int32_t K, int epi, hipStream_t s, const LnFold* fold = nullptr,
                            float* scratch = nullptr, size_t scratch_bytes = 0);
hipError_t launch_gemm_f16(const f16_t* x, const f16_t* w, const f16_t* bias, const f16_t* res, f16_t* y,
                           int64_t M, int32_t N, int32_t K, int epi, hipStream_t s, const LnFold* fold = nullptr,
                           float* scratch = nullptr, size_t scratch_bytes = 0);
// gemm_ksplit.hip: small tiles (rows x columns), the wavefronts of a workgroup along K.  Plain epilogues only.
enum class KsplitTile { k32x32, k64x32, k64x64 };
template <typename E>
hipError_t launch_gemm_ksplit(KsplitTile tile, const E* x, const E* w, const E* bias, const E* res, E* y, int64_t M,
                              int32_t N, int32_t K, int epi, hipStream_t s);
// gemm_ring.hip: tiles of rows x columns, per_cu workgroups on a CU; with parts > 1, K cut over that many workgroups, whose
// fp32 sums go through scratch (parts * M * N floats; plain epilogues only)
struct RingShape { int16_t rows, cols, per_cu; };
constexpr RingShape kRingShapes[] = {{64, 64, 2},  {64, 96, 2},   {96, 96, 2},   {96, 128, 1},  {128, 128, 1}, {128, 128, 2},
                                     {96, 192, 1}, {128, 192, 1}, {160, 192, 1}, {128, 256, 1}, {160, 256, 1}};
constexpr int kRingCount = sizeof(kRingShapes) / sizeof(kRingShapes[0]);
template <typename E>
hipError_t launch_gemm_ring(int shape, const E* x, const E* w, const E* bias, const E* res, E* y, int64_t M, int32_t N, int32_t K,
                            int epi, const LnFold& lf, hipStream_t s, int32_t parts = 1, float* scratch = nullptr);
// gemm_skinny.hip: M <= 64 rows (a generation step), bound by streaming W once.  With `partial` (fp32 scratch;
// gemm_skinny_partial_bytes is what the best plan takes) K may be cut over several workgroups.
bool gemm_skinny_takes(int64_t M, int32_t N, int32_t K, int epi);
size_t gemm_skinny_partial_bytes(int64_t M, int32_t N, int32_t K);
LinearPlan gemm_skinny_plan_of(int64_t M, int32_t N, int32_t K, size_t scratch_bytes);
template <typename E>
hipError_t launch_gemm_skinny(const E* x, const E* w, const E* bias, const E* res, E* y, int64_t M, int32_t N,
                              int32_t K, int epi, hipStream_t s, float* partial = nullptr, size_t partial_bytes = 0);
// y = epilogue(sum over kz < KS of partial[kz][M][N] + b), the parts added in the order of kz
template <typename E>
hipError_t launch_partial_reduce(const float* partial, int32_t KS, const E* bias, const E* res, E* y, int64_t M,
                                 int32_t N, int epi, hipStream_t s);
// decode_attention.hip, model_ends.hip (dtype 1 or 2 only).  scratch (optional, fp32): room for the states of keys cut
// over workgroups, decode_attention_scratch_bytes for the most parts; what fits is used.  arrived (with it): B * nh
// counters that are zero when the launch starts
size_t decode_attention_scratch_bytes(int64_t B, int32_t nh, int32_t d);
hipError_t launch_decode_attention(const void* qkv, void* k_cache, void* v_cache, const int32_t* lens, int32_t B,
                                   int32_t S_cap, int32_t nh, int32_t d, int dtype, void* out, hipStream_t s,
                                   float* scratch = nullptr, size_t scratch_bytes = 0, int32_t* arrived = nullptr);
hipError_t launch_embed_packed(const int32_t* ids, const int32_t* cu, const int32_t* positions, int32_t B, int64_t T,
                               const void* wte, int32_t V, const void* wpe, int32_t P, int32_t H, int dtype, void* x,
                               hipStream_t s);
hipError_t launch_cache_fill(const void* qkv, const int32_t* cu, int32_t B, int64_t T, int64_t a_bytes, int32_t S_cap,
                             void* kc, void* vc, hipStream_t s);
hipError_t launch_last_rows(const void* x, const int32_t* cu, int32_t B, int64_t row_bytes, void* out, hipStream_t s);
// ln_fold.hip (dtype 1 or 2 only)
hipError_t launch_fold_weights(const void* w, const void* b, const void* gamma, const void* beta, int32_t N, int32_t K,
                               int dtype, void* wf, float* colsum, float* bias_f, hipStream_t s);
hipError_t launch_row_stats(const void* x, int64_t M, int32_t K, float eps, int dtype, float* stats, hipStream_t s);
hipError_t launch_merge_partials(const float* partial, int64_t M, int32_t P, float eps, float* stats, hipStream_t s);
// attention_f32.hip / attention_mfma.hip
// T: rows of qkv (>= cu[B]; bounds or shapes the launch, the work follows cu)
hipError_t launch_attention_f32(const float* qkv, float* out, const int32_t* cu, int64_t T, int32_t B, int32_t max_len,
                                int32_t nh, int32_t d, hipStream_t s);
hipError_t launch_attention_bf16(const bf16_t* qkv, bf16_t* out, const int32_t* cu, int64_t T, int32_t B,
                                 int32_t max_len, int32_t nh, int32_t d, hipStream_t s);
hipError_t launch_attention_f16(const f16_t* qkv, f16_t* out, const int32_t* cu, int64_t T, int32_t B,
                                int32_t max_len, int32_t nh, int32_t d, hipStream_t s);
hipError_t launch_attention_padded_bf16(const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* out,
                                        const int32_t* cu, int32_t B, int32_t S, int32_t nh, int32_t d, hipStream_t s);
hipError_t launch_attention_padded_f16(const f16_t* q, const f16_t* k, const f16_t* v, f16_t* out,
                                       const int32_t* cu, int32_t B, int32_t S, int32_t nh, int32_t d, hipStream_t s);
// drce.hip (head_bytes = bytes of one head's slice of a row: d * element size)
hipError_t launch_rebuild_qkv(const void* qkv, void* q, void* k, void* v, const int32_t* cu, int32_t B, int32_t S,
                              int32_t nh, int32_t head_bytes, hipStream_t s);
hipError_t launch_remove_padding_heads(const void* o, void* out, const int32_t* cu, int32_t B, int32_t S, int32_t nh,
                                       int32_t head_bytes, hipStream_t s);

}  // namespace energon
