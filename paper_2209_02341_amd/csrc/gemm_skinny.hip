// 16-bit linear layer for few rows (M <= 64): y[M,N] = epilogue(x[M,K] W[N,K]^T + b).
// This is the shape of a generation step, one token per sequence: every weight is used M times
// only, so the contraction is bound by streaming W from HBM once (N*K*e bytes), not by the
// matrix cores.  Design for gfx950:
//  * a workgroup owns 16, 32, 64 or 80 output columns (rows of W) and all of K, or 1/KS of it; its 4
//    wavefronts split that in interleaved slabs of 64 (wavefront w takes slabs w, w + 4, ...) and
//    add their partial sums through LDS at the end, in a fixed order.  With K cut over KS
//    workgroups (only where the caller provides room for KS fp32 partial results) a second small
//    kernel adds the parts in a fixed order and applies the epilogue.  Deterministic, no atomics;
//  * a slab of W (16 to 80 rows x 128 bytes) and the same slab of x (16 MT rows x 128 bytes) go
//    from global memory straight to LDS (global_load_lds_dwordx4, whole 128-byte lines) into a
//    ring that is private to the wavefront, 2 to 4 slabs deep (the depth made no measurable
//    difference): no barrier and no staging register in the streaming loop.  x is read again by every workgroup, from the L2; fetched as whole lines it
//    costs the W stream 20 % (measured in a probe: 24.7 -> 29.6 us for a 157 MB matrix), as 64-byte
//    operand gathers into registers 60 %.  The XOR swizzle of the 256x256 kernel keeps the operand
//    reads free of bank conflicts;
//  * v_mfma_f32_16x16x32: x rows are the A operand (row tiles of 16, MT of them), W rows the B
//    operand; at these sizes the matrix cores are idle most of the time by design.
#include "common.h"
#include <algorithm>

namespace energon {

namespace {

typedef __attribute__((address_space(1))) const void* sk_gptr_t;
typedef __attribute__((address_space(3))) void* sk_lptr_t;

constexpr int kSkWaves = 4;     // a workgroup's share of K is split over this many wavefronts

// MT row tiles of x (16 rows each), NT row tiles of W (= 16 NT output columns per workgroup)
template <int MT, int NT, int D> struct SkCfg {
  static constexpr int kBN = 16 * NT;
  static constexpr int kSlotVecs = (16 * NT + 16 * MT) * 8;      // uint4 per ring slot: W rows, then x rows
  static constexpr int kDepth = D;                               // slabs in flight per wavefront
  static constexpr int kRedLd = kBN + 4;                         // floats per row of the reduction buffer:
                                                                 // rows 4 apart land 16 banks apart
  static constexpr size_t kRing = (size_t)kSkWaves * kDepth * kSlotVecs * 16;
  static constexpr size_t kRed = (size_t)kSkWaves * MT * 16 * kRedLd * sizeof(float);
  static constexpr size_t kLds = kRing > kRed ? kRing : kRed;
};

// grid = (ceil(N / BN), KS).  Workgroup (nb, kz) contracts slabs [kz * KT / KS, (kz + 1) * KT / KS) of K for
// columns 16 NT nb ..; with partial == nullptr (KS = 1) it applies the epilogue and writes y, otherwise
// it writes its fp32 sums to partial[kz][M][N] and skinny_reduce_kernel finishes the job.  RAGGED: the last block has
// fewer columns than BN (N % 8 == 0); an instance of its own, because the address of every load would pay for it.
template <typename E, int MT, int NT, int kD, bool RAGGED>
__global__ __launch_bounds__(kSkWaves * 64) void gemm_skinny_kernel(const E* __restrict__ x, const E* __restrict__ w,
                                                                   const E* __restrict__ bias, const E* res, E* y,
                                                                   float* __restrict__ partial, int32_t M, int32_t N,
                                                                   int32_t K, int epi) {
  static_assert(MT == 1 || MT == 2 || MT == 4, "row tiles of x");
  using Cfg = SkCfg<MT, NT, kD>;
  constexpr int D = Cfg::kDepth, SV = Cfg::kSlotVecs, BN = Cfg::kBN, RLD = Cfg::kRedLd;
  constexpr int GW = 2 * NT, GX = 2 * MT;   // 8-row groups of W and x per slab
  constexpr int G = GW + GX;                // direct-to-LDS instructions per slab
  extern __shared__ uint4 lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t n0 = blockIdx.x * BN;
  const int32_t KTs = K / 64 / (int32_t)gridDim.y;            // slabs of this workgroup
  const int32_t s0 = (int32_t)blockIdx.y * KTs;               // its first slab
  const int32_t ns = (KTs - wave + kSkWaves - 1) / kSkWaves;  // slabs of this wavefront (>= 0)

  uint4* ring = lds + wave * (D * SV);
  const int lrow = lane & 15, lq = lane >> 4;

  // A row group = 8 rows x 128 bytes in lane order, lane l landing in slot l % 8 of row l / 8 and
  // fetching the chunk the swizzle puts there (even groups are rows 0..7 of a 16-row tile, odd
  // groups rows 8..15).  Addresses are a wavefront-uniform base (first row of the group, this
  // workgroup's first slab) plus a 32-bit per-lane offset, so that advancing along K is scalar
  // arithmetic.  x rows are clamped to M - 1: rows past M are computed and dropped.
  const uint32_t row_b = (uint32_t)K * (uint32_t)sizeof(E);
  const uint32_t ch_even = (uint32_t)(((lane & 7) ^ swz16(lane >> 3)) * 16);
  const uint32_t ch_odd = (uint32_t)(((lane & 7) ^ swz16((lane >> 3) | 8)) * 16);
  const uint32_t woff_even = (uint32_t)(lane >> 3) * row_b + ch_even, woff_odd = (uint32_t)(lane >> 3) * row_b + ch_odd;
  const char* wbase = reinterpret_cast<const char*>(w + (size_t)n0 * K) + (size_t)s0 * 128;   // uniform
  const int32_t groups = (N - n0 + 7) >> 3;   // 8-row groups of W that exist; those past the end repeat the last
  const char* xbase = reinterpret_cast<const char*>(x) + (size_t)s0 * 128;                    // uniform
  uint32_t xoff[GX];
#pragma unroll
  for (int j = 0; j < GX; ++j) xoff[j] = (uint32_t)min(8 * j + (lane >> 3), M - 1) * row_b + ((j & 1) ? ch_odd : ch_even);
  // operand reads from a ring slot: row l % 16 of a 16-row tile, chunk (4 ks + l / 16) ^ swizzle
  uint32_t foff[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) foff[ks] = (uint32_t)(lrow * 8 + ((ks * 4 + lq) ^ swz16(lrow)));

  f32x4 acc[MT][NT];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // slab i of this wavefront -> ring slot i % D
  auto issue = [&](int32_t slot, int32_t i) {
    const size_t kb = (size_t)(wave + i * kSkWaves) * 128;
    uint4* dst = ring + slot * SV;
#pragma unroll
    for (int j = 0; j < GW; ++j)
      __builtin_amdgcn_global_load_lds((sk_gptr_t)(wbase + (size_t)(8 * (RAGGED ? min(j, groups - 1) : j)) * row_b + kb +
                                                   ((j & 1) ? woff_odd : woff_even)),
                                       (sk_lptr_t)(dst + j * 64), 16, 0, 0);
#pragma unroll
    for (int j = 0; j < GX; ++j)
      __builtin_amdgcn_global_load_lds((sk_gptr_t)(xbase + kb + xoff[j]), (sk_lptr_t)(dst + (GW + j) * 64), 16, 0, 0);
  };

  for (int32_t u = 0; u < D && u < ns; ++u) issue(u, u);
  int32_t slot = 0;
  for (int32_t i = 0; i < ns; ++i) {
    // Loads return in order.  Behind slab i's loads are those of the next D - 1 slabs while they
    // all exist; on the last D - 1 trips fewer are outstanding and the wait is for everything.
    if (i + D <= ns) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * G) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const uint4* slab = ring + slot * SV;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      vec8<E> wb[NT], xa[MT];
#pragma unroll
      for (int j = 0; j < NT; ++j) wb[j] = *reinterpret_cast<const vec8<E>*>(&slab[j * 128 + foff[ks]]);
#pragma unroll
      for (int t = 0; t < MT; ++t) xa[t] = *reinterpret_cast<const vec8<E>*>(&slab[(NT + t) * 128 + foff[ks]]);
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[t][j] = Mfma<E>::m16x16x32(xa[t], wb[j], acc[t][j]);
    }
    if (i + D < ns) {
      // the slot is refilled by the load unit, which is not ordered with this wavefront's LDS
      // reads: they must have returned first
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      issue(slot, i + D);
    }
    slot = slot + 1 == D ? 0 : slot + 1;
  }

  // Sum over the wavefronts through LDS (the rings are free once every wavefront is here; each
  // has waited for its own last load), then the epilogue: thread -> row, 4 columns.
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();
  float* red = reinterpret_cast<float*>(lds);
  constexpr int kRedWave = MT * 16 * RLD;
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        red[wave * kRedWave + (16 * t + 4 * lq + e) * RLD + 16 * j + lrow] = acc[t][j][e];
  __syncthreads();
  constexpr int TPR = BN / 4;   // threads per output row
  constexpr int RPT = kSkWaves * 64 / TPR;   // rows at a time; the threads left over (80 columns) have none
  const int32_t c4 = (tid % TPR) * 4;
  if (tid / TPR >= RPT || (RAGGED && n0 + c4 >= N)) return;
  for (int32_t m = tid / TPR; m < MT * 16 && m < M; m += RPT) {
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int wv = 0; wv < kSkWaves; ++wv) {
      const float4 p = *reinterpret_cast<const float4*>(&red[wv * kRedWave + m * RLD + c4]);
      v[0] += p.x; v[1] += p.y; v[2] += p.z; v[3] += p.w;
    }
    const size_t off = (size_t)m * N + n0 + c4;
    if (partial != nullptr) {
      *reinterpret_cast<float4*>(partial + (size_t)blockIdx.y * M * N + off) = make_float4(v[0], v[1], v[2], v[3]);
      continue;
    }
    if (bias != nullptr) {
      const vec4<E> b4 = *reinterpret_cast<const vec4<E>*>(bias + n0 + c4);
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] += static_cast<float>(b4[q]);
    }
    if (epi == EPI_BIAS_GELU) {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = gelu_erf(v[q]);
    }
    if (epi == EPI_BIAS_RESIDUAL) {
      const vec4<E> r4 = *reinterpret_cast<const vec4<E>*>(res + off);
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] += static_cast<float>(r4[q]);
    }
    vec4<E> o;
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = static_cast<E>(v[q]);
    *reinterpret_cast<vec4<E>*>(y + off) = o;
  }
}

// y = epilogue(sum over kz of partial[kz] + b): the partial sums are added in the order of kz.  A few hundred
// kilobytes: what it takes is its launch and one memory latency, so bias, residual and the parts (four at a time) are
// all requested before the first is used.
template <typename E>
__global__ __launch_bounds__(256) void skinny_reduce_kernel(const float* __restrict__ partial, int32_t KS,
                                                            const E* __restrict__ bias, const E* res, E* y, int32_t M,
                                                            int32_t N, int epi) {
  const size_t i4 = (size_t)blockIdx.x * 256 + threadIdx.x;   // group of 4 columns
  const size_t total4 = (size_t)M * N / 4;
  if (i4 >= total4) return;
  const size_t off = i4 * 4, stride = (size_t)M * N;
  const int32_t n = (int32_t)(off % N);
  vec4<E> b4, r4;
#pragma unroll
  for (int q = 0; q < 4; ++q) b4[q] = r4[q] = static_cast<E>(0.f);
  if (bias != nullptr) b4 = *reinterpret_cast<const vec4<E>*>(bias + n);
  if (epi == EPI_BIAS_RESIDUAL) r4 = *reinterpret_cast<const vec4<E>*>(res + off);
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  for (int32_t k0 = 0; k0 < KS; k0 += 4) {
    float4 p[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) p[k] = *reinterpret_cast<const float4*>(partial + (size_t)min(k0 + k, KS - 1) * stride + off);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (k0 + k < KS) { v[0] += p[k].x; v[1] += p[k].y; v[2] += p[k].z; v[3] += p[k].w; }
  }
  vec4<E> o;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float t = v[q];
    if (bias != nullptr) t += static_cast<float>(b4[q]);
    if (epi == EPI_BIAS_GELU) t = gelu_erf(t);
    if (epi == EPI_BIAS_RESIDUAL) t += static_cast<float>(r4[q]);
    o[q] = static_cast<E>(t);
  }
  *reinterpret_cast<vec4<E>*>(y + off) = o;
}

template <typename E, int MT, int NT, int kD>
hipError_t launch_sk(const E* x, const E* w, const E* bias, const E* res, E* y, float* partial, int32_t KS, int32_t M,
                     int32_t N, int32_t K, int epi, hipStream_t s) {
  constexpr size_t lds = SkCfg<MT, NT, kD>::kLds;
  const bool ragged = N % (16 * NT) != 0;
  const auto kern = ragged ? gemm_skinny_kernel<E, MT, NT, kD, true> : gemm_skinny_kernel<E, MT, NT, kD, false>;
  static LdsAttrOnce once[2];
  {
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds, once[ragged]);
    if (e != hipSuccess) return e;
  }
  kern<<<dim3((unsigned)((N + 16 * NT - 1) / (16 * NT)), (unsigned)KS), dim3(kSkWaves * 64), lds, s>>>(x, w, bias, res, y,
                                                                                                     partial, M, N, K, epi);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || partial == nullptr) return e;
  return launch_partial_reduce<E>(partial, KS, bias, res, y, M, N, epi, s);
}

template <typename E, int NT, int D1, int D2, int D4>
hipError_t launch_nt(const E* x, const E* w, const E* bias, const E* res, E* y, float* partial, int32_t KS, int32_t M,
                     int32_t N, int32_t K, int epi, hipStream_t s) {
  if (M <= 16) return launch_sk<E, 1, NT, D1>(x, w, bias, res, y, partial, KS, M, N, K, epi, s);
  if (M <= 32) return launch_sk<E, 2, NT, D2>(x, w, bias, res, y, partial, KS, M, N, K, epi, s);
  return launch_sk<E, 4, NT, D4>(x, w, bias, res, y, partial, KS, M, N, K, epi, s);
}

}  // namespace

template <typename E>
hipError_t launch_partial_reduce(const float* partial, int32_t KS, const E* bias, const E* res, E* y, int64_t M,
                                 int32_t N, int epi, hipStream_t s) {
  const size_t total4 = (size_t)M * N / 4;   // N % 4 == 0 for every caller (N % 8 == 0 is an ABI rule)
  if (total4 == 0) return hipSuccess;
  skinny_reduce_kernel<E><<<dim3((unsigned)((total4 + 255) / 256)), dim3(256), 0, s>>>(partial, KS, bias, res, y,
                                                                                       (int32_t)M, N, epi);
  return hipGetLastError();
}
template hipError_t launch_partial_reduce<bf16_t>(const float*, int32_t, const bf16_t*, const bf16_t*, bf16_t*, int64_t,
                                                  int32_t, int, hipStream_t);
template hipError_t launch_partial_reduce<f16_t>(const float*, int32_t, const f16_t*, const f16_t*, f16_t*, int64_t,
                                                 int32_t, int, hipStream_t);

bool gemm_skinny_takes(int64_t M, int32_t N, int32_t K, int epi) {
  return M >= 1 && M <= 64 && N % 8 == 0 && K % 64 == 0 && epi >= EPI_BIAS && epi <= EPI_BIAS_RESIDUAL;
}

// Columns per workgroup (16 nt) and parts of K (ks, their sums in at most `cap` bytes of scratch): the least expected
// time, which is the longer of W from HBM (5.8 TB/s) and the busiest CU's share of W and x (40 KB/us with all CUs at work, up
// to 65 with fewer and narrow blocks); cutting K costs 4 us for the second kernel.  Wide blocks read x less often (a
// hundredth of the bytes read decides a tie).  Two cases lie outside that model:
//  * K of less than about 1800, where the latency of a workgroup's few slabs counts: 16 columns as long as each CU gets
//    one such block (us, 32 columns / 16: 64 x 3072 x 768 4.6 / 3.9, 16 x 4096 x 1024 3.7 / 3.4);
//  * 17 to 32 rows and 512 or more blocks of 32 columns, of which two share a CU, so that one's first loads and sums hide
//    behind the other: 32 columns up to K = 3072 (us, 64 or 80 columns / 32: 32 x 50304 x 1024 23.6 / 18.6, 32 x 32000 x
//    3072 32.0 / 30.0).  Not where K is a multiple of 2048, whose rows meet in the same memory channels (32 x 32000 x 2048
//    23.3 / 27.9);
//  * 80 columns not up to K = 3072 where 64 still are one block per CU: the longer prologue and epilogue are not repaid (us,
//    80 / 64 columns: 16 x 16384 x 768 5.5 / 4.2, 16 x 12288 x 1536 8.0 / 7.3; at K = 4096 16 x 16384 21.7 / 22.1).
// Measured (us, weights from HBM, M = 2 / 32 / 64; before: 32 or 64 columns, 8 parts or none):
//   5120 x 20480  48 -> 39 / 50 -> 41 / 66 -> 45     20480 x 5120  40 -> 37 / 48 -> 39 / -
//   5120 x 5120   12.3 -> 12.3 / 17.6 -> 16.2 / 22.5 -> 18.5     15360 x 5120 29 / 31 / 36 (80 columns at M = 2, else 64 as before)
struct SkinnyPlan { int32_t nt, ks; size_t scratch; };
static SkinnyPlan gemm_skinny_plan(int64_t M, int32_t N, int32_t K, size_t cap) {
  const int32_t KT = K / 64, mt = M <= 16 ? 1 : M <= 32 ? 2 : 4;
  if (mt == 2 && (N + 31) / 32 >= 512 && K <= 3072 && K % 2048 != 0) return {2, 1, 0};
  const float hbm_us = (float)N * (float)K * (2.0f / 5.8e6f);
  SkinnyPlan best{1, 1, 0};
  float best_us = 1e30f;
  for (const int32_t nt : {5, 4, 2, 1}) {
    const int32_t blocks = (N + 16 * nt - 1) / (16 * nt);
    const float slab_kb = 2.048f * (float)(nt + mt);   // of one workgroup
    for (const int32_t ks : {1, 2, 4, 5, 8}) {
      const int32_t wgs = blocks * ks;
      if (ks > 1 && (wgs > 512 || KT % ks != 0 || KT / ks < 4)) continue;
      if (nt == 5 && ks == 1 && KT <= 48 && N <= 256 * 64) continue;
      const size_t scratch = ks > 1 ? (size_t)ks * (size_t)M * N * sizeof(float) : 0;
      if (scratch > cap) continue;
      const bool latency = nt == 1 && ks == 1 && blocks <= 256 && KT <= 28;
      const float rate = latency ? 60.0f : std::min(nt >= 4 ? 42.0f : 65.0f, std::max(40.0f, 7680.0f / (float)wgs));   // KB/us of one CU
      const float cu_us = (float)((wgs + 255) >> 8) * (float)(KT / ks) * slab_kb / rate;
      const float us = (ks > 1 ? 4.0f : 0.0f) + std::max(hbm_us, cu_us) + (float)blocks * (float)KT * slab_kb * 1.0e-5f;
      if (us < best_us) { best_us = us; best = {nt, ks, scratch}; }
    }
  }
  return best;
}

LinearPlan gemm_skinny_plan_of(int64_t M, int32_t N, int32_t K, size_t scratch_bytes) {
  const SkinnyPlan p = gemm_skinny_plan(M, N, K, scratch_bytes);
  return {LinearPlan::kFewRows, M <= 16 ? 16 : M <= 32 ? 32 : 64, 16 * p.nt, p.ks};
}

size_t gemm_skinny_partial_bytes(int64_t M, int32_t N, int32_t K) { return gemm_skinny_plan(M, N, K, SIZE_MAX).scratch; }

template <typename E>
hipError_t launch_gemm_skinny(const E* x, const E* w, const E* bias, const E* res, E* y, int64_t M, int32_t N,
                              int32_t K, int epi, hipStream_t s, float* partial, size_t partial_bytes) {
  if (!gemm_skinny_takes(M, N, K, epi)) return hipErrorInvalidValue;
  const SkinnyPlan plan = gemm_skinny_plan(M, N, K, partial != nullptr ? partial_bytes : 0);
  float* const p = plan.ks > 1 ? partial : nullptr;
  switch (plan.nt) {   // slabs in flight per wavefront for up to 16, 32, 64 rows: what fits beside another workgroup
    case 5: return launch_nt<E, 5, 2, 2, 2>(x, w, bias, res, y, p, plan.ks, (int32_t)M, N, K, epi, s);
    case 4: return launch_nt<E, 4, 2, 2, 2>(x, w, bias, res, y, p, plan.ks, (int32_t)M, N, K, epi, s);
    case 2: return launch_nt<E, 2, 4, 2, 2>(x, w, bias, res, y, p, plan.ks, (int32_t)M, N, K, epi, s);
    default: return launch_nt<E, 1, 4, 4, 3>(x, w, bias, res, y, p, plan.ks, (int32_t)M, N, K, epi, s);
  }
}

template hipError_t launch_gemm_skinny<bf16_t>(const bf16_t*, const bf16_t*, const bf16_t*, const bf16_t*, bf16_t*,
                                               int64_t, int32_t, int32_t, int, hipStream_t, float*, size_t);
template hipError_t launch_gemm_skinny<f16_t>(const f16_t*, const f16_t*, const f16_t*, const f16_t*, f16_t*, int64_t,
                                              int32_t, int32_t, int, hipStream_t, float*, size_t);

}  // namespace energon
