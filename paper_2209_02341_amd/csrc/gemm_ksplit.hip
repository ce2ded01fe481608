// 16-bit linear layer  y[M,N] = epilogue(x[M,K] W[N,K]^T + b)  for problems of a few dozen to a few hundred rows whose
// tiles do not fill the chip: every wavefront of a workgroup computes the whole output tile over its own part
// of K, and the partial sums meet in LDS, added in a fixed order (deterministic, no scratch in memory).
//  * wavefront w takes slabs of 64 k (128 bytes of a row) w, w + WK, ...; a slab of W rows and x rows goes from global
//    memory straight into an LDS ring that is private to the wavefront (global_load_lds_dwordx4, whole lines): no
//    barrier in the loop, WK chains of loads per tile instead of one.  What bounds such a problem is the
//    latency of that chain and the idle CUs: 387 x 1024 x 4096, 112 tiles of 64 x 64 with 64 slabs one behind the
//    other, took 36 us (20 us with three slabs in flight); 64 x 32 tiles over four wavefronts 10.6.  More wavefronts
//    or more slabs in flight (8; 3 or 4) changed nothing or lost;
//  * v_mfma_f32_16x16x32, W rows as A operand and x rows as B operand: a lane ends up with four consecutive columns
//    of a row, which leave as vectors of whole row segments after the sum.
#include "common.h"

namespace energon {

namespace {

typedef __attribute__((address_space(1))) const void* kp_gptr_t;
typedef __attribute__((address_space(3))) void* kp_lptr_t;

// TN x TM tiles of 16 x 16 (columns x rows of y) per workgroup, WK wavefronts along K, kDepth slabs in flight each.
template <typename E, int TM, int TN, int WK, int kDepth>
__global__ __launch_bounds__(WK * 64) void gemm_ksplit_kernel(const E* __restrict__ x, const E* __restrict__ w,
                                                             const E* __restrict__ bias, const E* res, E* y, int64_t M,
                                                             int32_t N, int32_t K, int epi, int32_t tiles_m,
                                                             int32_t tiles_n) {
  using Cfg = WaveRings<TM, TN, WK, kDepth>;
  constexpr int G = 2 * (TM + TN);   // 1 KiB loads (8 rows x 128 bytes) per slab
  extern __shared__ uint4 lds[];
  int64_t m0;
  int32_t n0;
  if (!tile_origin<16 * TM, 16 * TN>(tiles_m, tiles_n, m0, n0)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane & 15, lq = lane >> 4;
  const int32_t ns = (K / 64 - wave + WK - 1) / WK;   // slabs of this wavefront
  uint4* const ring = lds + wave * (kDepth * Cfg::kSlotVecs);

  // Lane l of a load lands in slot l % 8 of row l / 8 of its 8-row group and fetches the chunk that the swizzle
  // keeps there; rows past the edge read the last row and are dropped.  A wavefront-uniform base (the tile's
  // first row, the slab) plus 32-bit offsets: 64 rows x K x 2 bytes, K < 2^24.
  uint32_t ow[2 * TN], ox[2 * TM];
#pragma unroll
  for (int g = 0; g < 2 * TN; ++g) {
    const int row = 8 * g + (lane >> 3);
    ow[g] = ((uint32_t)min(row, N - 1 - n0) * (uint32_t)K + (uint32_t)((lane & 7) ^ swz16(row & 15)) * 8u) * 2u;
  }
  const int64_t lim = M - 1 - m0;
#pragma unroll
  for (int g = 0; g < 2 * TM; ++g) {
    const int row = 8 * g + (lane >> 3);
    ox[g] = ((uint32_t)(row < lim ? row : lim) * (uint32_t)K + (uint32_t)((lane & 7) ^ swz16(row & 15)) * 8u) * 2u;
  }
  const char* const wbase = reinterpret_cast<const char*>(w + (size_t)n0 * K);
  const char* const xbase = reinterpret_cast<const char*>(x + (size_t)m0 * K);
  auto issue = [&](int32_t slot, int32_t i) {
    const size_t k = (size_t)(wave + i * WK) * 128;
    uint4* dst = ring + slot * Cfg::kSlotVecs;
#pragma unroll
    for (int g = 0; g < 2 * TN; ++g)
      __builtin_amdgcn_global_load_lds((kp_gptr_t)(wbase + k + ow[g]), (kp_lptr_t)(dst + g * 64), 16, 0, 0);
#pragma unroll
    for (int g = 0; g < 2 * TM; ++g)
      __builtin_amdgcn_global_load_lds((kp_gptr_t)(xbase + k + ox[g]), (kp_lptr_t)(dst + (2 * TN + g) * 64), 16, 0, 0);
  };

  f32x4 acc[TN][TM];
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  uint32_t foff[2];   // operand reads: row l % 16 of a 16-row tile, chunk 4 ks + l / 16
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) foff[ks] = (uint32_t)(lrow * 8 + ((4 * ks + lq) ^ swz16(lrow)));

  for (int32_t u = 0; u < kDepth && u < ns; ++u) issue(u, u);
  int32_t slot = 0;
  for (int32_t i = 0; i < ns; ++i) {
    // loads return in order; behind slab i's are those of the next kDepth - 1 slabs while they all exist
    if (i + kDepth <= ns) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kDepth - 1) * G) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const uint4* slab = ring + slot * Cfg::kSlotVecs;
    vec8<E> wb[2][TN], xa[2][TM];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int t = 0; t < TN; ++t) wb[ks][t] = *reinterpret_cast<const vec8<E>*>(&slab[t * 128 + foff[ks]]);
#pragma unroll
      for (int t = 0; t < TM; ++t) xa[ks][t] = *reinterpret_cast<const vec8<E>*>(&slab[(TN + t) * 128 + foff[ks]]);
    }
    if (i + kDepth < ns) {
      // the slot is refilled by the load unit, which is not ordered with this wavefront's LDS reads
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      issue(slot, i + kDepth);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) acc[a][b] = Mfma<E>::m16x16x32(wb[ks][a], xa[ks][b], acc[a][b]);
    slot = slot + 1 == kDepth ? 0 : slot + 1;
  }

  // the rings are free once every wavefront is here (each has waited for its own last load)
  __syncthreads();
  f32x4* const red = reinterpret_cast<f32x4*>(lds);
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) red[(wave * TN * TM + a * TM + b) * 64 + lane] = acc[a][b];
  __syncthreads();
  constexpr int kQuads = 4 * TN;   // groups of 4 columns per row of the tile: neighbouring threads, one row segment
#pragma unroll
  for (int i = tid; i < 16 * TM * kQuads; i += WK * 64) {
    const int r = i / kQuads, q = i % kQuads;
    const int64_t m = m0 + r;
    const int32_t n = n0 + 4 * q;
    if (m >= M || n >= N) continue;   // N % 8 == 0
    const int at = ((q >> 2) * TM + (r >> 4)) * 64 + (q & 3) * 16 + (r & 15);
    f32x4 v = red[at];
#pragma unroll
    for (int k = 1; k < WK; ++k) v += red[k * TN * TM * 64 + at];
    const size_t off = (size_t)m * N + n;
    if (bias != nullptr) {
      const vec4<E> b4 = *reinterpret_cast<const vec4<E>*>(bias + n);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += static_cast<float>(b4[e]);
    }
    if (epi == EPI_BIAS_GELU) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = gelu_erf(v[e]);
    }
    if (epi == EPI_BIAS_RESIDUAL) {
      const vec4<E> r4 = *reinterpret_cast<const vec4<E>*>(res + off);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += static_cast<float>(r4[e]);
    }
    vec4<E> o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = static_cast<E>(v[e]);
    *reinterpret_cast<vec4<E>*>(y + off) = o;
  }
}

template <typename E, int TM, int TN, int WK, int kDepth>
hipError_t launch_cfg(const E* x, const E* w, const E* bias, const E* res, E* y, int64_t M, int32_t N, int32_t K,
                      int epi, hipStream_t s) {
  constexpr int BM = 16 * TM, BN = 16 * TN;
  constexpr size_t lds = WaveRings<TM, TN, WK, kDepth>::kLds;
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  auto kern = gemm_ksplit_kernel<E, TM, TN, WK, kDepth>;
  static LdsAttrOnce once;
  const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds, once);
  if (e != hipSuccess) return e;
  const int32_t tiles_m = (int32_t)((M + BM - 1) / BM), tiles_n = (N + BN - 1) / BN;
  const int64_t grid = ((int64_t)tiles_m * tiles_n + kXcds - 1) / kXcds * kXcds;
  kern<<<dim3((unsigned)grid), dim3(WK * 64), lds, s>>>(x, w, bias, res, y, M, N, K, epi, tiles_m, tiles_n);
  return hipGetLastError();
}

}  // namespace

template <typename E>
hipError_t launch_gemm_ksplit(KsplitTile tile, const E* x, const E* w, const E* bias, const E* res, E* y, int64_t M,
                              int32_t N, int32_t K, int epi, hipStream_t s) {
  switch (tile) {
    case KsplitTile::k32x32: return launch_cfg<E, 2, 2, 4, 2>(x, w, bias, res, y, M, N, K, epi, s);
    case KsplitTile::k64x32: return launch_cfg<E, 4, 2, 4, 2>(x, w, bias, res, y, M, N, K, epi, s);
    case KsplitTile::k64x64: return launch_cfg<E, 4, 4, 4, 2>(x, w, bias, res, y, M, N, K, epi, s);
  }
  return hipErrorInvalidValue;
}
template hipError_t launch_gemm_ksplit<bf16_t>(KsplitTile, const bf16_t*, const bf16_t*, const bf16_t*, const bf16_t*,
                                               bf16_t*, int64_t, int32_t, int32_t, int, hipStream_t);
template hipError_t launch_gemm_ksplit<f16_t>(KsplitTile, const f16_t*, const f16_t*, const f16_t*, const f16_t*, f16_t*,
                                              int64_t, int32_t, int32_t, int, hipStream_t);

}  // namespace energon
