// fp32 linear layer  y = epilogue(x W^T + b)  on packed rows (paper Sec. 4.3: the linear
// layers see only valid tokens): the fp32 storage path, on the fp32 matrix instructions
// (v_mfma_f32_16x16x4_f32: fp32 products and sums, 157 TFLOP/s).
//
// These problems are small: what bounds them is latency, idle CUs and, from a few hundred rows on, bytes
// moved from the L2 per flop, not the matrix cores.  So:
//  * a workgroup owns a tile of 16, 32 or 64 rows and columns and all of K, which its 4 or 8 wavefronts cut
//    in interleaved slabs of 32 (128 bytes of a row); the partial sums meet in LDS at the end and are added
//    in a fixed order.  Every wavefront computes the whole tile, so a tile costs (rows + columns) * K * 4
//    bytes however many wavefronts share it;
//  * a slab of W rows and x rows goes from global memory straight into an LDS ring that is private to the
//    wavefront, two slabs deep (global_load_lds_dwordx4, whole 128-byte lines): no barrier and no
//    staging register in the loop.  (Operands loaded straight into the MFMA layout, 16 rows x 64 bytes per
//    instruction, ran at 14 bytes per clock and CU, a quarter of this: 387 x 3072 x 1024 44 -> 31 us.)
//  * an MFMA operand is one float per lane, row l % 16 and k = l / 16; since k may be walked in any order
//    that both operands share, a lane reads four consecutive floats, chunk l / 16 of the half slab, as one
//    16-byte LDS vector for four instructions, with the conflict-free swizzle of the 16-bit kernels;
//  * W rows are the A operand and x rows the B operand: a lane ends up with four consecutive columns of one
//    output row, so bias, residual and result move as 16-byte vectors.
// Against the former kernel (vector ALU, 64 x 64 LDS tile, 4 x 4 registers per lane): 387 x 4096 x 1024
// 214 -> 41 us, 387 x 1024 x 4096 596 -> 40 us, 76 x 256 x 1024 149 -> 4.1 us; 2048 x 2048 x 8192 runs at
// 125 TFLOP/s.
// The bf16 instructions on operands cut into three bf16 parts (Henry, Tang and Heinecke 2019) give no more than this: six products of
// parts run at 137 TFLOP/s (2048 x 6400 x 1600: 306 us against 398 here) but lose up to 2^-21 of a product, and bits of operands below
// 2^-110; all nine, with those operands found and a second pass for them, take 411 us.
#include "common.h"
#include <cmath>
#include <type_traits>

namespace energon {

namespace {

typedef __attribute__((address_space(1))) const void* f32_gptr_t;
typedef __attribute__((address_space(3))) void* f32_lptr_t;

// LayerNorm of the x rows on their way into a linear: gain, offset, and where the normalised rows go as well
struct LnRows {
  const float *gamma, *beta;
  float eps;
  float* u;
};
constexpr int kLnMaxK = 512;   // of a row: a wavefront holds it in registers, gain and offset lie in LDS

// wave_sum without LDS: halves and rows of 16 lanes are swapped (both operands the same: one result holds the one half, the other the
// other), and in a row a rotation by 8, 4, 2, 1 meets the same lane as the exclusive or, the values having that period by then:
// the same bits.
__device__ __forceinline__ float wave_sum_dpp(float v) {
  const auto both = [](auto p) { return __uint_as_float(p[0]) + __uint_as_float(p[1]); };
  v = both(__builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  v = both(__builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xf, 0xf, true));   // row_ror:8
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x124, 0xf, 0xf, true));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x122, 0xf, 0xf, true));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x121, 0xf, 0xf, true));
  return v;
}

// Rows m0 .. m0 + 15 of x normalised as layernorm_kernel does it (two passes over a row in registers), R of them per wavefront.
// What it reads is requested first, ahead of the slabs, without a branch, and the reductions of the R rows run side by side: one row
// after the other with its stores behind it, and that behind the loads of gain and offset, the linears of 77 x 768 x 256 and 77 x 1024 x
// 256 took 6.8 and 7.4 us, which is what a LayerNorm launch and the plain linear take; now 5.2 and 6.1.
template <int WK>
struct LnTile {
  static constexpr int V = kLnMaxK / 256, R = 16 / WK;
  static_assert(kLnMaxK / 4 <= WK * 64, "gain and offset: a vector per lane");
  f32x4 v[R][V], g, b;
  __device__ __forceinline__ void request(const float* __restrict__ x, const LnRows& ln, int64_t m0, int64_t M, int32_t K, int wave, int lane) {
    const int32_t vecs = K / 4, c = wave * 64 + lane;   // K % 4 == 0
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int64_t m = m0 + wave * R + r;
      const f32x4* row = reinterpret_cast<const f32x4*>(x + (size_t)(m < M ? m : M - 1) * K);
#pragma unroll
      for (int i = 0; i < V; ++i) v[r][i] = row[min(lane + 64 * i, vecs - 1)];   // past the end: left out of the sums
    }
    g = reinterpret_cast<const f32x4*>(ln.gamma)[min(c, vecs - 1)];
    b = reinterpret_cast<const f32x4*>(ln.beta)[min(c, vecs - 1)];
  }
  // mean and 1 / deviation to st, gain and offset to gb; with `write` the normalised rows to ln.u
  __device__ __forceinline__ void finish(const LnRows& ln, int64_t m0, int64_t M, int32_t K, bool write, int wave, int lane, float2* st, f32x4* gb) {
    const int32_t vecs = K / 4, cw = wave * 64 + lane;
    const float inv = 1.0f / (float)K;
    float mean[R], rstd[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      mean[r] = 0.f;
#pragma unroll
      for (int i = 0; i < V; ++i) mean[r] += lane + 64 * i < vecs ? (v[r][i][0] + v[r][i][1]) + (v[r][i][2] + v[r][i][3]) : 0.f;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) mean[r] = wave_sum_dpp(mean[r]);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      mean[r] *= inv;
      rstd[r] = 0.f;
#pragma unroll
      for (int i = 0; i < V; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float d = lane + 64 * i < vecs ? v[r][i][e] - mean[r] : 0.f;
          rstd[r] += d * d;
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) rstd[r] = wave_sum_dpp(rstd[r]);
#pragma unroll
    for (int r = 0; r < R; ++r) rstd[r] = rsqrtf(rstd[r] * inv + ln.eps);
    if (cw < vecs) {
      gb[cw] = g;
      gb[kLnMaxK / 4 + cw] = b;
    }
    if (lane == 0) {
#pragma unroll
      for (int r = 0; r < R; ++r) st[wave * R + r] = make_float2(mean[r], rstd[r]);
    }
    __syncthreads();
    if (write) {
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const int32_t c = lane + 64 * i;
        if (c >= vecs) continue;
        const f32x4 gc = gb[c], bc = gb[kLnMaxK / 4 + c];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int64_t m = m0 + wave * R + r;
          if (m < M) reinterpret_cast<f32x4*>(ln.u + (size_t)m * K)[c] = (v[r][i] - mean[r]) * rstd[r] * gc + bc;
        }
      }
    }
  }
};

// TN x TM tiles of 16 x 16 (columns x rows of y) per workgroup, WK wavefronts along K, kDepth slabs in flight each.
// LN: the x rows are normalised on the way (a launch of its own costs 3 to 4 us, of which the work is a fraction): every
// workgroup takes the statistics of its 16 rows while its first slabs are on their way, and the operands as they leave LDS.
template <int TM, int TN, int WK, int kDepth, bool LN = false>
__global__ __launch_bounds__(WK * 64) void gemm_f32_kernel(const float* __restrict__ x, const float* __restrict__ w,
                                                          const float* __restrict__ bias, const float* res, float* y,
                                                          int64_t M, int32_t N, int32_t K, int epi, int32_t tiles_m,
                                                          int32_t tiles_n, LnRows ln) {
  static_assert(!LN || TM == 1, "16 rows of statistics");
  using Cfg = WaveRings<TM, TN, WK, kDepth>;
  constexpr int G = 2 * (TM + TN);   // 1 KiB loads (8 rows x 128 bytes) per slab
  extern __shared__ f32x4 lds[];
  int64_t m0;
  int32_t n0;
  if (!tile_origin<16 * TM, 16 * TN>(tiles_m, tiles_n, m0, n0)) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lrow = lane & 15, lq = lane >> 4;

  // slabs of 32 k (128 bytes of a row): wavefront w takes slabs w, w + WK, ...; the last slab may be partial
  const int32_t slabs = (K + 31) >> 5;
  const int32_t ns = (slabs - wave + WK - 1) / WK;
  f32x4* ring = lds + wave * (kDepth * Cfg::kSlotVecs);

  // Lane l of a load lands in slot l % 8 of row l / 8 of its 8-row group and fetches the chunk that the
  // swizzle keeps there.  Rows past the edge read the last row and are dropped; chunks past K (in the last
  // slab only) read the row's last chunk and are replaced by zeros when they are used.
  const char *pw[2 * TN], *px[2 * TM];
  uint32_t chunk[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) chunk[p] = (uint32_t)((lane & 7) ^ swz16((lane >> 3) + 8 * p));
#pragma unroll
  for (int g = 0; g < 2 * TN; ++g) {
    const int32_t n = n0 + 8 * g + (lane >> 3);
    pw[g] = reinterpret_cast<const char*>(w + (size_t)(n < N ? n : N - 1) * K);
  }
#pragma unroll
  for (int g = 0; g < 2 * TM; ++g) {
    const int64_t m = m0 + 8 * g + (lane >> 3);
    px[g] = reinterpret_cast<const char*>(x + (size_t)(m < M ? m : M - 1) * K);
  }
  const uint32_t last_chunk = (uint32_t)K * 4u - 16u;   // byte offset of a row's last chunk (K < 2^24)
  auto issue = [&](int32_t slot, int32_t i) {
    const uint32_t k = (uint32_t)(wave + i * WK) * 128u;
    f32x4* dst = ring + slot * Cfg::kSlotVecs;
    uint32_t off[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) off[p] = min(k + chunk[p] * 16u, last_chunk);
#pragma unroll
    for (int g = 0; g < 2 * TN; ++g)
      __builtin_amdgcn_global_load_lds((f32_gptr_t)(pw[g] + off[g & 1]), (f32_lptr_t)(dst + g * 64), 16, 0, 0);
#pragma unroll
    for (int g = 0; g < 2 * TM; ++g)
      __builtin_amdgcn_global_load_lds((f32_gptr_t)(px[g] + off[g & 1]), (f32_lptr_t)(dst + (2 * TN + g) * 64), 16, 0, 0);
  };

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  uint32_t foff[2];   // operand reads: row l % 16 of a 16-row tile, chunk 4 h + l / 16
#pragma unroll
  for (int h = 0; h < 2; ++h) foff[h] = (uint32_t)(lrow * 8 + ((4 * h + lq) ^ swz16(lrow)));

  __shared__ float2 ln_st[LN ? 16 : 1];
  __shared__ f32x4 ln_gb[LN ? kLnMaxK / 2 : 1];
  std::conditional_t<LN, LnTile<LN ? WK : 4>, char> ln_tile;
  if constexpr (LN) ln_tile.request(x, ln, m0, M, K, wave, lane);
  for (int32_t u = 0; u < kDepth && u < ns; ++u) issue(u, u);
  float mean = 0.f, rstd = 0.f;
  if constexpr (LN) {
    ln_tile.finish(ln, m0, M, K, n0 == 0, wave, lane, ln_st, ln_gb);
    mean = ln_st[lrow].x;
    rstd = ln_st[lrow].y;
  }
  int32_t slot = 0;
  for (int32_t i = 0; i < ns; ++i) {
    // loads return in order; behind slab i's are those of the next kDepth - 1 slabs while they all exist
    if (i + kDepth <= ns) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kDepth - 1) * G) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const f32x4* slab = ring + slot * Cfg::kSlotVecs;
    const int32_t left = K - (wave + i * WK) * 32;   // k's of this slab, uniform
    f32x4 wb[2][TN], xa[2][TM];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int t = 0; t < TN; ++t) wb[h][t] = slab[t * 128 + foff[h]];
#pragma unroll
      for (int t = 0; t < TM; ++t) xa[h][t] = slab[(TN + t) * 128 + foff[h]];
    }
    if constexpr (LN) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int32_t c = min((wave + i * WK) * 8 + 4 * h + lq, K / 4 - 1);   // past K: zeros below
        xa[h][0] = (xa[h][0] - mean) * rstd * ln_gb[c] + ln_gb[kLnMaxK / 4 + c];
      }
    }
    if (left < 32) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (16 * h + 4 * lq >= left) {   // K % 4 == 0: whole chunks
#pragma unroll
          for (int t = 0; t < TN; ++t) wb[h][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int t = 0; t < TM; ++t) xa[h][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    if (i + kDepth < ns) {
      // the slot is refilled by the load unit, which is not ordered with this wavefront's LDS reads
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      issue(slot, i + kDepth);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
          for (int b = 0; b < TM; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(wb[h][a][e], xa[h][b][e], acc[a][b], 0, 0, 0);
    slot = slot + 1 == kDepth ? 0 : slot + 1;
  }

  // the wavefronts' sums meet in LDS (the rings are free once every wavefront is here) and are added in order
  __syncthreads();
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) lds[(wave * TN * TM + a * TM + b) * 64 + lane] = acc[a][b];
  __syncthreads();
  for (int t = wave; t < TN * TM; t += WK) {
    f32x4 v = lds[t * 64 + lane];
#pragma unroll
    for (int k = 1; k < WK; ++k) v += lds[(k * TN * TM + t) * 64 + lane];
    // tile (t / TM, t % TM): row l % 16 of y's rows, columns 4 (l / 16) .. + 3
    const int64_t m = m0 + 16 * (t % TM) + lrow;
    const int32_t col = n0 + 16 * (t / TM) + 4 * lq;
    if (m >= M || col >= N) continue;   // N % 4 == 0
    const size_t off = (size_t)m * N + col;
    if (bias != nullptr) v += *reinterpret_cast<const f32x4*>(bias + col);
    if (epi == EPI_BIAS_GELU) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = gelu_erf(v[e]);
    }
    if (epi == EPI_BIAS_RESIDUAL) v += *reinterpret_cast<const f32x4*>(res + off);
    *reinterpret_cast<f32x4*>(y + off) = v;
  }
}

template <int TM, int TN, int WK, int kDepth, bool LN = false>
hipError_t launch_cfg(const float* x, const float* w, const float* bias, const float* res, float* y, int64_t M,
                      int32_t N, int32_t K, int epi, hipStream_t s, const LnRows& ln = {}) {
  constexpr int BM = 16 * TM, BN = 16 * TN;
  constexpr size_t lds = WaveRings<TM, TN, WK, kDepth>::kLds;
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  auto kern = gemm_f32_kernel<TM, TN, WK, kDepth, LN>;
  static LdsAttrOnce once;
  hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds, once);
  if (e != hipSuccess) return e;
  const int32_t tiles_m = (int32_t)((M + BM - 1) / BM), tiles_n = (N + BN - 1) / BN;
  const int64_t grid = ((int64_t)tiles_m * tiles_n + kXcds - 1) / kXcds * kXcds;
  if (grid * WK * 64 > kMaxGridThreads) return hipErrorInvalidConfiguration;
  kern<<<dim3((unsigned)grid), dim3(WK * 64), lds, s>>>(x, w, bias, res, y, M, N, K, epi, tiles_m, tiles_n, ln);
  return hipGetLastError();
}

}  // namespace

// Where the linear runs on 16 x 16 tiles and four wavefronts, at most two of them per CU, and rows are short: every workgroup reads
// its 16 rows once more and normalises them for itself.  77 rows, 256 / 768 / 1024 wide: the step 41 -> 33.5 us; but 40 rows,
// 1024 / 3072 / 4096 wide, with 576 and 768 workgroups: 40 -> 48.5.  Replayed from a graph, where a launch costs less, 3400 such layers
// take 0.955 of the time in the mean (0.86 to 1.04; the longest rows gain nothing).
bool gemm_f32_takes_ln(int64_t M, int32_t N, int32_t K) {
  return M > 0 && N > 16 && K > 64 && K <= kLnMaxK && ((M + 15) / 16) * ((N + 15) / 16) <= 512 &&
         (M <= 16 || ((M + 31) / 32) * ((N + 31) / 32) < 168);
}

hipError_t launch_gemm_f32_ln(const float* x, const float* gamma, const float* beta, float eps, float* u, const float* w,
                              const float* bias, float* y, int64_t M, int32_t N, int32_t K, int epi, hipStream_t s) {
  if (!gemm_f32_takes_ln(M, N, K) || epi == EPI_BIAS_RESIDUAL) return hipErrorInvalidValue;
  return launch_cfg<1, 1, 4, 2, true>(x, w, bias, nullptr, y, M, N, K, epi, s, LnRows{gamma, beta, eps, u});
}

hipError_t launch_gemm_f32(const float* x, const float* w, const float* bias, const float* res, float* y, int64_t M,
                           int32_t N, int32_t K, int epi, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  const auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  const int64_t t16 = tiles(16, 16), t32 = tiles(32, 32), t64 = tiles(64, 64);
  const auto fits = [](int64_t n) { return n * 256 <= kMaxGridThreads; };
  // Large tiles move fewer bytes, small ones make more workgroups; where the lines lie (measured, us):
  //   16 x 16 where a side has no more than that, whatever the other: 100000 x 4 x 4 10 against 29 with 64 x 64 (15 with
  //     32 x 32), 300000 x 16 x 16 36 / 84 (47), 4 x 100000 x 64 11 / 33 (16);
  //   32 x 32 from 168 tiles: 130 x 1600 x 6400 (250) 34 against 48 with 16 x 16; 37 x 1600 x 1600 (100) 10.6 / 7.3;
  //   in between, where 32 x 32 would be one to two rounds of 256 CUs, 32 x 64 is one: 387 x 1024 x 1024
  //     (416) 12.8 against 14.4;
  //   64 x 64 where its whole rounds are expected to take less time than the smaller tiles' (fits to 181 shapes): 64 x 64
  //     against the smaller, 655 x 3072 x 1024 (528) 73 / 58, 700 x 3072 x 1024 73 / 60, 100000 x 64 x 64 38 / 34, but
  //     600 x 4800 x 1600 (750) 98 / 103, 2048 x 2048 x 8192 (1024) 571 / 663;
  //   16 x 16 with eight wavefronts along a long K while every CU has at most one tile: 17 x 2048 x 8192
  //     15.7 against 20.0 with four.
  //   K of two slabs at most: one wavefront, nothing to cut and no sums to meet: 32 x 32 8000 x 8000 x 4 104 against 263 (and 139 with
  //     64 x 64), 2000 x 2000 x 64 14 / 22, 300000 x 20 x 16 19 / 40; 16 x 16 1000000 x 4 x 4 37 / 81, 300 x 300 x 16 2.6 / 2.8.
  const bool narrow = (M <= 16 || N <= 16) && fits(t16);
  if (K <= 64) {
    if (narrow || t32 < 168) return launch_cfg<1, 1, 1, 2>(x, w, bias, res, y, M, N, K, epi, s);
    if (fits(t32)) return launch_cfg<2, 2, 1, 2>(x, w, bias, res, y, M, N, K, epi, s);
  }
  if (!narrow && t32 >= 168) {
    const double k = K;
    const double us64 = std::ceil(t64 / 256.0) * (9.0 + 0.0155 * k);
    const bool halves = t32 > 256 && t32 <= 512;
    const double us = halves ? std::ceil(tiles(32, 64) / 256.0) * (3.5 + 0.0088 * k) : 2.0 + t32 / 256.0 * (1.6 + 0.0049 * k);
    if (us64 < us || !fits(t32)) return launch_cfg<4, 4, 4, 2>(x, w, bias, res, y, M, N, K, epi, s);
    if (halves) return launch_cfg<2, 4, 4, 2>(x, w, bias, res, y, M, N, K, epi, s);
    return launch_cfg<2, 2, 4, 2>(x, w, bias, res, y, M, N, K, epi, s);
  }
  if (t16 <= 256 && K >= 2048) return launch_cfg<1, 1, 8, 2>(x, w, bias, res, y, M, N, K, epi, s);
  return launch_cfg<1, 1, 4, 2>(x, w, bias, res, y, M, N, K, epi, s);
}

}  // namespace energon
