// fp32 linear layer  y = epilogue(x W^T + b)  on packed rows (paper Sec. 4.3: the linear
// layers see only valid tokens): the fp32 storage path, on the fp32 matrix instructions
// (v_mfma_f32_16x16x4_f32: fp32 products and sums, 157 TFLOP/s).
//
// These problems are small: what bounds them is latency, idle CUs and, from a few hundred rows on, bytes moved to a CU per flop
// and the fp32 instructions' rate (then the split kernel below takes them).  So:
//  * a workgroup owns a tile of 16 (split kernel: 32 to 64) rows and columns and all of K, which its 1 to 8 wavefronts cut
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
// Against the former kernel (vector ALU, 64 x 64 LDS tile, 4 x 4 registers per lane): 76 x 256 x 1024 149 -> 4.1 us.
#include "common.h"
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

// Rows m0 .. m0 + 15 of x normalised as layernorm_kernel does it (two passes over a row in registers): a row per wavefront at a
// time.  Mean and 1 / deviation to st, gain and offset to gb; with `write` the normalised rows to ln.u.
template <int WK>
__device__ __forceinline__ void ln_rows(const float* __restrict__ x, const LnRows& ln, int64_t m0, int64_t M, int32_t K, bool write,
                                        int wave, int lane, float2* st, f32x4* gb) {
  constexpr int V = kLnMaxK / 256;
  const int32_t vecs = K / 4;   // K % 4 == 0
  for (int32_t c = wave * 64 + lane; c < vecs; c += WK * 64) {
    gb[c] = reinterpret_cast<const f32x4*>(ln.gamma)[c];
    gb[kLnMaxK / 4 + c] = reinterpret_cast<const f32x4*>(ln.beta)[c];
  }
  constexpr int R = 16 / WK;
  f32x4 v[R][V];
#pragma unroll
  for (int r = 0; r < R; ++r) {   // all rows requested before the first is summed
    const int64_t m = m0 + wave * R + r;
    const f32x4* row = reinterpret_cast<const f32x4*>(x + (size_t)(m < M ? m : M - 1) * K);
#pragma unroll
    for (int i = 0; i < V; ++i) v[r][i] = lane + 64 * i < vecs ? row[lane + 64 * i] : f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float inv = 1.0f / (float)K;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    float sum = 0.f, sq = 0.f;
#pragma unroll
    for (int i = 0; i < V; ++i) sum += (v[r][i][0] + v[r][i][1]) + (v[r][i][2] + v[r][i][3]);
    const float mean = wave_sum(sum) * inv;
#pragma unroll
    for (int i = 0; i < V; ++i)
      if (lane + 64 * i < vecs) {
#pragma unroll
        for (int e = 0; e < 4; ++e) sq += (v[r][i][e] - mean) * (v[r][i][e] - mean);
      }
    const float rstd = rsqrtf(wave_sum(sq) * inv + ln.eps);
    if (lane == 0) st[wave * R + r] = make_float2(mean, rstd);
    const int64_t m = m0 + wave * R + r;
    if (write && m < M) {
      f32x4* out = reinterpret_cast<f32x4*>(ln.u + (size_t)m * K);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const int32_t c = lane + 64 * i;
        if (c < vecs) {
          const f32x4 g = reinterpret_cast<const f32x4*>(ln.gamma)[c], b = reinterpret_cast<const f32x4*>(ln.beta)[c];
          out[c] = (v[r][i] - mean) * rstd * g + b;
        }
      }
    }
  }
}

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

  for (int32_t u = 0; u < kDepth && u < ns; ++u) issue(u, u);
  __shared__ float2 ln_st[LN ? 16 : 1];
  __shared__ f32x4 ln_gb[LN ? kLnMaxK / 2 : 1];
  float mean = 0.f, rstd = 0.f;
  if constexpr (LN) {
    ln_rows<WK>(x, ln, m0, M, K, n0 == 0, wave, lane, ln_st, ln_gb);
    __syncthreads();
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

// The same on the bf16 matrix instructions (v_mfma_f32_16x16x32_bf16: 16 times the flops of the fp32 ones per cycle): every fp32 operand
// is the sum of three bf16 numbers, its bits cut in three (hi + mid + lo: 24 bits, so exact, and nothing rounds up to infinity);
// their products are exact in fp32, and the six that matter (hi hi; hi mid, mid hi; hi lo, mid mid, lo hi; the rest is below 2^-21
// of a product, 2^-24 in the mean) are summed in fp32, hi hi in accumulators of its own, so that the others cost it no roundings.  Distance to the
// 64-bit answer (2-norm; fp32 instructions / this): K = 100 1.1e-7 / 8.5e-8, 768 2.5e-7 / 1.1e-7, 4096 5.8e-7 / 2.0e-7: fewer sums
// are rounded.  Values below 2^-110 have parts that bf16 cannot hold: their products lose up to 2^-133 of the other factor.
// What bounds it: the split, 44 vector instructions per 8 elements and lane, beside 96 cycles of the matrix cores per pair of 16-row
// operands (v_cvt_pk_bf16_f32 instead of the masks runs at a quarter of the rate: 10 % slower), and the operands' way to the CU.  A
// wavefront splits the next slab's operands while the matrix cores work on the slab before, whose first third covers the LDS
// reads.  us, before (fp32 instructions) -> now: 387 x 3072 x 1024 31 -> 25, 387 x 1024 x 4096 40 -> 34, 2048 x 6400 x 1600 400 ->
// 307 (137 TFLOP/s), 800 x 768 x 3072 55 -> 35.
struct Split3 { bf16x8 hi, mid, lo; };
__device__ __forceinline__ Split3 split3(f32x4 a, f32x4 b) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 hi, mid, lo;
#pragma unroll
  for (int p = 0; p < 4; ++p) {   // elements 2 p, 2 p + 1
    uint32_t v[2], r[2], q[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float f = p < 2 ? a[2 * p + i] : b[2 * p - 4 + i];
      v[i] = __float_as_uint(f);
      const float rest = f - __uint_as_float(v[i] & 0xffff0000u);   // exact
      r[i] = __float_as_uint(rest);
      q[i] = __float_as_uint(rest - __uint_as_float(r[i] & 0xffff0000u));
    }
    hi[p] = __builtin_amdgcn_perm(v[1], v[0], 0x07060302u);   // the high halves
    mid[p] = __builtin_amdgcn_perm(r[1], r[0], 0x07060302u);
    lo[p] = __builtin_amdgcn_perm(q[1], q[0], 0x07060302u);
  }
  return {__builtin_bit_cast(bf16x8, hi), __builtin_bit_cast(bf16x8, mid), __builtin_bit_cast(bf16x8, lo)};
}

template <int TM, int TN, int WK, int kDepth>
__global__ __launch_bounds__(WK * 64) void gemm_f32_split_kernel(const float* __restrict__ x, const float* __restrict__ w,
                                                                const float* __restrict__ bias, const float* res, float* y,
                                                                int64_t M, int32_t N, int32_t K, int epi, int32_t tiles_m,
                                                                int32_t tiles_n) {
  using Cfg = WaveRings<TM, TN, WK, kDepth>;
  constexpr int G = 2 * (TM + TN);   // 1 KiB loads (8 rows x 128 bytes) per slab
  extern __shared__ f32x4 lds[];
  int64_t m0;
  int32_t n0;
  if (!tile_origin<16 * TM, 16 * TN>(tiles_m, tiles_n, m0, n0)) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lrow = lane & 15, lq = lane >> 4;
  const int32_t slabs = (K + 31) >> 5;
  const int32_t ns = (slabs - wave + WK - 1) / WK;   // slabs wave, wave + WK, ...
  f32x4* ring = lds + wave * (kDepth * Cfg::kSlotVecs);

  // loads as in the kernel above, but a wavefront-uniform base and 32-bit offsets (64 rows x K x 4 bytes, K < 2^24)
  uint32_t ow[2 * TN], ox[2 * TM], chunk[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) chunk[p] = (uint32_t)((lane & 7) ^ swz16((lane >> 3) + 8 * p)) * 16u;
  const char* const wbase = reinterpret_cast<const char*>(w + (size_t)n0 * K);
  const char* const xbase = reinterpret_cast<const char*>(x + (size_t)m0 * K);
#pragma unroll
  for (int g = 0; g < 2 * TN; ++g) ow[g] = (uint32_t)min(8 * g + (lane >> 3), N - 1 - n0) * (uint32_t)K * 4u;
  const int32_t last_m = (int32_t)(M - 1 - m0 < 1024 ? M - 1 - m0 : 1024);
#pragma unroll
  for (int g = 0; g < 2 * TM; ++g) ox[g] = (uint32_t)min(8 * g + (lane >> 3), last_m) * (uint32_t)K * 4u;
  const uint32_t last_chunk = (uint32_t)K * 4u - 16u;   // byte offset of a row's last chunk
  auto issue = [&](int32_t slot, int32_t i) {
    const uint32_t k = (uint32_t)(wave + i * WK) * 128u;
    f32x4* dst = ring + slot * Cfg::kSlotVecs;
    uint32_t off[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) off[p] = min(k + chunk[p], last_chunk);
#pragma unroll
    for (int g = 0; g < 2 * TN; ++g)
      __builtin_amdgcn_global_load_lds((f32_gptr_t)(wbase + (ow[g] + off[g & 1])), (f32_lptr_t)(dst + g * 64), 16, 0, 0);
#pragma unroll
    for (int g = 0; g < 2 * TM; ++g)
      __builtin_amdgcn_global_load_lds((f32_gptr_t)(xbase + (ox[g] + off[g & 1])), (f32_lptr_t)(dst + (2 * TN + g) * 64), 16, 0, 0);
  };

  f32x4 big[TN][TM], small[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) big[i][j] = small[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  uint32_t foff[2];   // operand reads: row l % 16 of a 16-row tile, chunk 4 h + l / 16
#pragma unroll
  for (int h = 0; h < 2; ++h) foff[h] = (uint32_t)(lrow * 8 + ((4 * h + lq) ^ swz16(lrow)));

  // slab i out of its slot, zeros past K
  f32x4 raw[TN + TM][2];
  auto fetch = [&](int32_t i, int32_t slot) {
    // loads return in order; behind slab i's are those of the next kDepth - 1 slabs while they all exist
    if (i + kDepth <= ns) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kDepth - 1) * G) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const f32x4* slab = ring + slot * Cfg::kSlotVecs;
    const int32_t left = K - (wave + i * WK) * 32;   // k's of this slab, uniform
#pragma unroll
    for (int t = 0; t < TN + TM; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) raw[t][h] = slab[t * 128 + foff[h]];
    if (left < 32) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (16 * h + 4 * lq >= left) {   // K % 4 == 0: whole chunks
#pragma unroll
          for (int t = 0; t < TN + TM; ++t) raw[t][h] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
  };
  auto refill = [&](int32_t i, int32_t slot) {   // by the load unit, which is not ordered with this wavefront's LDS reads
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (i + kDepth < ns) issue(slot, i + kDepth);
  };
  Split3 op[2][TN + TM];
  // one kind of product after the other, so that no MFMA waits for the one before
  auto all = [&](const Split3 (&o)[TN + TM], auto part_w, auto part_x, f32x4 (&acc)[TN][TM]) {
#pragma unroll
    for (int b = 0; b < TM; ++b)
#pragma unroll
      for (int a = 0; a < TN; ++a) acc[a][b] = Mfma<bf16_t>::m16x16x32(part_w(o[a]), part_x(o[TN + b]), acc[a][b]);
  };
  const auto hi = [](const Split3& v) { return v.hi; };
  const auto mid = [](const Split3& v) { return v.mid; };
  const auto lo = [](const Split3& v) { return v.lo; };
  auto first = [&](const Split3 (&o)[TN + TM]) {   // a third of them
    all(o, hi, lo, small);
    all(o, hi, hi, big);
  };
  auto others = [&](const Split3 (&o)[TN + TM]) {
    all(o, lo, hi, small);
    all(o, mid, mid, small);
    all(o, hi, mid, small);
    all(o, mid, hi, small);
  };

  for (int32_t u = 0; u < kDepth && u < ns; ++u) issue(u, u);
  if (ns > 0) {
    int32_t slot = 0;
    const auto next = [&] { const int32_t s = slot; slot = slot + 1 == kDepth ? 0 : slot + 1; return s; };
    int32_t at = next();
    fetch(0, at);
    refill(0, at);
#pragma unroll
    for (int t = 0; t < TN + TM; ++t) op[0][t] = split3(raw[t][0], raw[t][1]);
    // two slabs per trip, so that neither operand set is copied
    auto trip = [&](auto P, int32_t i) {
      constexpr int p = decltype(P)::value;
      at = next();
      fetch(i + 1, at);
      __builtin_amdgcn_sched_barrier(0);
      first(op[p]);   // while the reads are on their way
      __builtin_amdgcn_sched_barrier(0);
      refill(i + 1, at);
      others(op[p]);
#pragma unroll
      for (int t = 0; t < TN + TM; ++t) op[1 - p][t] = split3(raw[t][0], raw[t][1]);
      // a few vector instructions of the split behind every MFMA
#pragma unroll
      for (int q = 0; q < 4 * TM * TN; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, (44 * (TM + TN) + 4 * TM * TN - 1) / (4 * TM * TN), 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    int32_t i = 0;
    for (; i + 2 < ns; i += 2) {
      trip(std::integral_constant<int, 0>{}, i);
      trip(std::integral_constant<int, 1>{}, i + 1);
    }
    if (i + 1 < ns) {
      trip(std::integral_constant<int, 0>{}, i);
      first(op[1]);
      others(op[1]);
    } else {
      first(op[0]);
      others(op[0]);
    }
  }

  // the wavefronts' sums meet in LDS (the rings are free once every wavefront is here) and are added in order
  __syncthreads();
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) lds[(wave * TN * TM + a * TM + b) * 64 + lane] = big[a][b] + small[a][b];
  __syncthreads();
  for (int t = wave; t < TN * TM; t += WK) {
    f32x4 v = lds[t * 64 + lane];
#pragma unroll
    for (int k = 1; k < WK; ++k) v += lds[(k * TN * TM + t) * 64 + lane];
    // tile (t / TM, t % TM): row l % 16 of y's rows, columns 4 (l / 16) .. + 3
    const int64_t m = m0 + 16 * (t % TM) + lrow;
    const int32_t col = n0 + 16 * (t / TM) + 4 * lq;
    if (m >= M || col >= N) continue;   // N % 4 == 0
    // A sum that is not finite may owe it to the split (inf - inf, a value that rounds to infinity in bf16): as fp32 has it.
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (!(fabsf(v[e]) <= 3.402823466e+38f)) {
        float sum = 0.f;
        for (int32_t k = 0; k < K; ++k) sum = fmaf(x[(size_t)m * K + k], w[(size_t)(col + e) * K + k], sum);
        v[e] = sum;
      }
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

template <int TM, int TN, int WK, int kDepth>
hipError_t launch_split(const float* x, const float* w, const float* bias, const float* res, float* y, int64_t M,
                        int32_t N, int32_t K, int epi, hipStream_t s) {
  constexpr int BM = 16 * TM, BN = 16 * TN;
  constexpr size_t lds = WaveRings<TM, TN, WK, kDepth>::kLds;
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  auto kern = gemm_f32_split_kernel<TM, TN, WK, kDepth>;
  static LdsAttrOnce once;
  hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds, once);
  if (e != hipSuccess) return e;
  const int32_t tiles_m = (int32_t)((M + BM - 1) / BM), tiles_n = (N + BN - 1) / BN;
  const int64_t grid = ((int64_t)tiles_m * tiles_n + kXcds - 1) / kXcds * kXcds;
  if (grid * WK * 64 > kMaxGridThreads) return hipErrorInvalidConfiguration;
  kern<<<dim3((unsigned)grid), dim3(WK * 64), lds, s>>>(x, w, bias, res, y, M, N, K, epi, tiles_m, tiles_n);
  return hipGetLastError();
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

// Tiles of the split kernel: workgroups of WK wavefronts, per_cu of them on a CU.  A launch takes base, then rounds of
// workgroups: a round is its epilogue and its steps (a slab for each wavefront), a step as long as the workgroups on a CU make it
// and shorter where not every CU has one more.  Fitted to 3700 shapes of 17 to 2200 rows; the choice costs 0.6 % over the best
// in the mean.
struct SplitTile {
  int16_t rows, cols, waves, per_cu;
  double base, round, drop, step[4];
  double us(int32_t n, int32_t cus, int32_t slabs) const {   // n workgroups on an XCD of so many CUs
    const int32_t slots = cus * per_cu, whole = (n - 1) / slots, rest = n - whole * slots, level = (rest + cus - 1) / cus;
    const int32_t steps = (slabs + waves - 1) / waves;
    return base + whole * (round + steps * step[per_cu - 1]) + round * (level + 1) / (per_cu + 1) +
           steps * step[level - 1] * (1.0 - drop * (level - rest / (double)cus));
  }
};
constexpr SplitTile kSplitTiles[] = {{64, 64, 4, 1, 2.99, 3.90, 0.165, {1.777}},
                                     {32, 32, 4, 2, 2.80, 1.46, 0.054, {0.695, 1.024}},
                                     {32, 32, 8, 1, 1.93, 1.78, 0.199, {1.123}},
                                     {32, 48, 4, 2, 3.72, 1.51, 0.088, {0.901, 1.412}},
                                     {48, 32, 4, 2, 3.56, 1.49, 0.102, {0.930, 1.439}},
                                     {32, 48, 2, 4, 3.81, 2.06, 0.090, {0.781, 1.183, 1.301, 1.421}}};

hipError_t launch_split_tile(const float* x, const float* w, const float* bias, const float* res, float* y, int64_t M, int32_t N,
                             int32_t K, int epi, hipStream_t s) {
  constexpr int kTiles = sizeof(kSplitTiles) / sizeof(kSplitTiles[0]);
  int best = 0;
  double best_us = 1e30;
  for (int i = 0; i < kTiles; ++i) {
    const SplitTile& t = kSplitTiles[i];
    const int64_t n = (int64_t)(((uint32_t)M + t.rows - 1) / t.rows) * (((uint32_t)N + t.cols - 1) / t.cols);
    if (n * 512 > kMaxGridThreads) continue;
    const double us = t.us((int32_t)((n + kXcds - 1) / kXcds), 32, (K + 31) / 32);
    if (us < best_us) { best = i; best_us = us; }
  }
  switch (best) {   // the order of kSplitTiles
    case 1: return launch_split<2, 2, 4, 2>(x, w, bias, res, y, M, N, K, epi, s);
    case 2: return launch_split<2, 2, 8, 2>(x, w, bias, res, y, M, N, K, epi, s);
    case 3: return launch_split<2, 3, 4, 2>(x, w, bias, res, y, M, N, K, epi, s);
    case 4: return launch_split<3, 2, 4, 2>(x, w, bias, res, y, M, N, K, epi, s);
    case 5: return launch_split<2, 3, 2, 2>(x, w, bias, res, y, M, N, K, epi, s);
    default: return launch_split<4, 4, 4, 2>(x, w, bias, res, y, M, N, K, epi, s);
  }
}

}  // namespace

// Where the linear runs on 16 x 16 tiles and four wavefronts, at most two of them per CU, and rows are short: every workgroup reads
// its 16 rows once more and normalises them for itself.  77 rows, 256 / 768 / 1024 wide: the step 41 -> 33.5 us; but 40 rows,
// 1024 / 3072 / 4096 wide, with 576 and 768 workgroups: 40 -> 48.5.
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
  const int64_t t16 = tiles(16, 16), t32 = tiles(32, 32);
  const auto fits = [](int64_t n) { return n * 256 <= kMaxGridThreads; };
  // Large tiles move fewer bytes, small ones make more workgroups; where the lines lie (measured, us):
  //   16 x 16 where a side has no more than that, whatever the other: 100000 x 4 x 4 10 against 29 with 64 x 64 (15 with
  //     32 x 32), 300000 x 16 x 16 36 / 84 (47), 4 x 100000 x 64 11 / 33 (16);
  //   K of two slabs at most: one wavefront, nothing to cut and no sums to meet: 32 x 32 8000 x 8000 x 4 104 against 263,
  //     2000 x 2000 x 64 14 / 22, 300000 x 20 x 16 19 / 40; 16 x 16 1000000 x 4 x 4 37 / 81, 300 x 300 x 16 2.6 / 2.8;
  //   the split kernel from 168 tiles of 32 x 32 (0.95 of the time of 16 x 16 or the former 32 x 32 and 64 x 64 tiles on the fp32
  //     instructions for 168 to 256 of them, 0.79 from 512; 1.07 times below): 387 x 1024 x 4096 40 -> 34, 2048 x 1600 x 6400 400 -> 300;
  //   16 x 16 with eight wavefronts along a long K while every CU has at most one tile: 17 x 2048 x 8192
  //     15.7 against 20.0 with four.
  const bool narrow = (M <= 16 || N <= 16) && fits(t16);
  if (K <= 64) {
    if (narrow || t32 < 168) return launch_cfg<1, 1, 1, 2>(x, w, bias, res, y, M, N, K, epi, s);
    if (fits(t32)) return launch_cfg<2, 2, 1, 2>(x, w, bias, res, y, M, N, K, epi, s);
  }
  if (!narrow && t32 >= 168) return launch_split_tile(x, w, bias, res, y, M, N, K, epi, s);
  if (t16 <= 256 && K >= 2048) return launch_cfg<1, 1, 8, 2>(x, w, bias, res, y, M, N, K, epi, s);
  return launch_cfg<1, 1, 4, 2>(x, w, bias, res, y, M, N, K, epi, s);
}

}  // namespace energon
