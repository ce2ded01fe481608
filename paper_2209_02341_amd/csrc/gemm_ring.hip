// 16-bit linear layer  y[M,N] = epilogue(x[M,K] W[N,K]^T + b)  for problems of some hundred to a few thousand rows, whose
// 256x256 tiles would not fill the chip: smaller tiles, one per workgroup, a ring of slabs in LDS.
//
// What bounds such a problem is, per slab of 64 k, the longer of the matrix cores' time, at the rate that the power limit lets
// them run on random operands, and of the slab's way to the CU: a CU holds about 32 KB of lines in flight, however many loads
// are outstanding (measured: 51 KB/us from HBM, 90 from the memory-side cache, 130 from the L2).  So:
//  * four wavefronts in two rows and two columns, one per SIMD, each with (BM / 2) x (BN / 2) of the output on
//    v_mfma_f32_16x16x32, the sums in AGPRs: few operand bytes from LDS per flop;
//  * two sets of operand registers: while the MFMAs of one step of 32 k run, the operands of the next one are read
//    into the other set, so no MFMA waits for LDS.  MFMAs, reads and slab loads are ordered asm statements (the compiler
//    otherwise reads operands just before their use, with a wait of its own in front of every few MFMAs);
//  * S slabs in LDS, filled straight from global memory (global_load_lds_dwordx4, the swizzle of 16-row operands applied
//    on the global side), as many as fit.  One barrier per slab, between its two steps: past it the next slab has landed for
//    every wavefront and nobody reads the current one any more (its second operands are in registers), so the loads of the
//    slab S ahead go into its place during the second step and the first one of the next slab;
//  * results leave through LDS as whole row segments; rows and columns past the edge read the last one and are dropped.
// Against the former kernel of such tiles (compiler-scheduled, 32x32x16, one operand set), us on one / three sets of operands in
// turn: 2048 x 4096 x 4096 78 -> 59, 928 x 5120 x 5120 + residual 67 -> 54 / 72 -> 55, 333 x 5120 x 20480 + residual 95 -> 76 / 99 ->
// 87 (W then comes from HBM: 2.4 TB/s), 387 x 3072 x 1024 9.7 -> 7.9 / 9.8 -> 8.3.  Operands of zeros: 2048 x 4096 x 4096 46, which
// is what power takes.  More slabs in the ring, or the LDS reads spread over the MFMAs: no difference.
#include "common.h"
#include <type_traits>
#include <utility>

namespace energon {

namespace {

typedef __attribute__((address_space(1))) const void* ring_gptr_t;
typedef __attribute__((address_space(3))) void* ring_lptr_t;

template <typename F, int... I> __device__ __forceinline__ void each_of(std::integer_sequence<int, I...>, F f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void each(F f) { each_of(std::make_integer_sequence<int, N>{}, f); }

constexpr int kRingWaves = 4;   // 2 x 2

// LDS of a workgroup: the slabs, and in their place, on the way out, row tiles (of 16) of every wavefront, as many at a
// time as fit there.
constexpr int ring_stage_ld(int TN) { return TN * 16 + 4; }   // floats; 4 more spread the four row groups over the banks
constexpr size_t ring_lds(int TM, int TN, int S) { return (size_t)S * 32 * (TM + TN) * 128; }
constexpr int ring_rows_staged(int TM, int TN, int S) {
  int n = TM;
  while (TM % n != 0 || (size_t)kRingWaves * n * 16 * ring_stage_ld(TN) * sizeof(float) > ring_lds(TM, TN, S)) --n;
  return n;
}

#define RING_READ(dst, addr, off) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(off) : "memory")
#define RING_MFMA(acc, a, b)                                                                             \
  do {                                                                                                   \
    if constexpr (__is_same(E, bf16_t))                                                                  \
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));              \
    else                                                                                                 \
      asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));               \
  } while (0)

// TM x TN tiles of 16 x 16 (rows x columns) per wavefront, S slabs in LDS, PER_CU workgroups per CU.
// MODE 0: plain epilogues; 1: the LayerNorm-folded epilogues; 2: K cut into parts, the fp32 sums of part p to
// lf.partial + p * M * N (lf.partial is the caller's scratch here).
template <typename E, int TM, int TN, int S, int PER_CU, int MODE>
__global__ __launch_bounds__(kRingWaves * 64, PER_CU) void gemm_ring_kernel(const E* __restrict__ x, const E* __restrict__ w,
                                                                          const E* __restrict__ bias, const E* res, E* y,
                                                                          int64_t M, int32_t N, int32_t K, int epi,
                                                                          int32_t tiles_m, int32_t tiles_n, int32_t parts, LnFold lf) {
  constexpr int BM = 32 * TM, BN = 32 * TN;
  constexpr int GA = BM / 8 / kRingWaves, GB = BN / 8 / kRingWaves, G = GA + GB;   // 1 KiB loads (8 rows) per wavefront and slab
  constexpr uint32_t kSlab = (BM + BN) * 128;
  static_assert(S >= 2 && S <= 5 && 3 * G < 64, "the waits below");
  static_assert(ring_lds(TM, TN, S) * PER_CU <= 160 * 1024, "LDS of a CU");
  static_assert(TM * TN >= TM + TN, "an operand read behind every MFMA at most");
  extern __shared__ uint4 smem[];   // [S][BM rows of x, BN rows of W][8 chunks of 16 bytes]

  // Which tile and which part of K: the parts one behind the other, the tiles of a part in bands of kGroupM row tiles;
  // every XCD takes an equal run of them (workgroup id modulo 8), so that its workgroups share x and W slabs in its L2.
  int64_t m0;
  int32_t n0, part;
  {
    const int32_t tiles = tiles_m * tiles_n, xcd = blockIdx.x % kXcds;
    const int64_t units = (int64_t)tiles * parts;
    const int32_t from = (int32_t)(units * xcd / kXcds), to = (int32_t)(units * (xcd + 1) / kXcds);
    const int32_t u = from + (int32_t)(blockIdx.x / kXcds);
    if (u >= to) return;
    part = u / tiles;
    const int32_t idx = u - part * tiles, band = idx / (kGroupM * tiles_n), first = band * kGroupM;
    const int32_t rows = min(kGroupM, tiles_m - first), r = idx - band * kGroupM * tiles_n;
    m0 = (int64_t)(first + r % rows) * BM;
    n0 = (r / rows) * BN;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave >> 1) * (TM * 16), wn0 = (wave & 1) * (TN * 16);

  // this workgroup's slabs: all of K or its part of it
  const int32_t slabs = K / 64;
  const int32_t kb = MODE == 2 ? (int32_t)((int64_t)slabs * part / parts) : 0;
  const int32_t KT = MODE == 2 ? (int32_t)((int64_t)slabs * (part + 1) / parts) - kb : slabs;

  // Slab loads: a wavefront-uniform base that advances by 128 bytes per slab plus 32-bit offsets (the launcher checks
  // that a tile's rows fit).  Lane l of a load lands in slot l % 8 of row l / 8 of its 8-row group and fetches the chunk that the
  // swizzle keeps there.
  const char* xk = reinterpret_cast<const char*>(x + (size_t)m0 * K) + (size_t)kb * 128;
  const char* wk = reinterpret_cast<const char*>(w + (size_t)n0 * K) + (size_t)kb * 128;
  uint32_t oa[GA], ob[GB];
  const int64_t last_m = M - 1 - m0;
  const int32_t last_n = N - 1 - n0;
#pragma unroll
  for (int i = 0; i < GA; ++i) {
    const int row = (wave + i * kRingWaves) * 8 + (lane >> 3);
    oa[i] = ((uint32_t)(row < last_m ? row : last_m) * (uint32_t)K + (uint32_t)((lane & 7) ^ swz16(row & 15)) * 8u) * 2u;
  }
#pragma unroll
  for (int i = 0; i < GB; ++i) {
    const int row = (wave + i * kRingWaves) * 8 + (lane >> 3);
    ob[i] = ((uint32_t)(row < last_n ? row : last_n) * (uint32_t)K + (uint32_t)((lane & 7) ^ swz16(row & 15)) * 8u) * 2u;
  }
  const auto load = [&](auto ic, uint32_t st) {   // load i of the slab at xk / wk, into the slab buffer at byte st
    constexpr int i = decltype(ic)::value;
    char* const dst = reinterpret_cast<char*>(smem) + st;
    if constexpr (i < GA)
      __builtin_amdgcn_global_load_lds((ring_gptr_t)(xk + oa[i]), (ring_lptr_t)(dst + (wave + i * kRingWaves) * 1024), 16, 0, 0);
    else
      __builtin_amdgcn_global_load_lds((ring_gptr_t)(wk + ob[i - GA]),
                                       (ring_lptr_t)(dst + BM * 128 + (wave + (i - GA) * kRingWaves) * 1024), 16, 0, 0);
  };

  // operand fragments of step ks of a slab: lane l holds row l % 16, chunk 4 ks + l / 16; tile t adds t * 2048
  const int lrow = lane & 15, lq = lane >> 4;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(ring_lptr_t)smem;
  uint32_t aaddr[2], baddr[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const uint32_t chunk = (uint32_t)((ks * 4 + lq) ^ swz16(lrow)) * 16u;
    aaddr[ks] = lds0 + (uint32_t)(wm0 + lrow) * 128u + chunk;
    baddr[ks] = lds0 + (uint32_t)(BM + wn0 + lrow) * 128u + chunk;
  }

  // The compiler sees no MFMA (asm statements) and adds no wait states between a register write and an MFMA that reads
  // it: the zeros are written here, before the prologue's loads and barrier.
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));

  // prologue: the first S slabs requested, the first one waited for, its first operands read
  uint32_t st = 0;
  for (int u = 0; u < S && u < KT; ++u) {
    each<G>([&](auto i) { load(i, st); });
    st += kSlab;
    xk += 128;
    wk += 128;
  }
  if (KT >= S) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 1) * G) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  vec8<E> fa[2][TM], fb[2][TN];
#pragma unroll
  for (int t = 0; t < TM; ++t) RING_READ(fa[0][t], aaddr[0], t * 2048);
#pragma unroll
  for (int t = 0; t < TN; ++t) RING_READ(fb[0][t], baddr[0], t * 2048);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");

  // One step of 32 k: the MFMAs of operand set P, rows of tiles walked back and forth (consecutive MFMAs share an
  // operand: less power); behind the first of them the reads of set 1 - P (READ); over all of them, spread evenly, half of
  // a slab's loads (LOAD 1, 2: which; 0: none).  A load occupies the CU's one load path for 16 cycles, so a slab's loads all in
  // one step would wait for it, and the MFMAs behind them with them.
  const auto step = [&](auto Pc, auto READc, auto LOADc, uint32_t ra, uint32_t rb, uint32_t st_load) {
    constexpr int P = decltype(Pc)::value, NM = TM * TN, NR = TM + TN, LOAD = decltype(LOADc)::value;
    constexpr bool READ = decltype(READc)::value;
    constexpr int from = LOAD == 2 ? (G + 1) / 2 : 0, count = LOAD == 2 ? G - from : (G + 1) / 2;
    static_assert(count <= NM, "a load behind every MFMA at most");
    each<NM>([&](auto ic) {
      constexpr int I = decltype(ic)::value, i = I / TN, j = (i & 1) ? TN - 1 - I % TN : I % TN;
      RING_MFMA(acc[i][j], fa[P][i], fb[P][j]);
      if constexpr (READ && I < NR) {
        if constexpr (I == 0) RING_READ(fa[1 - P][0], ra, 0);
        else if constexpr (I <= TN) RING_READ(fb[1 - P][I - 1], rb, (I - 1) * 2048);
        else RING_READ(fa[1 - P][I - TN], ra, (I - TN) * 2048);
      }
      constexpr int l = I * count / NM;
      if constexpr (LOAD != 0 && (I + 1) * count / NM > l) load(std::integral_constant<int, from + l>{}, st_load);
    });
  };
  using Yes = std::true_type;
  using No = std::false_type;
  using Set0 = std::integral_constant<int, 0>;
  using Set1 = std::integral_constant<int, 1>;
  using Half1 = std::integral_constant<int, 1>;
  using Half2 = std::integral_constant<int, 2>;

  st = 0;   // the current slab's buffer
  const auto after = [&](uint32_t s) { s += kSlab; return s == S * kSlab ? 0u : s; };
  // Between the steps of a slab: the reads of its second operands are back and, of this wavefront's loads, all but those of
  // the `behind` slabs behind the next one (loads return in order).
  const auto meet = [&](int behind) {
    if (S >= 5 && behind >= 3) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(3 * G) : "memory");
    else if (S >= 4 && behind >= 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * G) : "memory");
    else if (S >= 3 && behind >= 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(G) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
  };
  int32_t kt = 0;
  step(Set0{}, Yes{}, No{}, aaddr[1], baddr[1], 0);
  for (; kt + S < KT; ++kt) {
    meet(S - 2);
    const uint32_t free = st;   // slab kt's place takes slab kt + S
    st = after(st);
    step(Set1{}, Yes{}, Half1{}, aaddr[0] + st, baddr[0] + st, free);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    step(Set0{}, Yes{}, Half2{}, aaddr[1] + st, baddr[1] + st, free);
    xk += 128;
    wk += 128;
  }
  for (; kt + 1 < KT; ++kt) {   // the last S slabs: nothing left to request
    meet(KT - 2 - kt);
    st = after(st);
    step(Set1{}, Yes{}, No{}, aaddr[0] + st, baddr[0] + st, 0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    step(Set0{}, Yes{}, No{}, aaddr[1] + st, baddr[1] + st, 0);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  step(Set1{}, No{}, No{}, 0, 0, 0);
  // the matrix cores run empty before the compiler, which knows of no MFMA in flight, touches an accumulator
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));

  // Epilogue: PR row tiles at a time through this wavefront's part of the LDS; a lane then owns 8 consecutive columns of
  // a row.  What the rows need from memory is requested before the staging.
  constexpr int LD = ring_stage_ld(TN), PR = ring_rows_staged(TM, TN, S), PASSES = TM / PR;
  constexpr int LPR = TN * 2, RPI = 64 / LPR;            // lanes per row, rows per iteration
  constexpr int IT = (PR * 16 + RPI - 1) / RPI;
  int lane_e = lane;   // nothing of the epilogue above the loop
  asm volatile("" : "+v"(lane_e));
  float* const stage = reinterpret_cast<float*>(smem) + wave * (PR * 16 * LD);
  const int er = lane_e & 15, eq = lane_e >> 4;
  const int c8 = (lane_e % LPR) * 8, r0 = lane_e / LPR;
  const int32_t col = n0 + wn0 + c8;
  const bool col_ok = col < N && r0 < RPI;   // N % 8 == 0: whole chunks
  float bv[8], cv[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) bv[q] = cv[q] = 0.f;
  if (MODE == 1 && col_ok) {
#pragma unroll
    for (int q = 0; q < 8; ++q) { bv[q] = lf.bias[col + q]; cv[q] = lf.colsum[col + q]; }
  }
  if (MODE == 0 && bias != nullptr && col_ok) {
    const vec8<E> b8 = *reinterpret_cast<const vec8<E>*>(bias + col);
#pragma unroll
    for (int q = 0; q < 8; ++q) bv[q] = static_cast<float>(b8[q]);
  }
  const bool residual = MODE == 0 && epi == EPI_BIAS_RESIDUAL;
  const bool gelu = MODE == 0 ? epi == EPI_BIAS_GELU : MODE == 1 && epi == EPI_LNFOLD_GELU;
  __syncthreads();   // the slabs are no longer read
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    const int64_t mp = m0 + wm0 + pass * (PR * 16);
    vec8<E> rpre[IT];
    float2 spre[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int r = it * RPI + r0;
      const bool ok = col_ok && r < PR * 16 && mp + r < M;
      if (residual && ok) rpre[it] = *reinterpret_cast<const vec8<E>*>(res + (size_t)(mp + r) * N + col);
      if (MODE == 1 && ok) spre[it] = *reinterpret_cast<const float2*>(lf.stats + 2 * (mp + r));
    }
#pragma unroll
    for (int ii = 0; ii < PR; ++ii)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) stage[(ii * 16 + eq * 4 + e) * LD + j * 16 + er] = acc[pass * PR + ii][j][e];
    __builtin_amdgcn_wave_barrier();   // a wavefront's LDS accesses stay in order
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int r = it * RPI + r0;
      if (!(col_ok && r < PR * 16 && mp + r < M)) continue;
      const float4 lo = *reinterpret_cast<const float4*>(&stage[r * LD + c8]);
      const float4 hi = *reinterpret_cast<const float4*>(&stage[r * LD + c8 + 4]);
      const size_t off = (size_t)(mp + r) * N + col;
      if constexpr (MODE == 2) {
        float* const p = lf.partial + (size_t)part * M * N + off;
        *reinterpret_cast<float4*>(p) = lo;
        *reinterpret_cast<float4*>(p + 4) = hi;
      } else {
        float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        if constexpr (MODE == 1) {   // r (v - mu c) + b
          const float rmu = spre[it].y * spre[it].x;
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] = fmaf(spre[it].y, v[q], fmaf(-rmu, cv[q], bv[q]));
        } else {
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] += bv[q];
        }
        if (gelu) {
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] = gelu_erf(v[q]);
        }
        if (residual) {
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] += static_cast<float>(rpre[it][q]);
        }
        vec8<E> o;
#pragma unroll
        for (int q = 0; q < 8; ++q) o[q] = static_cast<E>(v[q]);
        *reinterpret_cast<vec8<E>*>(y + off) = o;
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

template <typename E, int TM, int TN, int S, int PER_CU, int MODE>
hipError_t launch_ring_cfg(const E* x, const E* w, const E* bias, const E* res, E* y, int64_t M, int32_t N, int32_t K, int epi,
                           const LnFold& lf, hipStream_t s, int32_t parts) {
  constexpr int BM = 32 * TM, BN = 32 * TN;
  auto kern = gemm_ring_kernel<E, TM, TN, S, PER_CU, MODE>;
  static LdsAttrOnce once;   // per element type and configuration
  hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), ring_lds(TM, TN, S), once);
  if (e != hipSuccess) return e;
  const int64_t tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  const int64_t grid = (tiles_m * tiles_n * parts + kXcds - 1) / kXcds * kXcds;
  if (grid * (kRingWaves * 64) > kMaxGridThreads) return hipErrorInvalidConfiguration;
  kern<<<dim3((unsigned)grid), dim3(kRingWaves * 64), ring_lds(TM, TN, S), s>>>(x, w, bias, res, y, M, N, K, epi, (int32_t)tiles_m,
                                                                               (int32_t)tiles_n, parts, lf);
  return hipGetLastError();
}

#undef RING_READ
#undef RING_MFMA

template <typename E, int MODE>
hipError_t launch_ring_mode(int shape, const E* x, const E* w, const E* bias, const E* res, E* y, int64_t M, int32_t N, int32_t K,
                            int epi, const LnFold& lf, hipStream_t s, int32_t parts) {
  switch (shape) {   // the order of kRingShapes
    case 0: return launch_ring_cfg<E, 2, 2, 5, 2, MODE>(x, w, bias, res, y, M, N, K, epi, lf, s, parts);
    case 1: return launch_ring_cfg<E, 2, 3, 4, 2, MODE>(x, w, bias, res, y, M, N, K, epi, lf, s, parts);
    case 2: return launch_ring_cfg<E, 3, 3, 3, 2, MODE>(x, w, bias, res, y, M, N, K, epi, lf, s, parts);
    case 3: return launch_ring_cfg<E, 3, 4, 5, 1, MODE>(x, w, bias, res, y, M, N, K, epi, lf, s, parts);
    case 4: return launch_ring_cfg<E, 4, 4, 5, 1, MODE>(x, w, bias, res, y, M, N, K, epi, lf, s, parts);
    case 5: return launch_ring_cfg<E, 4, 4, 2, 2, MODE>(x, w, bias, res, y, M, N, K, epi, lf, s, parts);
    case 6: return launch_ring_cfg<E, 3, 6, 4, 1, MODE>(x, w, bias, res, y, M, N, K, epi, lf, s, parts);
    case 7: return launch_ring_cfg<E, 4, 6, 4, 1, MODE>(x, w, bias, res, y, M, N, K, epi, lf, s, parts);
    case 8: return launch_ring_cfg<E, 5, 6, 3, 1, MODE>(x, w, bias, res, y, M, N, K, epi, lf, s, parts);
    case 9: return launch_ring_cfg<E, 4, 8, 3, 1, MODE>(x, w, bias, res, y, M, N, K, epi, lf, s, parts);
    case 10: return launch_ring_cfg<E, 5, 8, 3, 1, MODE>(x, w, bias, res, y, M, N, K, epi, lf, s, parts);
  }
  return hipErrorInvalidValue;
}
static_assert(kRingCount == 11 && kRingShapes[5].per_cu == 2 && kRingShapes[7].cols == 192 && kRingShapes[10].rows == 160, "order of launch_ring_mode");

}  // namespace

template <typename E>
hipError_t launch_gemm_ring(int shape, const E* x, const E* w, const E* bias, const E* res, E* y, int64_t M, int32_t N, int32_t K,
                            int epi, const LnFold& lf, hipStream_t s, int32_t parts, float* scratch) {
  if (parts > 1) {
    LnFold sums;
    sums.partial = scratch;
    const hipError_t e = launch_ring_mode<E, 2>(shape, x, w, bias, res, y, M, N, K, epi, sums, s, parts);
    return e != hipSuccess ? e : launch_partial_reduce<E>(scratch, parts, bias, res, y, M, N, epi, s);
  }
  if (epi == EPI_LNFOLD || epi == EPI_LNFOLD_GELU) return launch_ring_mode<E, 1>(shape, x, w, bias, res, y, M, N, K, epi, lf, s, 1);
  return launch_ring_mode<E, 0>(shape, x, w, bias, res, y, M, N, K, epi, lf, s, 1);
}
template hipError_t launch_gemm_ring<bf16_t>(int, const bf16_t*, const bf16_t*, const bf16_t*, const bf16_t*, bf16_t*, int64_t,
                                             int32_t, int32_t, int, const LnFold&, hipStream_t, int32_t, float*);
template hipError_t launch_gemm_ring<f16_t>(int, const f16_t*, const f16_t*, const f16_t*, const f16_t*, f16_t*, int64_t, int32_t,
                                            int32_t, int, const LnFold&, hipStream_t, int32_t, float*);

}  // namespace energon
