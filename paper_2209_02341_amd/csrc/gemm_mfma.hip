// 16-bit (bf16 or fp16) linear layer  y[M,N] = epilogue(x[M,K] W[N,K]^T + b)  on packed rows: the dense
// contractions that the paper (Sec. 3.1, Sec. 5.5) reports as >95 % of a large layer's time
// and that the padding removal (Sec. 4.3) shrinks from B*S rows to T rows.
//
// Design for gfx950:
//  * both operands are contiguous along K, so x rows feed the MFMA A operand and W rows the
//    B operand with the same 16-byte chunks; fp32 accumulators;
//  * a BM x BN output tile per workgroup, K walked in slabs of 64 (128 bytes per row), two
//    slab buffers in LDS, filled straight from global memory (global_load_lds_dwordx4);
//  * an LDS row is 8 chunks of 16 bytes; chunk c of row r is stored in slot c ^ swizzle(r), chosen
//    per MFMA form so that a wavefront's operand read meets no bank conflict (measured).  Slabs
//    are moved in 1 KiB groups = 8 rows x 8 slots in lane order, the lane that lands in slot s of
//    row r fetching chunk s ^ swizzle(r): full 128-byte lines on the global side;
//  * workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2, so the id is
//    remapped to give every XCD a contiguous run of tiles, ordered in bands of 8 row tiles:
//    the 32 tiles resident on an XCD form an 8 x 4 block that shares x and W slabs in that L2;
//  * epilogue in fp32: + bias, GeLU(erf) or + residual, one rounding to the storage type.
// The kernel here, gemm_mfma_sched_kernel, takes problems of whole rounds of 256x256 tiles: 4 wavefronts x 128x128 = 8 x 8
// tiles of v_mfma_f32_16x16x32 with the 256 accumulators in AGPRs; the slab loop is hand-scheduled (MFMA, LDS reads and the next
// slab's loads interleaved in asm); edge tiles are shifted inwards, so nothing is clamped or predicated; the epilogue goes
// through LDS and leaves as 16-byte non-temporal stores.  Smaller ones: gemm_ring.hip, gemm_ksplit.hip.
// tile_plan chooses between those and this kernel with every tile cut along K, ring_instead between it and the ring for one or two rounds.
#include "common.h"
#include <algorithm>
#include <cmath>
#include <vector>

namespace energon {

constexpr int BK = 64;            // K elements per slab
constexpr int kChunks = BK / 8;   // 16-byte chunks per LDS row

typedef __attribute__((address_space(1))) const void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// Epilogue of one wavefront's 128x128 tile (8 x 8 accumulator tiles of 16x16; in each the lane
// holds column lane % 16, rows 4 * (lane / 16) + e) through LDS, for tiles that lie wholly
// inside the matrix.  The accumulators go to LDS as fp32, 64 rows at a time, rows padded to 132
// floats so that the four lane groups of a store (4 rows apart) hit different banks; each lane
// then owns 8 consecutive columns of a row: bias, GeLU / residual are applied there in fp32 and the
// row segment leaves as one 16-byte store, 16 lanes per 256-byte row segment.  One rounding,
// full-line writes, marked non-temporal: y is not read again by this kernel and would only push
// x / W slabs out of the L2 (measured: 1.4 % faster).
constexpr int kEpiLd = 132;
constexpr int kEpiWaveFloats = 64 * kEpiLd;

// Sum over the 16 lanes of a DPP row (lanes 16 k .. 16 k + 15), left in every one of them:
// neighbour, other pair of the quad, other quad of the half row, other half row.
__device__ __forceinline__ float row16_sum(float v) {
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xF, 0xF, true));  // row_half_mirror
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xF, 0xF, true));  // row_mirror
  return v;
}

// MODE selects what is compiled in, so that each instantiation carries only the registers of the
// epilogues it serves (compiled all together they push a hundred accumulators out to scratch memory
// after every tile):
//   0  the plain epilogues (bias, bias + GeLU, bias + residual);
//   1  the LayerNorm-folded epilogues (EPI_LNFOLD, EPI_LNFOLD_GELU): row statistics read, no residual;
//   2  bias + residual with the row statistics of the rounded result written to lf.partial.
constexpr int kEpiPlain = 0, kEpiFolded = 1, kEpiResidualStats = 2;
template <typename E, int MODE>
__device__ __forceinline__ void store_tile_coalesced(const f32x4 (&acc)[8][8], const E* __restrict__ bias,
                                                     const E* res, E* y, int32_t N, int epi, int64_t mw,
                                                     int32_t nw, int lane, float* stage, const LnFold& lf,
                                                     float* raw = nullptr) {
  // raw (plain mode only): the workgroup holds a piece of a tile cut along K; its fp32 sums go, without
  // any epilogue, to raw[256][256] (row-major, this wavefront's quadrant at the offsets it has in the
  // tile), through the same staging, 32 bytes per lane and row.
  constexpr bool fold = MODE == kEpiFolded;
  constexpr bool stats = MODE == kEpiResidualStats;
  const bool residual = MODE == kEpiResidualStats || (MODE == kEpiPlain && epi == EPI_BIAS_RESIDUAL);
  const bool gelu = MODE == kEpiFolded ? epi == EPI_LNFOLD_GELU : (MODE == kEpiPlain && epi == EPI_BIAS_GELU);
  const int lrow = lane & 15, lq = lane >> 4;
  const int rr = lane >> 4, c8 = (lane & 15) * 8;
  float bv[8], cv[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) cv[q] = 0.f;
  if (fold) {
    const float4 b0 = *reinterpret_cast<const float4*>(lf.bias + nw + c8), b1 = *reinterpret_cast<const float4*>(lf.bias + nw + c8 + 4);
    const float4 c0 = *reinterpret_cast<const float4*>(lf.colsum + nw + c8), c1 = *reinterpret_cast<const float4*>(lf.colsum + nw + c8 + 4);
    bv[0] = b0.x; bv[1] = b0.y; bv[2] = b0.z; bv[3] = b0.w; bv[4] = b1.x; bv[5] = b1.y; bv[6] = b1.z; bv[7] = b1.w;
    cv[0] = c0.x; cv[1] = c0.y; cv[2] = c0.z; cv[3] = c0.w; cv[4] = c1.x; cv[5] = c1.y; cv[6] = c1.z; cv[7] = c1.w;
  } else if (bias != nullptr) {
    const vec8<E> b8 = *reinterpret_cast<const vec8<E>*>(bias + nw + c8);
#pragma unroll
    for (int q = 0; q < 8; ++q) bv[q] = static_cast<float>(b8[q]);
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) bv[q] = 0.f;
  }
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    // What the rows of this pass need from global memory (residual segments, row statistics) is
    // requested before the staging, so that its latency passes behind the barriers and the LDS
    // traffic instead of stalling every row of the loop below.
    vec8<E> rpre[16];
    float2 spre[16];
    if (residual && raw == nullptr) {
#pragma unroll
      for (int it = 0; it < 16; ++it)
        rpre[it] = *reinterpret_cast<const vec8<E>*>(res + (size_t)(mw + pass * 64 + it * 4 + rr) * N + nw + c8);
    }
    if (fold) {
#pragma unroll
      for (int it = 0; it < 16; ++it)
        spre[it] = *reinterpret_cast<const float2*>(lf.stats + 2 * (mw + pass * 64 + it * 4 + rr));
    }
    __syncthreads();  // the slab buffers (first pass) / the previous pass's rows are no longer read
#pragma unroll
    for (int ii = 0; ii < 4; ++ii)
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          stage[(ii * 16 + lq * 4 + e) * kEpiLd + j * 16 + lrow] = acc[pass * 4 + ii][j][e];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < 16; ++it) {
      const int r = it * 4 + rr;
      const float4 lo = *reinterpret_cast<const float4*>(&stage[r * kEpiLd + c8]);
      const float4 hi = *reinterpret_cast<const float4*>(&stage[r * kEpiLd + c8 + 4]);
      if (MODE == kEpiPlain && raw != nullptr) {
        float* dst = raw + (size_t)(pass * 64 + r) * 256 + c8;
        *reinterpret_cast<float4*>(dst) = lo;
        *reinterpret_cast<float4*>(dst + 4) = hi;
        continue;
      }
      float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      const size_t off = (size_t)(mw + pass * 64 + r) * N + nw + c8;
      if (fold) {  // r (v - mu c) + b as two multiply-adds
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
      __builtin_nontemporal_store(o, reinterpret_cast<vec8<E>*>(y + off));
      if (stats) {  // the 16 lanes of this row hold one 128-column segment of it
        float s1 = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) s1 += static_cast<float>(o[q]);
        s1 = row16_sum(s1);
        const float seg_mean = s1 * (1.0f / kStatSeg);
        float s2 = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) { const float d = static_cast<float>(o[q]) - seg_mean; s2 += d * d; }
        s2 = row16_sum(s2);
        if ((lane & 15) == 0)
          *reinterpret_cast<float2*>(lf.partial + ((size_t)(mw + pass * 64 + r) * (N / kStatSeg) + nw / kStatSeg) * 2) =
              make_float2(s1, s2);
      }
    }
  }
}

// ---- hand-scheduled 256x256 kernel ----------------------------------------------------------
// Work decomposition.  The kernel is persistent: 8 * wgs workgroups (one per CU: 128 KiB of LDS each),
// workgroup id b running on XCD b % 8 as its workgroup j = b / 8.  Every XCD owns a fixed sequence
// of tiles, and its workgroups walk it in rounds: workgroup j takes tiles j, j + wgs, j + 2 wgs, ...
// so the tiles resident on an XCD at one time are wgs consecutive ones of its sequence, a compact
// block that shares x and W slabs in that XCD's L2.
//   raster 0: the tiles in bands of kGroupM row tiles, column by column inside a band, cut in 8 equal
//             runs, one per XCD (resident block: 8 x 4 tiles);
//   raster 1: XCD x owns row tiles [x R, (x + 1) R), R = tiles_m / 8, walked in bands of at most
//             kGroupM rows, column by column inside a band (resident block: min(R, 8) rows x wgs /
//             min(R, 8) columns), all XCDs moving through the columns of W together, so that a W slab
//             comes from HBM once and reaches the other seven L2s from the memory-side cache; the
//             tiles_m % 8 leftover row tiles are dealt column-wise, 1/8 to each XCD, at the end.
// With pieces = P > 1 the tiles of an XCD beyond its last full round (fewer than wgs) are not run as
// one more, partly empty round: each is cut along K into P chunks of the same even length (the last
// one shorter), chunk borders at the same slabs for every tile, and the rem * P pieces are dealt to
// the XCD's workgroups chunk by chunk (piece q = chunk * rem + tile, workgroup j takes q = j, j + wgs,
// ...).  Workgroups of a round thus walk the same slabs at the same time and keep sharing x and W
// slabs in the L2, as whole tiles do.  (Cutting the remainder's slabs into wgs equal contiguous
// shares, the textbook stream-K cut, balances better but starts every workgroup at a different K
// offset: measured on the tensor-parallel shard's QKV shape it took the L2 hit rate down far enough
// to make the launch 1.7 times slower than with whole tiles.)  A piece leaves its fp32 accumulators
// (row-major 256 x 256) in the caller's scratch, slot tile * P + chunk of its XCD; a second kernel adds the P pieces of
// every cut tile in ascending K order and applies the epilogue: deterministic, no atomics, no
// workgroup waits for another.  The tail of a launch is then a short, well filled round instead of
// a long, partly empty one: that matters where a tile is long and rounds are few (the
// tensor-parallel shard: 312 tiles of 192 slabs on 256 CUs).
struct SchedPlan {
  int32_t tiles_m, tiles_n, kt;   // kt: slabs of 64 along K per tile
  int32_t wgs;                    // workgroups per XCD
  int32_t raster;                 // 0 / 1, see above
  int32_t pieces;                 // P: 1 = remainder tiles run whole
  int32_t slots;                  // room for pieces in the scratch, per XCD
};
struct XcdShare { int32_t n_tiles, dp_rounds, rem, chunk; };   // chunk: slabs per piece

__host__ __device__ inline int32_t sched_chunk(int32_t kt, int32_t pieces) {
  int32_t c = (kt + pieces - 1) / pieces;
  return c + (c & 1);
}

__host__ __device__ inline XcdShare xcd_share(const SchedPlan& p, int32_t x) {
  XcdShare s;
  if (p.raster == 1) {
    const int32_t rows = p.tiles_m / kXcds, left = (p.tiles_m - kXcds * rows) * p.tiles_n;
    const int32_t q = (left + kXcds - 1) / kXcds;
    const int32_t mine = left - x * q;
    s.n_tiles = rows * p.tiles_n + (mine < 0 ? 0 : (mine > q ? q : mine));
  } else {
    const int32_t total = p.tiles_m * p.tiles_n, per = (total + kXcds - 1) / kXcds;
    const int32_t mine = total - x * per;
    s.n_tiles = mine < 0 ? 0 : (mine > per ? per : mine);
  }
  if (p.pieces > 1) {
    s.dp_rounds = s.n_tiles / p.wgs;
    s.rem = s.n_tiles - s.dp_rounds * p.wgs;
    s.chunk = sched_chunk(p.kt, p.pieces);
  } else {
    s.dp_rounds = (s.n_tiles + p.wgs - 1) / p.wgs;   // the last one possibly not full
    s.rem = 0;
    s.chunk = p.kt;
  }
  return s;
}

// Tile l of XCD x's sequence -> (row tile, column tile).
__host__ __device__ inline void sched_tile(const SchedPlan& p, int32_t x, int32_t l, int32_t& tm, int32_t& tn) {
  if (p.raster == 1) {
    const int32_t rows = p.tiles_m / kXcds, main_n = rows * p.tiles_n;
    if (l < main_n) {   // the XCD's rows in bands of kGroupM, column by column inside a band
      const int32_t band = l / (kGroupM * p.tiles_n);
      const int32_t first = band * kGroupM;
      const int32_t band_m = rows - first < kGroupM ? rows - first : kGroupM;
      const int32_t r = l - band * kGroupM * p.tiles_n;
      tn = r / band_m;
      tm = x * rows + first + (r - tn * band_m);
    } else {
      const int32_t left_rows = p.tiles_m - kXcds * rows;
      const int32_t q = (left_rows * p.tiles_n + kXcds - 1) / kXcds;
      const int32_t g = x * q + (l - main_n);
      tn = g / left_rows;
      tm = kXcds * rows + (g - tn * left_rows);
    }
  } else {
    const int32_t total = p.tiles_m * p.tiles_n, per = (total + kXcds - 1) / kXcds;
    const int32_t idx = x * per + l;
    const int32_t band = idx / (kGroupM * p.tiles_n);
    const int32_t first_m = band * kGroupM;
    const int32_t band_m = p.tiles_m - first_m < kGroupM ? p.tiles_m - first_m : kGroupM;
    const int32_t r = idx - band * kGroupM * p.tiles_n;
    tn = r / band_m;
    tm = first_m + (r - tn * band_m);
  }
}

// The work of workgroup `wg` of XCD `xcd`, in the order it is done: whole tiles first, then pieces of
// the XCD's cut tiles.  next() yields tile l of the XCD's sequence, the slabs [kb, kb + n) of it, and
// the scratch slot of the piece inside the XCD's slots (-1: the whole tile, finished by this
// workgroup).  Shared by the kernel and the host-side check of the decomposition.
struct SchedWalker {
  XcdShare share;
  int32_t wgs, wg, kt, pieces, n_whole, n_chunks, q_stop, done, q;
  __host__ __device__ SchedWalker(const SchedPlan& p, int32_t xcd, int32_t wg_) {
    share = xcd_share(p, xcd);
    wgs = p.wgs; wg = wg_; kt = p.kt; pieces = p.pieces;
    if (p.pieces > 1) n_whole = share.dp_rounds;
    else n_whole = share.n_tiles > wg ? (share.n_tiles - wg + wgs - 1) / wgs : 0;
    n_chunks = (kt + share.chunk - 1) / share.chunk;   // <= pieces
    q_stop = share.rem * n_chunks;
    done = 0;
    q = wg;
  }
  __host__ __device__ bool next(int32_t& l, int32_t& kb, int32_t& n, int32_t& slot) {
    if (done < n_whole) {
      l = done * wgs + wg;
      kb = 0;
      n = kt;
      slot = -1;
      ++done;
      return true;
    }
    if (q < q_stop) {
      const int32_t c = q / share.rem, t = q - c * share.rem;
      l = share.dp_rounds * wgs + t;
      kb = c * share.chunk;
      n = kt - kb < share.chunk ? kt - kb : share.chunk;
      slot = t * pieces + c;
      q += wgs;
      return true;
    }
    return false;
  }
};

constexpr int kPartFloats = 256 * 256;   // one piece's accumulators

// The slab loop is written as ordered inline-asm statements so that the issue order is exactly
// the one below (the compiler otherwise re-serialises LDS reads and MFMAs, and it must not copy
// or spill a register whose load is still in flight).  One wavefront per SIMD, 128x128 per
// wavefront = 8 x 8 tiles of v_mfma_f32_16x16x32_bf16 (measured on random operands under the
// chip's power limit: 16 % more flops per second than the 32x32x16 form).
// A slab of 64 along K is two MFMA steps of 32; a step is four quadrants of 16 MFMAs, one half
// (4 fragments) of the A operands against one half of the B operands.  There is ONE set of
// operand registers: the quadrants are walked in an order in which each half is released at
// least one quadrant before its successor is needed,
//   even step:  (aL,bL) (aL,bH) (aH,bH) (aH,bL)      odd step:  (aL,bH) (aL,bL) (aH,bL) (aH,bH)
// and every quadrant carries the 4 LDS reads that refill the half released last, 2 global loads
// and 2 LDS writes of staged chunks (see ENERGON_QUAD and ENERGON_SLAB): LDS and memory traffic
// is even over the loop.  One barrier per slab; a fetched chunk has 1.75 slab times to arrive.
// What the compiler cannot see inside asm statements it cannot guard: this code itself keeps
// the wait states between an MFMA and the first read of its result (end of the slab loop) and
// between a register write and an MFMA reading it (accumulator zeroing).
#define ENERGON_DS_READ(dst, addr, off) \
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(off) : "memory")
#define ENERGON_MFMA(acc, a, b)                                                                          \
  do {                                                                                                   \
    if constexpr (__is_same(E, bf16_t))                                                                  \
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));              \
    else                                                                                                 \
      asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));               \
  } while (0)

template <typename E, int BM, int BN, int WM, int WN, int MODE>
__global__ __launch_bounds__(WM* WN * 64) void gemm_mfma_sched_kernel(const E* __restrict__ x,
                                                                    const E* __restrict__ w,
                                                                    const E* __restrict__ bias,
                                                                    const E* res, E* y, int64_t M,
                                                                    int32_t N, int32_t K, int epi, SchedPlan plan,
                                                                    float* __restrict__ part, LnFold lf) {
  constexpr int NW = WM * WN;
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int TM = WTM / 16, TN = WTN / 16;
  constexpr int GA = BM / 8 / NW, GB = BN / 8 / NW;
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "row groups must divide evenly");
  static_assert((BM + BN) * 128 == 65536, "stage stride is assumed to be 64 KiB");
  static_assert(TM == 8 && TN == 8 && GA + GB == 16, "the hand schedule is written for 4 x (128x128)");
  static_assert(BM * BN == kPartFloats, "a piece's accumulators");
  extern __shared__ uint4 smem[];  // [2][BM + BN][kChunks]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform, kept in an SGPR
  const int wm0 = (wave / WN) * WTM, wn0 = (wave % WN) * WTN;

  // This workgroup's share: whole tiles first, then its pieces of the XCD's cut tiles.
  const int32_t xcd = blockIdx.x % kXcds;
  SchedWalker walk(plan, xcd, blockIdx.x / kXcds);

  for (;;) {
    // ---- next piece of work: tile l of the XCD's sequence, slabs [kb, kb + KT) of it ----
    int32_t l, kb, KT, slot;
    if (!walk.next(l, kb, KT, slot)) break;
    // non-null: the piece does not cover its tile
    float* const piece_out = slot < 0 ? nullptr : part + ((size_t)xcd * plan.slots + (size_t)slot) * kPartFloats;
    int32_t tm, tn;
    sched_tile(plan, xcd, l, tm, tn);
    int64_t m0 = (int64_t)tm * BM;
    int32_t n0 = tn * BN;
    // Ragged edges: the last tile of a row / column of tiles is shifted back so that it ends at
    // M / N (needs M >= BM, N >= BN).  It overlaps its neighbour; both compute bit-identical values
    // for the shared elements, so no load is clamped and no store is predicated.
    if (m0 > M - BM) m0 = M - BM;
    if (n0 > N - BN) n0 = N - BN;

    // Per-lane addresses are derived afresh for every piece from an opaque copy of the lane id: kept
    // alive across the epilogue instead, they would cost it registers it does not have.
    int lane_i = lane;
    asm volatile("" : "+v"(lane_i));
    // MFMA operand fragment of a 16-row tile for the step ks (32 along K = chunks 4 ks .. 4 ks + 3
    // of the slab row): lane l holds row l % 16, chunk 4 ks + l / 16.  LDS byte address of that
    // chunk for tile 0; tile t adds t * 2048 (16 rows), and swz depends on row % 16 only.
    const int lrow = lane_i & 15, lq = lane_i >> 4;
    uint32_t aaddr[2], baddr[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const uint32_t chunk = (uint32_t)((ks * 4 + lq) ^ swz16(lrow)) * 16u;
      aaddr[ks] = (uint32_t)(wm0 + lrow) * 128u + chunk;
      baddr[ks] = (uint32_t)(BM + wn0 + lrow) * 128u + chunk;
    }
    // Slab loads go straight from global memory to LDS (global_load_lds_dwordx4: no staging
    // register, no LDS store instruction; LDS stores from registers would occupy the LDS pipeline
    // longer than all the operand reads).  One instruction moves a row group: 8 rows x 128 bytes =
    // 1 KiB of LDS in lane order, lane l landing in slot l % 8 of row l / 8 and fetching the chunk
    // that the swizzle puts there.  The 64 row groups of a slab fall in four classes by the operand
    // half that reads them -- AL / AH: x rows 0..63 / 64..127 of each wavefront row, BL / BH likewise
    // for W -- and every wavefront moves 4 groups of each class, of its own parity (swz(row) depends
    // on row % 16 = 8 * (group parity) + l / 8, so one per-lane offset serves all its groups).
    const uint32_t voff = ((uint32_t)(lane_i >> 3) * (uint32_t)K +
                           (uint32_t)(((lane_i & 7) ^ swz16((wave & 1) * 8 + (lane_i >> 3))) * 8)) * 2u;

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
    // The compiler sees no MFMA (they are inside asm statements) and so adds no wait states between
    // a register write and an MFMA that reads it: have the zeros written here, before the prologue.
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));

    const char* gsrc[4][4];  // [class AL, BH, BL, AH][j]: global address of the group's first row, slab kb
    uint32_t ldst[4][4];     // its LDS byte offset in buffer 0
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool is_a = (c == 0 || c == 3), high = (c == 1 || c == 3);
        const int gl = 2 * ((wave >> 1) * 4 + j) + (wave & 1);           // 0..15 within the class
        const int g = gl + (gl >= 8 ? 8 : 0) + (high ? 8 : 0);            // row group within the operand's 32
        gsrc[c][j] = reinterpret_cast<const char*>((is_a ? x + (size_t)m0 * K : w + (size_t)n0 * K) + (size_t)(8 * g) * K) +
                     (size_t)kb * (BK * 2);
        ldst[c][j] = (uint32_t)((is_a ? 0 : BM * 128) + g * 1024);
      }
#define ENERGON_DMA(c, j, kt_, buf)                                                                     \
  __builtin_amdgcn_global_load_lds((gptr_t)(gsrc[c][j] + (size_t)(kt_) * (BK * 2) + voff),              \
                                   (lptr_t)(reinterpret_cast<char*>(smem) + (buf) * 0x10000 + ldst[c][j]), 16, 0, 0)

    vec8<E> fa[TM], fb[TN];  // the operand fragments: x-row tiles, W-row tiles
#define ENERGON_RA(t, ks) ENERGON_DS_READ(fa[t], aaddr[ks], (t) * 2048)
#define ENERGON_RB(t, ks) ENERGON_DS_READ(fb[t], baddr[ks], (t) * 2048)
#define ENERGON_MF(i, j) ENERGON_MFMA(acc[i][j], fa[i], fb[j])
#define ENERGON_NONE do { } while (0)
// Wait for this wavefront's LDS reads and for all but its newest `n` slab loads, then meet the
// other wavefronts: what they have read may now be overwritten, what they have fetched may be read.
#define ENERGON_SYNC(n)                                                   \
  do {                                                                    \
    asm volatile("s_waitcnt vmcnt(" #n ") lgkmcnt(0)" ::: "memory");      \
    __builtin_amdgcn_s_barrier();                                         \
  } while (0)

// One quadrant: the 16 MFMAs of A tiles ai..ai+3 against B tiles bj..bj+3 (rows walked back and
// forth, so that consecutive MFMAs share an operand: measurably less power) with, slotted between
// them, four LDS reads R0..R3 (fragments of a half that the previous quadrants have released) and
// up to four slab loads D0..D3; TAIL is the synchronisation that ends it (the reads are back on
// leaving in any case).
#define ENERGON_QUAD(ai, bj, R0, R1, R2, R3, D0, D1, D2, D3, TAIL)                              \
  do {                                                                                         \
    ENERGON_MF(ai + 0, bj + 0); R0; ENERGON_MF(ai + 0, bj + 1); R1;                             \
    ENERGON_MF(ai + 0, bj + 2); R2; ENERGON_MF(ai + 0, bj + 3); R3;                             \
    ENERGON_MF(ai + 1, bj + 3); D0; ENERGON_MF(ai + 1, bj + 2); D1;                             \
    ENERGON_MF(ai + 1, bj + 1); D2; ENERGON_MF(ai + 1, bj + 0); D3;                             \
    ENERGON_MF(ai + 2, bj + 0); ENERGON_MF(ai + 2, bj + 1); ENERGON_MF(ai + 2, bj + 2); ENERGON_MF(ai + 2, bj + 3); \
    ENERGON_MF(ai + 3, bj + 3); ENERGON_MF(ai + 3, bj + 2); ENERGON_MF(ai + 3, bj + 1); ENERGON_MF(ai + 3, bj + 0); \
    TAIL;                                                                                      \
  } while (0)
#define ENERGON_READS_BACK asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory")

    const int klast = KT - 1;
    // Prologue: slab 0 into buffer 0 (waited for), slab 1 into buffer 1 (in flight), the fragments
    // of the first quadrant in registers.  Load order within a slab is AL, BH, BL, AH throughout.
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) ENERGON_DMA(c, j, 0, 0);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) ENERGON_DMA(c, j, (1 < klast ? 1 : klast), 1);
    asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    ENERGON_RA(0, 0); ENERGON_RA(1, 0); ENERGON_RA(2, 0); ENERGON_RA(3, 0);
    ENERGON_RB(0, 0); ENERGON_RB(1, 0); ENERGON_RB(2, 0); ENERGON_RB(3, 0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");

    // Slab kt is consumed from buffer kt & 1 while slab kt+1 (other buffer) is landing.  Quadrants
    // 2, 3, 4, 5 hold the last reads of the classes AL, BH, BL, AH of slab kt; the barrier that
    // ends each of them frees that class's rows in the current buffer, and the loads of the same
    // class of slab kt+2 follow in the next two quadrants.  Reads of slab kt+1 start in quadrant 6
    // (AL), 7 (BL), then 0 (BH) and 1 (AH) of the next slab: the barriers ending quadrants 5, 6 and
    // 0 are preceded by waits for exactly those classes (loads return in order; the count is the
    // number of loads issued after the class's last).  A load thus has 8 to 10 quadrants, a good
    // slab time, to arrive, and loads are issued in every quadrant but three.
#define ENERGON_SLAB(kt_, cur, nxt)                                                                     \
  {                                                                                                     \
    const int kl2 = (kt_) + 2 < KT ? (kt_) + 2 : klast;                                                 \
    ENERGON_QUAD(0, 0, ENERGON_RB(4, 0), ENERGON_RB(5, 0), ENERGON_RB(6, 0), ENERGON_RB(7, 0),           \
                 ENERGON_NONE, ENERGON_NONE, ENERGON_NONE, ENERGON_NONE, ENERGON_SYNC(16));             \
    ENERGON_QUAD(0, 4, ENERGON_RA(4, 0), ENERGON_RA(5, 0), ENERGON_RA(6, 0), ENERGON_RA(7, 0),           \
                 ENERGON_NONE, ENERGON_NONE, ENERGON_NONE, ENERGON_NONE, ENERGON_READS_BACK);           \
    ENERGON_QUAD(4, 4, ENERGON_RA(0, 1), ENERGON_RA(1, 1), ENERGON_RA(2, 1), ENERGON_RA(3, 1),           \
                 ENERGON_NONE, ENERGON_NONE, ENERGON_NONE, ENERGON_NONE, ENERGON_SYNC(16));             \
    ENERGON_QUAD(4, 0, ENERGON_RB(4, 1), ENERGON_RB(5, 1), ENERGON_RB(6, 1), ENERGON_RB(7, 1),           \
                 ENERGON_DMA(0, 0, kl2, cur), ENERGON_DMA(0, 1, kl2, cur), ENERGON_NONE, ENERGON_NONE,   \
                 ENERGON_SYNC(18));                                                                     \
    ENERGON_QUAD(0, 4, ENERGON_RB(0, 1), ENERGON_RB(1, 1), ENERGON_RB(2, 1), ENERGON_RB(3, 1),           \
                 ENERGON_DMA(0, 2, kl2, cur), ENERGON_DMA(0, 3, kl2, cur), ENERGON_DMA(1, 0, kl2, cur),  \
                 ENERGON_DMA(1, 1, kl2, cur), ENERGON_SYNC(22));                                        \
    ENERGON_QUAD(0, 0, ENERGON_RA(4, 1), ENERGON_RA(5, 1), ENERGON_RA(6, 1), ENERGON_RA(7, 1),           \
                 ENERGON_DMA(1, 2, kl2, cur), ENERGON_DMA(1, 3, kl2, cur), ENERGON_DMA(2, 0, kl2, cur),  \
                 ENERGON_DMA(2, 1, kl2, cur), ENERGON_SYNC(22));                                        \
    _Pragma("unroll") for (int ks = 0; ks < 2; ++ks) { aaddr[ks] ^= 0x10000u; baddr[ks] ^= 0x10000u; }  \
    ENERGON_QUAD(4, 0, ENERGON_RA(0, 0), ENERGON_RA(1, 0), ENERGON_RA(2, 0), ENERGON_RA(3, 0),           \
                 ENERGON_DMA(2, 2, kl2, cur), ENERGON_DMA(2, 3, kl2, cur), ENERGON_DMA(3, 0, kl2, cur),  \
                 ENERGON_DMA(3, 1, kl2, cur), ENERGON_SYNC(18));                                        \
    ENERGON_QUAD(4, 4, ENERGON_RB(0, 0), ENERGON_RB(1, 0), ENERGON_RB(2, 0), ENERGON_RB(3, 0),           \
                 ENERGON_DMA(3, 2, kl2, cur), ENERGON_DMA(3, 3, kl2, cur), ENERGON_NONE, ENERGON_NONE,   \
                 ENERGON_READS_BACK);                                                                   \
  }
    for (int kt = 0; kt < KT; kt += 2) {  // KT is even (K % 128 == 0 and chunks of even length)
      ENERGON_SLAB(kt, 0, 1)
      ENERGON_SLAB(kt + 1, 1, 0)
      // Last trip only: let the MFMA pipeline run empty before control leaves the loop.  Past this
      // point the compiler moves accumulators between registers as it pleases, and it knows of no
      // MFMA in flight (they are inside asm statements), so it would add none of the wait states
      // that a read of a matrix-core result needs.
      asm volatile("s_cmp_lt_i32 %0, %1\n\t"
                   "s_cbranch_scc1 .Lenergon_more_%=\n\t"
                   "s_nop 15\n\ts_nop 15\n\ts_nop 15\n"
                   ".Lenergon_more_%=:"
                   :
                   : "s"(kt + 2), "s"(KT)
                   : "scc", "memory");
    }
#undef ENERGON_SLAB
    // Outstanding loads (the clamped refetches of the last slabs) still write to LDS.
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
#undef ENERGON_DMA
#undef ENERGON_QUAD
#undef ENERGON_SYNC
#undef ENERGON_READS_BACK
#undef ENERGON_NONE
#undef ENERGON_RA
#undef ENERGON_RB
#undef ENERGON_MF

    // The epilogue's per-lane addresses must not be computed (and kept live) above the slab loop,
    // where every VGPR is spoken for: route the lane id through an ordered asm statement.
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));
    // a piece of a cut tile leaves its raw sums (piece_out != nullptr), everything else its results
    store_tile_coalesced<E, MODE>(acc, bias, res, y, N, epi, m0 + wm0, n0 + wn0, lane_e,
                                  reinterpret_cast<float*>(smem) + wave * kEpiWaveFloats, lf,
                                  piece_out != nullptr ? piece_out + (size_t)wm0 * 256 + wn0 : nullptr);
    // the slab buffers (or the staging rows over them) are reused by the next piece's first loads
    __syncthreads();
  }
}

// Second kernel of a launch that cut tiles.  A workgroup finishes 16 rows of one cut tile (16 strips
// per tile): every thread owns 8 consecutive columns of a row, adds the P pieces' sums for them in
// ascending K order (all loads issued before the first add), applies bias, GeLU / residual in fp32,
// rounds once and stores 16 bytes.  blockIdx.x % 8 is the XCD that wrote the pieces.
constexpr int kFixStrips = 16;
template <typename E>
__global__ __launch_bounds__(512) void gemm_mfma_fixup_kernel(const float* __restrict__ part,
                                                             const E* __restrict__ bias, const E* res, E* y,
                                                             int64_t M, int32_t N, int epi, SchedPlan plan) {
  const int32_t xcd = blockIdx.x % kXcds, rest = blockIdx.x / kXcds;
  const int32_t t = rest / kFixStrips, strip = rest % kFixStrips;
  const XcdShare share = xcd_share(plan, xcd);
  if (t >= share.rem) return;
  const int32_t n_chunks = (plan.kt + share.chunk - 1) / share.chunk;
  const int tid = threadIdx.x;
  const int r = strip * 16 + (tid >> 5), c8 = (tid & 31) * 8;   // row and first column inside the tile
  const float* src = part + ((size_t)xcd * plan.slots + (size_t)t * plan.pieces) * kPartFloats + (size_t)r * 256 + c8;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int32_t c0 = 0; c0 < n_chunks; c0 += 4) {   // four pieces' loads in flight at a time
    float4 lo[4], hi[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const bool live = c0 + c < n_chunks;
      const float* p = src + (size_t)(live ? c0 + c : c0) * kPartFloats;
      lo[c] = *reinterpret_cast<const float4*>(p);
      hi[c] = *reinterpret_cast<const float4*>(p + 4);
      if (!live) { lo[c] = make_float4(0.f, 0.f, 0.f, 0.f); hi[c] = lo[c]; }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      v[0] += lo[c].x; v[1] += lo[c].y; v[2] += lo[c].z; v[3] += lo[c].w;
      v[4] += hi[c].x; v[5] += hi[c].y; v[6] += hi[c].z; v[7] += hi[c].w;
    }
  }
  int32_t tm, tn;
  sched_tile(plan, xcd, share.dp_rounds * plan.wgs + t, tm, tn);
  int64_t m0 = (int64_t)tm * 256;
  int32_t n0 = tn * 256;
  if (m0 > M - 256) m0 = M - 256;
  if (n0 > N - 256) n0 = N - 256;
  const int32_t n = n0 + c8;
  if (bias != nullptr) {
    const vec8<E> b8 = *reinterpret_cast<const vec8<E>*>(bias + n);
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] += static_cast<float>(b8[q]);
  }
  if (epi == EPI_BIAS_GELU) {
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = gelu_erf(v[q]);
  }
  const size_t off = (size_t)(m0 + r) * N + n;
  if (epi == EPI_BIAS_RESIDUAL) {
    const vec8<E> r8 = *reinterpret_cast<const vec8<E>*>(res + off);
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] += static_cast<float>(r8[q]);
  }
  vec8<E> o;
#pragma unroll
  for (int q = 0; q < 8; ++q) o[q] = static_cast<E>(v[q]);
  *reinterpret_cast<vec8<E>*>(y + off) = o;
}

// The 256x256 kernel needs whole tiles to shift at the edges, an even number of slabs, and enough
// tiles for most of the 256 CUs.  Shifted edge tiles overlap their neighbours: with the residual
// aliasing y, an overlapped element could be read after the neighbour's write, so that case
// needs whole tiles.
static bool takes_sched_kernel(int64_t M, int32_t N, int32_t K, bool res_aliases_y) {
  const int64_t big_tiles = ((M + 255) / 256) * ((N + 255) / 256);
  const bool overlap_safe = !res_aliases_y || (M % 256 == 0 && N % 256 == 0);
  return M >= 256 && N >= 256 && K % 128 == 0 && big_tiles >= 192 && overlap_safe;
}

bool gemm_takes_whole_rounds(int64_t M, int32_t N, int32_t K) { return takes_sched_kernel(M, N, K, false); }

// Row partials come from the 256x256 kernel's epilogue, one per 128-column segment, and a
// shifted column tile would count its overlap twice: whole column tiles only.
bool gemm_emits_row_partials(int64_t M, int32_t N, int32_t K, bool res_aliases_y) {
  return takes_sched_kernel(M, N, K, res_aliases_y) && N % 256 == 0;
}

// Workgroups per XCD for the persistent 256x256 kernel: one per CU (MI355X: 256 CUs in 8 XCDs).
static int32_t sched_wgs_per_xcd() {
  static int32_t cached[32] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 32;
  const bool tracked = dev >= 0 && dev < 32;
  if (tracked && cached[dev] > 0) return cached[dev];
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < kXcds) cus = 256;
  const int32_t v = cus / kXcds;
  if (tracked) cached[dev] = v;
  return v;
}

// Decomposition of a launch of the 256x256 kernel.  Raster: a row band per XCD once every XCD gets
// at least two row tiles (all XCDs then stream the same W columns at the same time), band order
// otherwise.  Pieces: the P in 1..8 (P rem <= 2 wgs: the scratch has 2 wgs slots per XCD) with the
// least expected time, in slab units of a busy chip (a 256x256x64 slab step takes about 1.55 us
// under the sustained power limit): the remainder's rounds of pieces, plus, for P > 1, each piece's
// start-up and accumulator store and the second kernel (it reads every piece once at about 3 TB/s
// including its own stores, after a launch gap).  P > 1 has to win by 3 % of the launch.
static SchedPlan sched_plan(int64_t M, int32_t N, int32_t K, bool can_split, int32_t wgs) {
  SchedPlan p;
  p.tiles_m = (int32_t)((M + 255) / 256);
  p.tiles_n = (N + 255) / 256;
  p.kt = K / BK;
  p.wgs = wgs;
  p.raster = p.tiles_m >= 2 * kXcds ? 1 : 0;
  p.pieces = 1;
  p.slots = 2 * wgs;
  if (!can_split) return p;
  // per XCD: full rounds and remainder tiles (they differ by a tile between XCDs)
  int32_t full[kXcds], rem[kXcds], rem_max = 0;
  for (int32_t x = 0; x < kXcds; ++x) {
    const int32_t n = xcd_share(p, x).n_tiles;
    full[x] = n / wgs;
    rem[x] = n - full[x] * wgs;
    rem_max = rem[x] > rem_max ? rem[x] : rem_max;
  }
  if (rem_max == 0) return p;
  const double slab_us = 1.55, piece_us = 6.0;
  auto launch_time = [&](int32_t P, int32_t chunk) {   // the slowest XCD sets the time
    double worst = 0;
    for (int32_t x = 0; x < kXcds; ++x) {
      const int32_t rounds = (rem[x] * P + wgs - 1) / wgs;
      const double t = (double)full[x] * p.kt * slab_us + rounds * (chunk * slab_us + (P > 1 ? piece_us : 0.0));
      worst = t > worst ? t : worst;
    }
    return worst;
  };
  const double whole = launch_time(1, p.kt);
  double best = whole;
  for (int32_t P = 2; P <= 8 && P * rem_max <= 2 * wgs; ++P) {
    const int32_t chunk = sched_chunk(p.kt, P), n_chunks = (p.kt + chunk - 1) / chunk;
    if (n_chunks != P || chunk < 8) continue;
    int32_t cut_tiles = 0;
    for (int32_t x = 0; x < kXcds; ++x) cut_tiles += rem[x];
    const double fix_us = 8.0 + (double)cut_tiles * P * (kPartFloats * 4.0) / 3.0e6;
    const double t = launch_time(P, chunk) + fix_us;
    if (t < best && whole - t > 0.03 * whole) {
      best = t;
      p.pieces = P;
    }
  }
  return p;
}

// the most cut tiles any XCD has under a plan
static int32_t sched_max_rem(const SchedPlan& p) {
  int32_t m = 0;
  for (int32_t x = 0; x < kXcds; ++x) {
    const int32_t r = xcd_share(p, x).rem;
    m = r > m ? r : m;
  }
  return m;
}

static size_t slots_bytes(int32_t per_xcd) { return (size_t)kXcds * per_xcd * kPartFloats * sizeof(float); }
static int32_t pieces_slots(int64_t M, int32_t N, int32_t pieces) {   // every tile of an XCD is cut
  return (int32_t)((((M + 255) / 256) * ((N + 255) / 256) + kXcds - 1) / kXcds) * pieces;
}
static size_t sched_scratch_bytes(int32_t wgs) { return slots_bytes(2 * wgs); }

size_t gemm_sched_scratch_bytes(int64_t M, int32_t N, int32_t K) {
  if (!takes_sched_kernel(M, N, K, false)) return 0;
  const int32_t wgs = sched_wgs_per_xcd();
  return sched_plan(M, N, K, true, wgs).pieces == 1 ? 0 : sched_scratch_bytes(wgs);
}

// How a shape that is too small for the 256x256 kernel's whole rounds runs, given `cap` bytes of scratch:
//   kSplit   32x32, 64x32 or 64x64 tiles, K cut over the four wavefronts of the workgroup (gemm_ksplit.hip);
//   kRing    one of eleven tiles of 64x64 to 160x256, four wavefronts (gemm_ring.hip), K whole or cut over ks workgroups
//            (sums in the scratch);
//   kPieces  the 256x256 kernel with every tile cut into pieces (needs M, N >= 256 and K % 128 == 0).
// The one with the least expected time, by a model that is fitted per tile to a sweep of 7300 shapes on all of them (65 to
// 5000 rows of every layer width and others, K of 64 to 32768, the three epilogues, three sets of operands in turn).  What the choice
// turns on is whole rounds: so many sizes, because each alone is the best by 10 to 45 % wherever its tiles just fill the CUs.  Measured
// (us; in brackets the same shape on the tiles of the kernel before this one):
//   387 x 4096 x 1024 + GeLU 10.1 64x64 [11.2]         928 x 5120 x 5120 + residual 54.9 128x192 [69.5]   200 x 20480 x 5120 70.4 128x192 [99]
//   600 x 4096 x 16384 84.7 160x256 in parts [102]     2280 x 4096 x 4096 68.0 160x256 [109]              333 x 5120 x 20480 87.7 128x256 in parts [105]
//   692 x 30536 x 192 21.9 128x128 [31.6]              5239 x 2840 x 192 + GeLU 20.7 128x128 [27.5]       369 x 1096 x 11456 + GeLU 21.4 96x128 in parts [26.2]
// Against the choice before (64x64, 128x128 and 128x256 tiles of a compiler-scheduled kernel), 9000 random shapes of some 8 us and more (66 to 8192
// rows), the time in the mean and how many take more than 3 % longer: widths that are multiples of 64 0.73, 15 of 5000; others 0.74, 9 of
// 2500; K of eight N and more 0.65, 3 of 1500; at most 1.14 times (65 to 128 rows and a W of 100 MB and more, which 128x256 in parts
// reads a little faster), but for a tall x over 256 columns in eight parts (3567 x 256 x 16384 52 -> 68, 4087 x 256 x 22016 72 -> 81: counting
// x in `weights` as well mends those and takes 1.05 times as long in the mean of what it changes).  What stayed on 64x64 tiles at K of 320
// and less and some 500 to 800 tiles loses up to 1.1 (8881 x 320 x 320 8.0 -> 8.8): three workgroups of that kernel shared a CU, two of
// this one do.
enum TileKind { kSplit, kRing, kPieces };
struct TilePlan { TileKind kind; KsplitTile split; int32_t ring, ks; size_t scratch; double us; };   // ks: parts of K (kPieces: pieces per tile)

// us = base + gelu + residual + n (round + residual_round) + steps * slab(n), n = tiles per CU; slab(n) through the given
// points, in proportion beyond the last.
struct TileTime {
  double base, gelu, residual, round, residual_round;
  struct { double n, us; } slab[11];
  double slab_us(double n) const {
    int i = 1;
    while (i < 10 && n > slab[i].n && slab[i + 1].n > 0) ++i;
    if (n > slab[i].n) return slab[i].us * n / slab[i].n;
    return slab[i - 1].us + (slab[i].us - slab[i - 1].us) * (n - slab[i - 1].n) / (slab[i].n - slab[i - 1].n);
  }
  double us(double n, int epi) const {   // without the slabs
    return base + n * round + (epi == EPI_BIAS_GELU ? gelu : 0.0) + (epi == EPI_BIAS_RESIDUAL ? residual + n * residual_round : 0.0);
  }
};
// Steps of four slabs, one per wavefront.  `round` is from calls replayed from graphs: the host bounds a call of 5 us that is not, which
// hid a quarter of it (1350 x 768 x 256 5.7 us on 64x64 tiles of the kernel before the ring, 6.9 on 32x32, 5.4 on 64x96).
constexpr TileTime kSplitTime[3] = {
    {2.18, 0.23, 0.27, 0.61, 0.08,
     {{0, 0.298}, {1, 0.345}, {1.003, 0.573}, {2, 0.662}, {2.003, 0.888}, {4, 1.261}, {4.003, 1.456}, {6, 1.934}, {16, 5.175}, {40, 12.477}}},
    {2.38, 0.43, 0.23, 1.94, 0.39,
     {{0, 0.454}, {1, 0.451}, {1.003, 1.050}, {2, 0.944}, {2.003, 1.580}, {3, 1.469}, {3.003, 1.969}, {4, 2.081}, {8, 4.395}, {20, 11.016}}},
    {3.54, 0.41, 0.18, 3.67, 1.05,
     {{0, 0.684}, {1, 0.645}, {1.003, 1.471}, {2, 1.345}, {2.003, 2.141}, {3, 2.174}, {3.003, 2.709}, {5, 3.701}, {10, 8.146}}}};
static_assert((int)KsplitTile::k32x32 == 0 && (int)KsplitTile::k64x32 == 1 && (int)KsplitTile::k64x64 == 2, "order of kSplitTime");

// Tiles of gemm_ring.hip: launch, then rounds of workgroups; a round is its epilogue and its slabs, a slab as long as the
// workgroups that share a CU make it, and shorter where not every CU has one more (power, memory).  `weights`: us per 100 MB of W;
// `cold`: what a slab takes longer where operands come from HBM: x and W of 85 MB and more together, which is where the sweep's three sets
// in turn outgrow the last cache's 256 MB (in a stack whose layers add up to more smaller ones do too, alone in a loop larger ones do
// not).  With W alone counted, a tall x took tiles that wait for it: 5462 x 512 x 22272 + GeLU 179 us on 96x128, 133 in pieces of
// 256x256; 2857 x 1024 x 16896 + residual 138 on 96x128, 105 on 160x256 in parts.  1500 shapes that this changed: 0.92 of the time in the mean.
// sums, sums_part, sums_res: the second kernel of a cut K, us and us per million outputs, for each part and for the residual.
struct RingTime {
  double base, round, drop, gelu, residual, weights, cold, sums, sums_part, sums_res, slab[2];
  // n workgroups on an XCD of so many CUs
  double us(int per_cu, int32_t n, int32_t cus, double slabs, int epi, bool streams) const {
    const double epilogue = round + (epi == EPI_BIAS_GELU || epi == EPI_LNFOLD_GELU ? gelu : 0.0) + (epi == EPI_BIAS_RESIDUAL ? residual : 0.0) +
                            (epi == EPI_LNFOLD || epi == EPI_LNFOLD_GELU ? 0.5 * round : 0.0);
    const int32_t whole = (n - 1) / (cus * per_cu), rest = n - whole * cus * per_cu;   // rounds before the last; the last one's workgroups
    const int level = rest <= cus ? 1 : 2;   // per_cu is 1 or 2
    return base + whole * (epilogue + slabs * slab[per_cu - 1]) + epilogue * (level + 1) / (per_cu + 1) +
           slabs * slab[level - 1] * (1.0 - (streams ? 0.0 : drop) * (level - rest / (double)cus));
  }
};
constexpr RingTime kRingTime[] = {   // the order of kRingShapes
    {2.82, 1.71, 0.146, 0.66, 0.31, 0.00, 0.49, 0.00, 0.00, 0.00, {0.188, 0.321}},
    {3.37, 2.03, 0.219, 1.23, 0.87, 1.75, 0.50, 0.00, 0.00, 0.00, {0.230, 0.408}},
    {3.35, 2.78, 0.222, 1.39, 1.28, 1.51, 0.48, 0.00, 0.00, 0.00, {0.314, 0.511}},
    {1.11, 4.96, 0.137, 1.26, 1.40, 4.26, 0.62, 0.39, 1.61, 0.00, {0.283}},
    {1.09, 5.76, 0.259, 1.65, 0.87, 4.34, 0.47, 0.00, 1.44, 0.21, {0.363}},
    {3.03, 4.06, 0.232, 2.17, 1.96, 2.46, 0.32, 0.00, 0.00, 0.00, {0.713, 0.807}},
    {1.29, 5.97, 0.259, 2.18, 0.72, 6.22, 0.48, 0.00, 1.10, 0.40, {0.394}},
    {1.05, 7.33, 0.331, 2.91, 1.02, 7.38, 0.24, 0.00, 0.85, 0.69, {0.500}},
    {0.50, 8.21, 0.290, 3.95, 1.48, 6.97, 0.16, 0.00, 0.90, 0.62, {0.586}},
    {0.39, 8.24, 0.302, 3.53, 1.52, 8.85, 0.14, 0.00, 0.93, 0.46, {0.632}},
    {0.72, 8.63, 0.311, 4.33, 6.02, 8.16, 0.05, 0.00, 0.92, 0.34, {0.759}}};
static_assert(sizeof(kRingTime) / sizeof(kRingTime[0]) == kRingCount, "one per tile");

// epi: one of EPI_BIAS, EPI_BIAS_GELU, EPI_BIAS_RESIDUAL (all plans) or the folded ones (kRing without parts only).
static TilePlan tile_plan(int64_t M, int32_t N, int32_t K, bool overlap_safe, int epi, size_t cap, int32_t wgs) {
  const bool plain = epi != EPI_LNFOLD && epi != EPI_LNFOLD_GELU;
  const int32_t KT = K / BK;
  const double cus = 8.0 * wgs;
  TilePlan best{kRing, KsplitTile::k64x64, 0, 1, 0, 1e30};
  const auto consider = [&](TilePlan t, double us) {
    if (t.scratch <= cap && us < best.us) { best = t; best.us = us; }
  };
  // (this function is called for every linear: 32-bit divisions where M allows; callers that only ask for a size may give any M)
  const bool narrow = M < ((int64_t)1 << 31);
  const auto tiles = [&](uint32_t bm, uint32_t bn) {
    const int64_t rows = narrow ? ((uint32_t)M + bm - 1) / bm : (M + bm - 1) / bm;
    return rows * (((uint32_t)N + bn - 1) / bn);
  };
  const auto fits = [](int64_t tiles, int64_t threads) { return tiles * threads <= kMaxGridThreads; };
  const double w_bytes = 2.0 * N * K;
  const bool from_hbm = 2.0 * K * ((double)M + N) > 85.0e6;   // see RingTime
  // Few rows and a W of 100 MB and more: hardly a line of W is in an L2 when a workgroup asks for it, so a slab does not get shorter where CUs
  // are idle, and 64 rows ask for each line more than once.  On all plans of 1190 shapes (65 to 400 rows, W of 85 to 260 MB) the choice then
  // costs 1.0 % over the best in the mean, 1.6 % without; 123 x 17216 x 3456 + residual 45.9 us on 64x96, 37.3 on 128x192 in parts.
  const bool streams = w_bytes > 100.0e6 && M <= 256;
  const double far = from_hbm ? 1.45 : 1.0;   // the same for the small tiles that cut K
  if (plain) {
    // a last step that not all four wavefronts take costs about half the difference to one that they do
    const double steps = 0.5 * ((KT + 3) / 4 + 0.25 * KT);
    const KsplitTile split[3] = {KsplitTile::k32x32, KsplitTile::k64x32, KsplitTile::k64x64};
    const int64_t n[3] = {tiles(32, 32), tiles(64, 32), tiles(64, 64)};
    for (int i = 0; i < 3; ++i)
      if (fits(n[i], 256)) consider({kSplit, split[i], 0, 1, 0}, kSplitTime[i].us(n[i] / cus, epi) + steps * far * kSplitTime[i].slab_us(n[i] / cus));
  }
  const double elems = (double)M * N, res = epi == EPI_BIAS_RESIDUAL ? 1.0 : 0.0;
  // No ring tile wins where 32x32 ones are one round and K is short (0.4 us of host time saved on calls that it bounds).
  const bool tiny = plain && KT <= 64 && tiles(32, 32) <= 8 * wgs;
  if (!tiny) {
    const bool spills = 2.0 * (M + N) * K > 256.0e6;   // x and W do not both fit the last cache: another round reads them again
    for (int i = 0; i < kRingCount; ++i) {
      const RingShape& shape = kRingShapes[i];
      const int64_t n = tiles(shape.rows, shape.cols);
      if (!fits(n, 256) || (int64_t)K * 2 * std::max(shape.rows, shape.cols) > UINT32_MAX) continue;   // a tile's rows in 32-bit byte offsets
      if (shape.rows >= M + 64) continue;   // a smaller one does
      // K whole, or cut where the tiles alone leave CUs idle: into as many parts of six slabs at least as fill them, one less or half
      const int32_t fill = plain && shape.per_cu == 1 && n <= 4 * wgs ? std::min({8 * wgs / (int32_t)n, 8, KT / 6}) : 1;
      for (const int32_t parts : {1, fill, fill - 1, (fill + 1) / 2}) {
        if (parts < 1) continue;
        const int32_t units = (int32_t)n * parts;   // fits() above
        const double cold = from_hbm ? kRingTime[i].cold + (streams && shape.rows == 64 && M > 64 ? 0.2 : 0.0) : 0.0;
        double us = kRingTime[i].us(shape.per_cu, (units + kXcds - 1) / kXcds, wgs, (parts > 1 ? (KT + parts - 1) / parts : KT) * (1.0 + cold),
                                    parts > 1 ? EPI_BIAS : epi, streams) + kRingTime[i].weights * 1.0e-8 * w_bytes;
        if (streams) us *= 0.92;
        if (spills && units > 8 * wgs * shape.per_cu) us *= 1.2;
        if (parts > 1) us = 1.05 * (us + kRingTime[i].sums + elems * 1.0e-6 * (kRingTime[i].sums_part * parts + kRingTime[i].sums_res * res));
        consider({kRing, KsplitTile::k64x64, i, parts, parts > 1 ? (size_t)parts * (size_t)M * N * sizeof(float) : 0}, us);
        if (fill <= 1) break;
      }
    }
  }
  if (plain && M >= 256 && N >= 256 && K % 128 == 0 && overlap_safe) {
    const int64_t big = tiles(256, 256);
    for (int32_t P = 2; P <= 8; ++P) {
      const int64_t rem = (big + kXcds - 1) / kXcds;   // tiles of an XCD
      const int32_t chunk = sched_chunk(KT, P);
      // one round at most of every XCD's workgroups, and slots for it (two per workgroup)
      if (rem >= wgs || rem * P > 2 * wgs || (KT + chunk - 1) / chunk != P || chunk < 8) continue;
      const double rounds = std::ceil((double)rem * P / wgs);
      consider({kPieces, KsplitTile::k64x64, 0, P, slots_bytes(pieces_slots(M, N, P))},
               8.2 + rounds * (1.1 + 1.228 * chunk) + (0.388 * big * P * kPartFloats * 4.0 + 0.394 * res * elems) / 1.0e6);
    }
  }
  return best;
}

// The persistent kernel takes what gives it 192 tiles, but up to some 400 of them are one or two rounds with much of the last one
// empty, and a ring tile can fill its own better: expected times of both, the persistent kernel's fitted to 1100 shapes of 192
// to 420 tiles (its slab time is the mean over W from HBM and from the last cache, which RingTime tells apart).  Taken where the ring kernel is
// expected to need under 0.87 of the time: 1000 such shapes 0.71 of the time in the mean, four more than 3 % slower, at most 1.15 (3074 x 5120 x
// 1280 + residual 75 -> 53 us, 306 x 24576 x 8192 204 -> 133; 997 x 22272 x 896 + residual 61 -> 70); between that and 1 the two come out as
// they may (0.97: a sixth of all shapes more than 3 % slower).
static double sched_us(const SchedPlan& p, int64_t M, int32_t N, int epi) {
  const double slab = 1.47, epilogue = 9.26 + (epi == EPI_BIAS_GELU ? 6.1 : 0.0) + (epi == EPI_BIAS_RESIDUAL ? 4.43 : 0.0);
  double worst = 0;
  int32_t cut = 0;
  for (int32_t x = 0; x < kXcds; ++x) {
    const XcdShare s = xcd_share(p, x);
    const int32_t full = s.n_tiles / p.wgs, rem = s.n_tiles - full * p.wgs;
    double t = full * (epilogue + p.kt * slab);
    if (p.pieces > 1) {
      t += (rem * p.pieces + p.wgs - 1) / p.wgs * (s.chunk * slab + 5.32);
      cut += rem;
    } else if (rem > 0) {
      t += epilogue + p.kt * slab * (1.0 - 0.452 * (1.0 - rem / (double)p.wgs));
    }
    worst = t > worst ? t : worst;
  }
  const double second = p.pieces > 1 ? 0.349e-6 * cut * p.pieces * (kPartFloats * 4.0) + (epi == EPI_BIAS_RESIDUAL ? 0.202e-6 * M * N : 0.0) : 0.0;
  return 1.15 + worst + second;
}
static bool ring_instead(int64_t M, int32_t N, int32_t K, int epi, const SchedPlan& p, TilePlan& t) {
  if ((int64_t)p.tiles_m * p.tiles_n >= 420 || N % 64 != 0) return false;   // the sweep behind it had multiples of 64 only
  t = tile_plan(M, N, K, true, epi, 0, p.wgs);
  return t.kind == kRing && t.us < 0.87 * sched_us(p, M, N, epi);
}

static SchedPlan pieces_plan(int64_t M, int32_t N, int32_t K, int32_t pieces, int32_t wgs) {
  SchedPlan p;
  p.tiles_m = (int32_t)((M + 255) / 256);
  p.tiles_n = (N + 255) / 256;
  p.kt = K / BK;
  p.wgs = wgs;
  p.raster = 0;
  p.pieces = pieces;
  p.slots = pieces_slots(M, N, pieces);
  return p;
}

size_t gemm_scratch_bytes(int64_t M, int32_t N, int32_t K) {
  if (takes_sched_kernel(M, N, K, false)) return gemm_sched_scratch_bytes(M, N, K);
  if (M <= 0 || gemm_skinny_takes(M, N, K, EPI_BIAS)) return 0;   // few rows: planned for by the generation step only
  size_t need = 0;   // of whichever epilogue the call turns out to have
  for (const int epi : {EPI_BIAS, EPI_BIAS_GELU, EPI_BIAS_RESIDUAL})
    need = std::max(need, tile_plan(M, N, K, true, epi, SIZE_MAX, sched_wgs_per_xcd()).scratch);
  return need;
}

// Host-side check of the decomposition for one shape (what the kernels would do, replayed with the
// same functions): every tile is either finished whole by exactly one workgroup or cut into pieces
// whose slab ranges are even, start where the previous one ended and add up to the tile; the pieces of
// a tile occupy the slots its second-kernel workgroups read, in ascending K order; no slot is used
// twice or lies outside the XCD's.  0 if all of that holds, else a positive code naming the
// first violation; -1 if the 256x256 kernel does not take the shape.
int gemm_sched_selfcheck(int64_t M, int32_t N, int32_t K, int32_t wgs, int32_t can_split, int32_t* pieces_out) {
  if (wgs < 1) return -1;
  SchedPlan p;
  if (takes_sched_kernel(M, N, K, false)) {
    p = sched_plan(M, N, K, can_split != 0, wgs);
  } else {
    if (!can_split) return -1;
    const TilePlan t = tile_plan(M, N, K, true, EPI_BIAS, SIZE_MAX, wgs);
    if (t.kind != kPieces) return -1;
    p = pieces_plan(M, N, K, t.ks, wgs);
  }
  if (pieces_out) *pieces_out = p.pieces;
  const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n;
  std::vector<int32_t> covered(tiles, 0);     // slabs covered so far (pieces must arrive in K order per tile)
  std::vector<int8_t> whole(tiles, 0);
  for (int32_t x = 0; x < kXcds; ++x) {
    const XcdShare sh = xcd_share(p, x);
    std::vector<int8_t> slot_used(p.slots, 0);
    // pieces of one tile are produced by different workgroups: collect (tile, kb, n, slot) and sort by kb
    struct Piece { int64_t tile; int32_t kb, n, slot; };
    std::vector<Piece> pieces;
    int64_t seen = 0;
    for (int32_t wg = 0; wg < wgs; ++wg) {
      SchedWalker walk(p, x, wg);
      int32_t l, kb, n, slot;
      while (walk.next(l, kb, n, slot)) {
        if (l < 0 || l >= sh.n_tiles) return 1;
        int32_t tm, tn;
        sched_tile(p, x, l, tm, tn);
        if (tm < 0 || tm >= p.tiles_m || tn < 0 || tn >= p.tiles_n) return 2;
        const int64_t tile = (int64_t)tm * p.tiles_n + tn;
        if (n <= 0 || (n & 1) || (kb & 1) || kb < 0 || kb + n > p.kt) return 3;
        if (slot < 0) {
          if (kb != 0 || n != p.kt || whole[tile] || covered[tile]) return 4;
          whole[tile] = 1;
          covered[tile] = p.kt;
        } else {
          if (slot >= p.slots || slot_used[slot]) return 5;
          slot_used[slot] = 1;
          pieces.push_back({tile, kb, n, slot});
        }
        ++seen;
      }
    }
    std::sort(pieces.begin(), pieces.end(), [](const Piece& a, const Piece& b) { return a.tile != b.tile ? a.tile < b.tile : a.kb < b.kb; });
    for (const Piece& q : pieces) {
      if (whole[q.tile] || covered[q.tile] != q.kb) return 6;
      covered[q.tile] += q.n;
    }
    // what the second kernel reads: cut tile t of this XCD = tile dp_rounds * wgs + t, slots t * P + c, c ascending
    const int32_t n_chunks = (p.kt + sh.chunk - 1) / sh.chunk;
    for (int32_t t = 0; t < sh.rem; ++t) {
      int32_t tm, tn;
      sched_tile(p, x, sh.dp_rounds * wgs + t, tm, tn);
      const int64_t tile = (int64_t)tm * p.tiles_n + tn;
      int32_t kb = 0;
      for (int32_t c = 0; c < n_chunks; ++c) {
        bool found = false;
        for (const Piece& q : pieces)
          if (q.slot == t * p.pieces + c) { found = q.tile == tile && q.kb == kb; kb += q.n; break; }
        if (!found) return 7;
      }
      if (kb != p.kt) return 8;
    }
    if (sh.rem > wgs || (p.pieces > 1 && sh.rem * p.pieces > p.slots)) return 9;
    (void)seen;
  }
  for (int64_t t = 0; t < tiles; ++t)
    if (covered[t] != p.kt) return 10;
  return 0;
}

template <typename E, int MODE>
static hipError_t launch_sched(const E* x, const E* w, const E* bias, const E* res, E* y, int64_t M, int32_t N,
                               int32_t K, int epi, const LnFold& lf, hipStream_t s, const SchedPlan& plan,
                               float* scratch) {
  constexpr size_t slabs = 2 * (size_t)(256 + 256) * kChunks * sizeof(uint4);
  constexpr size_t epi_stage = 4 * (size_t)kEpiWaveFloats * sizeof(float);
  constexpr size_t lds = slabs > epi_stage ? slabs : epi_stage;
  static LdsAttrOnce attr_main;   // per element type and MODE
  auto kern = gemm_mfma_sched_kernel<E, 256, 256, 2, 2, MODE>;
  hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds, attr_main);
  if (e != hipSuccess) return e;
  kern<<<dim3((unsigned)(kXcds * plan.wgs)), dim3(256), lds, s>>>(x, w, bias, res, y, M, N, K, epi, plan, scratch, lf);
  e = hipGetLastError();
  if (e != hipSuccess || plan.pieces == 1) return e;
  const int32_t max_rem = sched_max_rem(plan);
  gemm_mfma_fixup_kernel<E><<<dim3((unsigned)(kXcds * max_rem * kFixStrips)), dim3(512), 0, s>>>(scratch, bias, res, y, M, N,
                                                                                                  epi, plan);
  return hipGetLastError();
}

template <typename E>
static hipError_t launch_gemm_mfma(const E* x, const E* w, const E* bias, const E* res, E* y, int64_t M, int32_t N,
                                   int32_t K, int epi, hipStream_t s, const LnFold* fold, float* scratch,
                                   size_t scratch_bytes) {
  if (M <= 0) return hipSuccess;
  if (scratch == nullptr) scratch_bytes = 0;
  const LnFold lf = fold != nullptr ? *fold : LnFold{};
  const bool wants_fold = epi == EPI_LNFOLD || epi == EPI_LNFOLD_GELU;
  if (wants_fold && (lf.stats == nullptr || lf.colsum == nullptr || lf.bias == nullptr)) return hipErrorInvalidValue;
  if (lf.partial != nullptr && (epi != EPI_BIAS_RESIDUAL || !gemm_emits_row_partials(M, N, K, res == y)))
    return hipErrorInvalidValue;
  if (lf.partial == nullptr && gemm_skinny_takes(M, N, K, epi))
    return launch_gemm_skinny<E>(x, w, bias, res, y, M, N, K, epi, s, scratch, scratch_bytes);
  const int32_t wgs = sched_wgs_per_xcd();
  if (takes_sched_kernel(M, N, K, res == y)) {
    // the LayerNorm-folded epilogues and the row statistics live in the main kernel only: no cutting there
    const bool plain = !wants_fold && lf.partial == nullptr;
    const SchedPlan plan = sched_plan(M, N, K, plain && scratch_bytes >= sched_scratch_bytes(wgs), wgs);
    if (wants_fold) return launch_sched<E, kEpiFolded>(x, w, bias, res, y, M, N, K, epi, lf, s, plan, nullptr);
    if (!plain) return launch_sched<E, kEpiResidualStats>(x, w, bias, res, y, M, N, K, epi, lf, s, plan, nullptr);
    TilePlan t;
    if (ring_instead(M, N, K, epi, plan, t)) return launch_gemm_ring<E>(t.ring, x, w, bias, res, y, M, N, K, epi, lf, s);
    return launch_sched<E, kEpiPlain>(x, w, bias, res, y, M, N, K, epi, lf, s, plan, scratch);
  }
  // Shifted edge tiles of the 256x256 kernel overlap: not with the residual aliasing y (see takes_sched_kernel).
  const bool overlap_safe = res != y || (M % 256 == 0 && N % 256 == 0);
  const TilePlan t = tile_plan(M, N, K, overlap_safe, epi, scratch_bytes, wgs);
  if (t.kind == kSplit) return launch_gemm_ksplit<E>(t.split, x, w, bias, res, y, M, N, K, epi, s);
  if (t.kind == kPieces)
    return launch_sched<E, kEpiPlain>(x, w, bias, res, y, M, N, K, epi, lf, s, pieces_plan(M, N, K, t.ks, wgs), scratch);
  return launch_gemm_ring<E>(t.ring, x, w, bias, res, y, M, N, K, epi, lf, s, t.ks, scratch);
}

LinearPlan gemm_plan(int64_t M, int32_t N, int32_t K, int epi, bool res_aliases_y, size_t scratch_bytes) {
  if (gemm_skinny_takes(M, N, K, epi)) return gemm_skinny_plan_of(M, N, K, scratch_bytes);
  const bool plain = epi != EPI_LNFOLD && epi != EPI_LNFOLD_GELU;
  const int32_t wgs = sched_wgs_per_xcd();
  if (takes_sched_kernel(M, N, K, res_aliases_y)) {
    const SchedPlan p = sched_plan(M, N, K, plain && scratch_bytes >= sched_scratch_bytes(wgs), wgs);
    TilePlan t;
    if (plain && ring_instead(M, N, K, epi, p, t)) return {LinearPlan::kTiles, kRingShapes[t.ring].rows, kRingShapes[t.ring].cols, 1};
    return {LinearPlan::kPersistent, 256, 256, p.pieces};
  }
  const TilePlan t = tile_plan(M, N, K, !res_aliases_y || (M % 256 == 0 && N % 256 == 0), epi, scratch_bytes, wgs);
  switch (t.kind) {
    case kSplit: return {LinearPlan::kWaves, t.split == KsplitTile::k32x32 ? 32 : 64, t.split == KsplitTile::k64x64 ? 64 : 32, 1};
    case kPieces: return {LinearPlan::kPersistent, 256, 256, t.ks};
    default: return {LinearPlan::kTiles, kRingShapes[t.ring].rows, kRingShapes[t.ring].cols, t.ks};
  }
}

hipError_t launch_gemm_bf16(const bf16_t* x, const bf16_t* w, const bf16_t* bias, const bf16_t* res, bf16_t* y,
                            int64_t M, int32_t N, int32_t K, int epi, hipStream_t s, const LnFold* fold,
                            float* scratch, size_t scratch_bytes) {
  return launch_gemm_mfma<bf16_t>(x, w, bias, res, y, M, N, K, epi, s, fold, scratch, scratch_bytes);
}

hipError_t launch_gemm_f16(const f16_t* x, const f16_t* w, const f16_t* bias, const f16_t* res, f16_t* y, int64_t M,
                           int32_t N, int32_t K, int epi, hipStream_t s, const LnFold* fold, float* scratch,
                           size_t scratch_bytes) {
  return launch_gemm_mfma<f16_t>(x, w, bias, res, y, M, N, K, epi, s, fold, scratch, scratch_bytes);
}

}  // namespace energon
