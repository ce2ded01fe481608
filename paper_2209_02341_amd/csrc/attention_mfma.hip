// Causal attention (bf16 or fp16 storage) over each sequence's real length, on packed rows.  The paper
// (Sec. 4.3) rebuilds the padding around the attention core; here the core itself is
// variable-length, so nothing is rebuilt inside a layer and no score is computed for a pad.
//
// One workgroup (4 wavefronts, two workgroups per CU) = one (sequence, head, block of 128 queries); each wavefront
// owns 32 queries.  Keys / values come in tiles of 32 keys through a ring of four stages in LDS, shared by the
// wavefronts and worked on two tiles at a time; tiles above the causal diagonal are never visited.
//
// Everything is computed transposed so that a query is a *column* of every MFMA result
// (v_mfma_f32_32x32x16_bf16 / _f16: the lane holds column l % 32, rows 8 (e / 4) + 4 (l / 32) + e % 4):
//   S^T[key, query] = K[key, :] . Q[query, :]      A operand = K rows, B operand = Q rows
//   O^T[dd,  query] += V^T[dd, key] . P^T[key, query]
// so the online-softmax state (running max, running sum) is one scalar per lane, and the
// exponentiated scores are already laid out as the B operand of the second product: no
// cross-lane movement of P.  The contraction index (key) may be enumerated in any order as long as both
// operands agree, so the V operand takes it in the order the accumulators have, as two transposed LDS reads of four
// keys each (ds_read_b64_tr_b16) from the rows as they were fetched: V is never written a second time.
// Q, K and V rows go from global memory straight to LDS (whole 128- or 256-byte row pieces, the swizzle applied on
// the global side).
//
// What bounds it: per 32 keys a wavefront has 512 matrix-core cycles (d = 128) and about 730 of the vector ALU
// (16 exponentials per lane at a quarter of the rate, and, per pair of tiles, 64 multiplications that rescale the
// accumulators), with two wavefronts per SIMD to overlap them; on short sequences the fixed cost of a block, about
// 4 us of dependent memory latencies (lengths, first rows, last stores) and 2 us between two workgroups of a slot.
// Measured (bf16, d = 128, before -> now): 8 sequences of 1536 .. 2047 tokens x 40 heads 524 -> 403 us, 8 of 2048 582 -> 450,
// 64 of very unequal length x 64 heads 734 -> 500, 32 of up to 512 x 40 94 -> 84, 64 of up to 64 x 40 29.1 -> 24.7;
// d = 64: 8 long x 25 165 -> 133, 50 of up to 200 x 16 16.6 -> 13.6.  Before, 8
// wavefronts of 16 queries read every operand from LDS twice as often and copied V into a transposed tile, with two
// barriers per 64 keys.  Following the running max only when it had moved by a factor of 2^8 saves the rescaling and
// another 10 %, but then the largest weight of a row is no longer exactly 1 and the error grows by a twentieth: not done.
#include "common.h"
#include <algorithm>
#include <type_traits>

namespace energon {

constexpr int kAttnWaves = 4, kWQ = 32, kBQ = kAttnWaves * kWQ;   // queries per wavefront, per workgroup
constexpr int kBKV = 32, kStages = 4;                             // keys per tile, tiles in LDS
constexpr float kLog2e = 1.4426950408889634f;

typedef __attribute__((address_space(3))) void* attn_lptr_t;

// 16-byte slot of chunk c of row r inside an LDS row: c ^ kswz(r) for rows read as 32-row operand tiles (lane l:
// row l % 32, chunk 2 ks + l / 32), c ^ vswz(r) for rows read transposed (8 rows x 64 bytes per instruction, of
// which half a wavefront takes 4 rows): all 64 banks once per pass.
template <int D> __device__ __forceinline__ int kswz(int row) {
  return D == 128 ? (row & 15) : ((row & 7) ^ ((row >> 3) & 1));
}
template <int D> __device__ __forceinline__ int vswz(int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); }

// 1 KiB from global memory straight to LDS: lane l's 16 bytes at base + off go to LDS byte dst + 16 l.  Written as an asm
// statement because the compiler puts a wait for every load in flight in front of each transposed LDS read
// when it sees the transfers (it cannot tell the tiles apart); attn_wait below counts them instead.  Nothing
// here writes a register but m0, which the compiler allocates to nothing (reserved; no other use in this kernel).
__device__ __forceinline__ void dma16(const char* base, uint32_t off, uint32_t dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(dst), "v"(off), "s"(base) : "memory");
}

// Wait for all but the newest n <= 2 tiles' loads of this wavefront (G instructions each; loads return in order) and
// for its LDS reads.
template <int G> __device__ __forceinline__ void attn_wait(int n) {
  if (n >= 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * G) : "memory");
  else if (n == 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(G) : "memory");
  else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

// Which (sequence, head, query block) this workgroup computes; false: none.  Workgroups run on XCD id % 8, each XCD
// in the order of its ids.  Three ways:
//  * n_qblocks > 0, group = 0: the last query block (the one with the most keys) of all (sequence, head) pairs, heads
//    fastest, then the blocks in front of it.  Longest first and dealt to the XCDs one by one, the chip stays
//    balanced whatever the number of pairs;
//  * n_qblocks > 0, group > 0: an XCD takes whole pairs, about kAttnGroup at a time in that order, so that the blocks that
//    share K and V meet in its L2; the pairs that the XCDs do not share evenly go first, their blocks dealt one by one;
//  * n_qblocks = 0 (packed, up to kAttnScan sequences, where max_len leaves a good part of the blocks without queries):
//    only blocks that have queries are counted, from a scan of the lengths by every wavefront, and the host
//    launches an upper bound.  A sequence's heads go to the XCDs in whole eights, the blocks of the others are dealt.
// Measured (us; order by pairs throughout / longest first throughout / as it is): 1 sequence of 32768 x 4 heads x 128
// 2056 / 1135 / 1135, 1 of 8192 x 12 heads 310 / 233 / 233, 32 of 512 x 40 heads 208 / 232 / 176, 8 of 2048 x 40
// heads x 128 (padded) 470 / 450 / 427, 16 of 512 x 40 heads 105 / 92 / 88, 8 of 512 x 40 heads 52.5 / 47.0 / 47.0.
constexpr int kAttnGroup = 8;
constexpr int kAttnScan = 256;

// Sum over lanes 0 .. l in every lane l: shifts inside rows of 16 lanes, then the last lane of the row (of the half)
// in front added to the rows behind it.
__device__ __forceinline__ int32_t wave_inclusive_sum(int32_t v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr 1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast 15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast 31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ bool attn_block(const int32_t* __restrict__ cu, int32_t B, int32_t nh, int32_t n_qblocks,
                                           int32_t group, int lane, int32_t& b, int32_t& h, int32_t& qb, int32_t& c0,
                                           int32_t& len) {
  const int32_t xcd = blockIdx.x % kXcds, j = blockIdx.x / kXcds;
  if (n_qblocks > 0) {
    const int32_t pairs = B * nh, whole = pairs / kXcds, rest = pairs - whole * kXcds;   // pairs per XCD, left over
    const int32_t dealt = (rest * n_qblocks + kXcds - 1) / kXcds;                         // their blocks per XCD
    int32_t pair, k;   // k: blocks behind this one in the sequence
    if (group == 0) {
      k = (int32_t)blockIdx.x / pairs;
      pair = (int32_t)blockIdx.x - k * pairs;
    } else if (j < dealt) {
      const int32_t u = xcd + kXcds * j;
      k = u / rest;
      pair = kXcds * whole + u - k * rest;
    } else {
      const int32_t per = group * n_qblocks, g = (j - dealt) / per, in = j - dealt - g * per;
      const int32_t size = min(group, whole - g * group);
      if (size <= 0) return false;
      k = in / size;
      pair = xcd + kXcds * (g * group + in - k * size);
    }
    if (k >= n_qblocks) return false;
    b = pair / nh;
    h = pair - b * nh;
    qb = n_qblocks - 1 - k;
    c0 = cu[b];
    len = cu[b + 1] - c0;
    return true;
  }
  // lane l: sequences per * l .. per * l + per - 1; a sequence of n query blocks has n * (nh / 8) on every XCD and of the
  // n * (nh % 8) others, numbered from the sequence's index times nh, those whose number is this XCD's modulo 8
  constexpr int kPer = kAttnScan / kWave;
  const int32_t per = (B + kWave - 1) / kWave, first = lane * per;
  const int32_t eights = nh / kXcds, rest = nh - eights * kXcds;
  int32_t at[kPer + 1], nb[kPer], w[kPer], mine = 0;
  at[0] = cu[min(first, B)];
#pragma unroll
  for (int k = 0; k < kPer; ++k) at[k + 1] = k < per ? cu[min(first + k + 1, B)] : 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    nb[k] = k < per ? (at[k + 1] - at[k] + kBQ - 1) / kBQ : 0;
    const int32_t p = (((first + k) * rest) & (kXcds - 1)) + kXcds - 1 - xcd;
    w[k] = nb[k] * eights + (p + nb[k] * rest) / kXcds - p / kXcds;
    mine += w[k];
  }
  const int32_t incl = wave_inclusive_sum(mine);
  if (j >= __builtin_amdgcn_readlane(incl, kWave - 1)) return false;
  const int src = __popcll(__ballot(incl <= j));   // the lane whose sequences hold block j
  int32_t r = j - __builtin_amdgcn_readlane(incl - mine, src);
  b = src * per;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int32_t n = __builtin_amdgcn_readlane(w[k], src);
    if (r < n) {
      const int32_t blocks = __builtin_amdgcn_readlane(nb[k], src);
      b += k;
      c0 = __builtin_amdgcn_readlane(at[k], src);
      len = __builtin_amdgcn_readlane(at[k + 1], src) - c0;
      const int32_t mixed = n - blocks * eights;   // this XCD's share of the dealt blocks comes first
      if (r < mixed) {
        const int32_t u = ((xcd - b * rest) & (kXcds - 1)) + kXcds * r, q = u / rest;
        h = kXcds * eights + u - q * rest;
        qb = blocks - 1 - q;
      } else {
        const int32_t i = (r - mixed) / blocks;
        h = xcd + kXcds * i;
        qb = blocks - 1 - (r - mixed - i * blocks);
      }
      break;
    }
    r -= n;
  }
  return true;
}

// PADDED = false: Q, K, V are thirds of the packed [T, 3A] rows, the output is packed [T, A], and
// only the len[b] real queries of a sequence are computed.  PADDED = true (the paper's own path,
// Sec. 4.3): q, k, v, out are [B, nh, S, d] with zeros at the pads, all S queries are computed,
// and a key is allowed iff it is <= the query and < len[b].
template <typename E, int D, bool PADDED>
__global__ __launch_bounds__(kAttnWaves * 64, D == 128 ? 2 : 3) void attention_mfma_kernel(
    const E* __restrict__ qptr, const E* __restrict__ kptr, const E* __restrict__ vptr, E* __restrict__ out,
    const int32_t* __restrict__ cu, int32_t B, int32_t nh, int32_t n_qblocks, int32_t group,
    int32_t S) {
  constexpr int KS = D / 16;                 // 16-wide steps of the head dimension (S^T contraction)
  constexpr int DB = D / 32;                 // 32-row blocks of O^T
  constexpr int KC = D / 8;                  // 16-byte chunks per row
  constexpr int ROWS = 64 / KC;              // rows moved by one direct-to-LDS instruction (1 KiB)
  constexpr int QDMA = kWQ / ROWS;           // such instructions for a wavefront's queries
  constexpr int KDMA = kBKV / ROWS / kAttnWaves;   // per wavefront and K (or V) tile
  constexpr int G = 2 * KDMA;                // per wavefront and stage
  constexpr int kTile = kBKV * KC;           // 16-byte vectors per K or V tile
  constexpr int kStage = 2 * kTile;
  static_assert(KDMA >= 1, "a tile is at least one instruction per wavefront");
  static_assert(kAttnWaves == 4 && kWQ == 32 && kBKV == 32 && kStages == 4, "the queries fill two stages, 8 rows a part");
  extern __shared__ uint4 lds[];             // [kStages][K tile, V tile]

  const int tid = threadIdx.x, lane = tid & 63;
  int32_t b, h, qb, c0, len;
  if (!attn_block(cu, B, nh, n_qblocks, group, lane, b, h, qb, c0, len)) return;
  const int32_t q0 = qb * kBQ;
  const int32_t n_queries = PADDED ? S : len;   // queries of this sequence that are computed
  if (q0 >= n_queries) return;  // whole workgroup leaves before any barrier

  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hf = lane >> 5;
  const int32_t A = nh * D;
  // row stride and first row of this (sequence, head) in each operand
  const size_t ld = PADDED ? (size_t)D : (size_t)3 * A;
  const size_t first = PADDED ? ((size_t)b * nh + h) * S * D : (size_t)c0 * ld + (size_t)h * D;

  const int32_t wq_first = q0 + kWQ * wave, wq_last = wq_first + kWQ - 1;
  const int32_t qi = wq_first + lq;
  const int32_t kv_end = min(q0 + kBQ, len);           // keys 0 .. kv_end-1 are needed
  const int32_t n_tiles = (kv_end + kBKV - 1) / kBKV;

  // Addresses inside this (sequence, head): a wavefront-uniform base plus a 32-bit byte offset
  // (the launcher checks that S rows fit in 32 bits).
  const char* qbytes = reinterpret_cast<const char*>(qptr + first);
  const char* kbytes = reinterpret_cast<const char*>(kptr + first);
  const char* vbytes = reinterpret_cast<const char*>(vptr + first);
  const uint32_t ld_b = (uint32_t)(ld * sizeof(E));
  // this lane's part of a transfer: row lr of the instruction's ROWS rows, LDS slot sl of that row
  const int lr = lane / KC, sl = lane % KC;
  uint32_t kcol[KDMA], vcol[KDMA];   // byte offset of the chunk this lane fetches, inside its row
#pragma unroll
  for (int i = 0; i < KDMA; ++i) {
    const int row = (wave * KDMA + i) * ROWS + lr;
    kcol[i] = (uint32_t)((sl ^ kswz<D>(row)) * 16);
    vcol[i] = (uint32_t)((sl ^ vswz<D>(row)) * 16);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(attn_lptr_t)lds;   // LDS byte address of the ring
  auto issue = [&](int32_t t) {   // K and V rows of tile t into its stage; keys past the end read the last row
    const uint32_t st = lds0 + (uint32_t)(t % kStages) * (kStage * 16);
#pragma unroll
    for (int i = 0; i < KDMA; ++i) {
      const int32_t row = (wave * KDMA + i) * ROWS;
      int32_t key = t * kBKV + row + lr; key = key < len ? key : len - 1;
      dma16(kbytes, (uint32_t)key * ld_b + kcol[i], st + row * (KC * 16));
      dma16(vbytes, (uint32_t)key * ld_b + vcol[i], st + (kTile + row * KC) * 16);
    }
  };

  // Prologue: the wavefront's queries go through the parts of the last two stages that its own loads of tiles 2
  // and 3 will fill (8 rows of each K and V tile; whole lines, the K tile's swizzle), so they are free for those
  // as soon as this wavefront has read its queries.
  auto q_vec = [&](int row) { return (2 + (row >> 4)) * kStage + ((row >> 3) & 1) * kTile + (wave * 8 + (row & 7)) * KC; };
#pragma unroll
  for (int i = 0; i < QDMA; ++i) {
    const int32_t row = i * ROWS + lr;
    const int32_t qc = min(wq_first + row, n_queries - 1);
    dma16(qbytes, (uint32_t)qc * ld_b + (uint32_t)((sl ^ kswz<D>(row)) * 16), lds0 + (uint32_t)q_vec(i * ROWS) * 16);
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
    if (t < n_tiles) issue(t);

  f32x16 oacc[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[i][e] = 0.f;
  // reference in log2 units (already scaled), running sum.  The reference starts at the lowest finite value: where every
  // score so far is -inf (products that overflow), a difference of two -inf would be NaN; so weights are 0 and nothing is lost.
  float m_run = kLowest, l_run = 0.f;
  const float sc = rsqrtf((float)D) * kLog2e;  // raw score -> log2 units

  uint32_t koff[KS], voff[DB];   // this lane's operand reads: 16-byte vectors of the K tile, bytes of the V tile
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) koff[ks] = (uint32_t)(lq * KC + ((2 * ks + hf) ^ kswz<D>(lq)));
  {
    // V is read transposed: in each group of 16 lanes, lane i gives the address of 4 elements, key row i / 4,
    // and receives column i of the 4 x 16 block.  Group g: dd 16 (g & 1) .., keys 4 (g >> 1) ..
    const int row = 4 * hf + ((lane & 15) >> 2), c = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
#pragma unroll
    for (int i = 0; i < DB; ++i) voff[i] = (uint32_t)((row * KC + ((4 * i + c) ^ vswz<D>(row))) * 16 + (lane & 1) * 8);
  }

  vec8<E> qf[KS];
  attn_wait<G>(min(2, n_tiles));   // the queries
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const vec8<E>*>(&lds[q_vec(lq) + ((2 * ks + hf) ^ kswz<D>(lq))]);
  attn_wait<G>(min(2, n_tiles));   // read
#pragma unroll
  for (int t = 2; t < 4; ++t)
    if (t < n_tiles) issue(t);

  // Tiles are worked on in pairs, so that the running max, the rescaling of the accumulators (nearly always due:
  // some query of 32 has a new max) and the barrier come once per 64 keys.  At the start of a pair: it has landed
  // (this wavefront's part) and this wavefront's reads of the pair before are back; past the barrier that holds
  // for every wavefront, so the stages of the pair before are free for the next one.
  auto advance = [&](int32_t t) {
    attn_wait<G>(t == 0 ? max(0, min(2, n_tiles - 2)) : 0);
    __builtin_amdgcn_s_barrier();
    if (t > 0) {
#pragma unroll
      for (int i = 2; i < 4; ++i)
        if (t + i < n_tiles) issue(t + i);
    }
  };
  // N = 2: tiles t, t + 1; N = 1: tile t only (the other one is above this wavefront's diagonal or past the end).
  // The second tile's K operands are read while the matrix cores work on the first, the V operands during the softmax.
  auto work = [&](auto n, int32_t t) {
    constexpr int N = decltype(n)::value;
    const int32_t k0 = t * kBKV;
    const uint4* const st0 = lds + (t & 2) * kStage;   // t is even: the pair's stages are adjacent
    vec8<E> kf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kf[ks] = *reinterpret_cast<const vec8<E>*>(&st0[koff[ks]]);
    f32x16 sacc[N];
    vec8<E> k2[KS];
#pragma unroll
    for (int a = 0; a < N; ++a)
#pragma unroll
      for (int e = 0; e < 16; ++e) sacc[a][e] = 0.f;
    if constexpr (N == 2) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) k2[ks] = *reinterpret_cast<const vec8<E>*>(&st0[kStage + koff[ks]]);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) sacc[0] = Mfma<E>::m32x32x16(kf[ks], qf[ks], sacc[0]);
    if constexpr (N == 2) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) sacc[1] = Mfma<E>::m32x32x16(k2[ks], qf[ks], sacc[1]);
    }
    vec4<E> vf[N][2][DB][2];
#pragma unroll
    for (int a = 0; a < N; ++a)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < DB; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            vf[a][s][i][j] = Mfma<E>::read_tr((attn_lptr_t)(st0 + a * kStage + kTile), voff[i] + (16 * s + 8 * j) * (D * 2));
    __builtin_amdgcn_sched_barrier(0);
    // Mask (only on tiles that touch the diagonal or, on the padded path, the end of the
    // sequence: wavefront-uniform), then the max of the raw scores.  Packed: the causal
    // mask also hides keys >= len (they are > every real query).  Padded: pad queries lie beyond
    // len, so keys >= len are masked explicitly.
    if (k0 + N * kBKV - 1 > wq_first || (PADDED && k0 + N * kBKV > len)) {
#pragma unroll
      for (int a = 0; a < N; ++a)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int32_t key = k0 + a * kBKV + 8 * (e >> 2) + 4 * hf + (e & 3);
          if (key > qi || (PADDED && key >= len)) sacc[a][e] = -INFINITY;
        }
    }
    float mx = sacc[0][0];
#pragma unroll
    for (int a = 0; a < N; ++a)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, sacc[a][e]);
    {  // the query's other keys are in lane ^ 32
      const auto o = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      mx = fmaxf(__uint_as_float(o[0]), __uint_as_float(o[1]));
    }
    const float m_new = fmaxf(m_run, mx * sc);
    const float corr = __builtin_amdgcn_exp2f(m_run - m_new);
    float psum[2] = {0.f, 0.f};
    vec8<E> pf[N][2];
#pragma unroll
    for (int a = 0; a < N; ++a)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sacc[a][e], sc, -m_new));
        psum[e & 1] += p;
        pf[a][e >> 3][e & 7] = static_cast<E>(p);
      }
    l_run = l_run * corr + (psum[0] + psum[1]);
    if (__any(m_new != m_run)) {                 // wavefront-uniform
#pragma unroll
      for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[i][e] *= corr;
    }
    m_run = m_new;
    // O^T += V^T P^T; step s: element j of lane half hf is key 16 s + 8 (j / 4) + 4 hf + j % 4, as in the accumulator
#pragma unroll
    for (int a = 0; a < N; ++a)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < DB; ++i)
          oacc[i] = Mfma<E>::m32x32x16(__builtin_shufflevector(vf[a][s][i][0], vf[a][s][i][1], 0, 1, 2, 3, 4, 5, 6, 7),
                                       pf[a][s], oacc[i]);
  };
  const int32_t n_mine = min(n_tiles, wq_last / kBKV + 1);   // tiles at or below this wavefront's diagonal
  int32_t t = 0;
  for (; t + 1 < n_mine; t += 2) {
    advance(t);
    work(std::integral_constant<int, 2>{}, t);
  }
  if (t < n_mine) {
    advance(t);
    work(std::integral_constant<int, 1>{}, t);
    t += 2;
  }
  for (; t < n_tiles; t += 2) advance(t);   // pairs above the diagonal: the other wavefronts' loads and barriers

  // Results leave through LDS as whole rows (straight from the accumulators a store would write 16 bytes of
  // each of 32 rows).  Every wavefront uses a part of its own, without a barrier: other wavefronts may still be
  // reading the last pair of tiles, so the parts lie in the other pair's stages.
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  const float inv = n_tiles > 0 ? 1.0f / l_tot : 0.f;   // no allowed key at all (len = 0): a zero row
  char* const os = reinterpret_cast<char*>(lds + ((((n_tiles - 1) & 2) ^ 2) + (wave >> 1)) * kStage + (wave & 1) * kTile);
#pragma unroll
  for (int i = 0; i < DB; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {   // dd 32 i + 8 j + 4 hf .. + 3 of query lq
      vec4<E> o4;
#pragma unroll
      for (int e = 0; e < 4; ++e) o4[e] = static_cast<E>(oacc[i][4 * j + e] * inv);
      *reinterpret_cast<vec4<E>*>(os + (lq * KC + ((4 * i + j) ^ kswz<D>(lq))) * 16 + 8 * hf) = o4;
    }
  const size_t old = PADDED ? (size_t)D : (size_t)A;
  E* const obase = (PADDED ? out + first : out + (size_t)c0 * A + (size_t)h * D) + (size_t)(wq_first + lr) * old + sl * 8;
  uint4 ov[QDMA];
#pragma unroll
  for (int i = 0; i < QDMA; ++i) ov[i] = *reinterpret_cast<const uint4*>(os + ((i * ROWS + lr) * KC + (sl ^ kswz<D>(i * ROWS + lr))) * 16);
  if (wq_last < n_queries) {
#pragma unroll
    for (int i = 0; i < QDMA; ++i) *reinterpret_cast<uint4*>(obase + (size_t)(i * ROWS) * old) = ov[i];
  } else {
#pragma unroll
    for (int i = 0; i < QDMA; ++i)
      if (wq_first + i * ROWS + lr < n_queries) *reinterpret_cast<uint4*>(obase + (size_t)(i * ROWS) * old) = ov[i];
  }
}

template <typename E, int D, bool PADDED>
static hipError_t launch_d(const E* q, const E* k, const E* v, E* out, const int32_t* cu, int64_t T, int32_t B,
                           int32_t max_len, int32_t nh, hipStream_t s) {
  auto kern = attention_mfma_kernel<E, D, PADDED>;
  constexpr size_t lds = kStages * 2 * (size_t)(kBKV * D * 2);
  static LdsAttrOnce once;
  {
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds, once);
    if (e != hipSuccess) return e;
  }
  const int32_t n_qblocks = (max_len + kBQ - 1) / kBQ;
  const int64_t pairs = (int64_t)B * nh, whole = pairs / kXcds, rest = pairs % kXcds, all = pairs * n_qblocks;
  // sum of ceil(len / kBQ) <= T / kBQ + B per head; where that is at least a fifth less than the blocks of max_len, the
  // blocks are counted by a scan (which costs a workgroup about half a microsecond), unless the launch is small and
  // at least half full, where balance is worth more: 8 sequences of up to 2048 x 25 heads x 64 103 against 80 us.
  // Without a scan, groups pay from three tenths full (400 of up to 1000 x 16 heads x 128, 0.66: 1.71 ms longest first, 1.15 in
  // groups; 300 x 12 heads x 64 with one of 4096 among short ones, 0.07: 135 and 200 us).
  const int64_t filled = T / kBQ + B, most = (int64_t)B * n_qblocks;
  const bool few = 2 * all <= 9 * 256 * (D == 128 ? 2 : 3);   // 4.5 rounds of 2 or 3 workgroups per CU
  const bool sparse = !PADDED && 5 * filled <= 4 * most;
  const bool scan = sparse && B <= kAttnScan && !(few && 2 * filled > most);
  const bool grouped = !scan && !few && n_qblocks > 1 && whole > 0 && (PADDED || 10 * filled > 3 * most);
  const int64_t groups = (whole + kAttnGroup - 1) / kAttnGroup;
  const int32_t group = grouped ? (int32_t)((whole + groups - 1) / groups) : 0;
  const int64_t per_xcd = scan ? filled * (nh / kXcds) + (filled * (nh % kXcds) + 7 * (int64_t)B) / kXcds
                        : grouped ? whole * n_qblocks + (rest * n_qblocks + kXcds - 1) / kXcds
                                  : (all + kXcds - 1) / kXcds;
  kern<<<dim3((unsigned)(per_xcd * kXcds)), dim3(kAttnWaves * 64), lds, s>>>(q, k, v, out, cu, B, nh, scan ? 0 : n_qblocks,
                                                                            group, max_len);
  return hipGetLastError();
}

template <typename E>
static hipError_t launch_packed(const E* qkv, E* out, const int32_t* cu, int64_t T, int32_t B, int32_t max_len,
                                int32_t nh, int32_t d, hipStream_t s) {
  if (B <= 0 || max_len <= 0) return hipSuccess;
  const size_t A = (size_t)nh * d;
  return d == 128 ? launch_d<E, 128, false>(qkv, qkv + A, qkv + 2 * A, out, cu, T, B, max_len, nh, s)
                  : launch_d<E, 64, false>(qkv, qkv + A, qkv + 2 * A, out, cu, T, B, max_len, nh, s);
}

template <typename E>
static hipError_t launch_padded(const E* q, const E* k, const E* v, E* out, const int32_t* cu, int32_t B, int32_t S,
                                int32_t nh, int32_t d, hipStream_t s) {
  if (B <= 0 || S <= 0) return hipSuccess;
  return d == 128 ? launch_d<E, 128, true>(q, k, v, out, cu, 0, B, S, nh, s)
                  : launch_d<E, 64, true>(q, k, v, out, cu, 0, B, S, nh, s);
}

hipError_t launch_attention_bf16(const bf16_t* qkv, bf16_t* out, const int32_t* cu, int64_t T, int32_t B,
                                 int32_t max_len, int32_t nh, int32_t d, hipStream_t s) {
  return launch_packed<bf16_t>(qkv, out, cu, T, B, max_len, nh, d, s);
}
hipError_t launch_attention_f16(const f16_t* qkv, f16_t* out, const int32_t* cu, int64_t T, int32_t B,
                                int32_t max_len, int32_t nh, int32_t d, hipStream_t s) {
  return launch_packed<f16_t>(qkv, out, cu, T, B, max_len, nh, d, s);
}
hipError_t launch_attention_padded_bf16(const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* out,
                                        const int32_t* cu, int32_t B, int32_t S, int32_t nh, int32_t d, hipStream_t s) {
  return launch_padded<bf16_t>(q, k, v, out, cu, B, S, nh, d, s);
}
hipError_t launch_attention_padded_f16(const f16_t* q, const f16_t* k, const f16_t* v, f16_t* out, const int32_t* cu,
                                       int32_t B, int32_t S, int32_t nh, int32_t d, hipStream_t s) {
  return launch_padded<f16_t>(q, k, v, out, cu, B, S, nh, d, s);
}

}  // namespace energon
