// The two layout kernels of the paper's own attention path (Sec. 4.3): the attention core
// stays padded there, so padding is rebuilt in front of it and removed behind it, each fused
// with the head transpose.
//   rebuild:  packed [T, 3A] (Q | K | V, head-major)  ->  q, k, v  [B, nh, S, d], zeros at pads
//   remove :  padded [B, nh, S, d]                    ->  packed [T, A]
// Both are plain copies in 16-byte vectors, HBM-bound: rebuild moves T*3A*e + B*S*3A*e bytes, remove 2*T*A*e.  Each
// writes in long runs and reads in head slices (128 or 256 bytes); all loads of a lane are issued before its first store.
//  * rebuild: a wavefront moves one head's slices of 32 (d = 128) or 64 consecutive positions, 8 KiB that are
//    contiguous on the head-major side; the four wavefronts of a workgroup take neighbouring heads.  (One wavefront per
//    position scattered a head's slice every S*d elements and found its head by two divisions per vector:
//    32 x 512 positions, 40 heads of 128, 160 -> 132 us, 5.8 TB/s.)
//  * remove: a wavefront writes one packed row.  (Moved the way rebuild is, scattering its stores, it takes twice as long.)
#include "common.h"

namespace energon {

constexpr int kMoveVecs = 8;   // 16-byte vectors per lane and batch

// This workgroup's sequence, first position and group of four heads; ids walk the groups of heads fastest, so that
// workgroups side by side read (or write) the same packed rows.
struct DrceBlock { int32_t b, s0, head; };
__device__ __forceinline__ DrceBlock drce_block(int32_t S, int32_t groups, int32_t positions) {
  const int32_t chunks = (S + positions - 1) / positions;
  const int32_t at = blockIdx.x / groups;
  const int32_t b = at / chunks;
  return {b, (at - b * chunks) * positions, (int32_t)(blockIdx.x - at * groups) * 4 + (int32_t)(threadIdx.x >> 6)};
}

// HV = 16-byte vectors per head, VECS = 16-byte vectors per lane
template <int HV, int VECS>
__global__ __launch_bounds__(256) void rebuild_qkv_kernel(const uint4* __restrict__ qkv, uint4* __restrict__ q,
                                                          uint4* __restrict__ k, uint4* __restrict__ v,
                                                          const int32_t* __restrict__ cu, int32_t S, int32_t nh,
                                                          int32_t groups) {
  constexpr int R = 64 / HV;   // positions per load of the wavefront
  const DrceBlock at = drce_block(S, groups, VECS * R);
  if (at.head >= 3 * nh) return;   // head of Q, K or V
  const int lane = threadIdx.x & 63, sub = lane % HV;
  const int32_t c0 = cu[at.b], len = cu[at.b + 1] - c0;
  const int32_t which = at.head / nh, h = at.head - which * nh, s = at.s0 + lane / HV;
  const uint4* src = qkv + ((size_t)(c0 + s) * 3 * nh + at.head) * HV + sub;
  uint4* dst = (which == 0 ? q : which == 1 ? k : v) + (((size_t)at.b * nh + h) * S + s) * HV + sub;
  uint4 r[VECS];
#pragma unroll
  for (int i = 0; i < VECS; ++i) {
    r[i] = make_uint4(0, 0, 0, 0);
    if (s + i * R < len) r[i] = src[(size_t)(i * R) * 3 * nh * HV];
  }
#pragma unroll
  for (int i = 0; i < VECS; ++i)
    if (s + i * R < S) dst[i * 64] = r[i];
}

// The same where a sequence has few positions: rows of a sequence's [nh, S] block, head after head, so that a wavefront's
// 8 KiB still are one run.
template <int HV>
__global__ __launch_bounds__(256) void rebuild_short_kernel(const uint4* __restrict__ qkv, uint4* __restrict__ q,
                                                            uint4* __restrict__ k, uint4* __restrict__ v,
                                                            const int32_t* __restrict__ cu, int32_t B, int32_t S,
                                                            int32_t nh, int32_t chunks) {
  constexpr int R = 64 / HV;   // rows per load of the wavefront
  const int32_t id = (int32_t)blockIdx.x * 4 + (int32_t)(threadIdx.x >> 6);
  const int32_t b = id / (3 * chunks), at = id - b * 3 * chunks, which = at / chunks;
  if (b >= B) return;
  const int lane = threadIdx.x & 63, sub = lane % HV;
  const int32_t c0 = cu[b], len = cu[b + 1] - c0, rows = nh * S;
  const int32_t row0 = (at - which * chunks) * (kMoveVecs * R) + lane / HV;
  const uint4* src = qkv + ((size_t)c0 * 3 + which) * nh * HV + sub;
  uint4* dst = (which == 0 ? q : which == 1 ? k : v) + (size_t)b * rows * HV + sub;
  uint4 r[kMoveVecs];
#pragma unroll
  for (int i = 0; i < kMoveVecs; ++i) {
    const int32_t row = row0 + i * R, h = row / S, s = row - h * S;
    r[i] = make_uint4(0, 0, 0, 0);
    if (row < rows && s < len) r[i] = src[((size_t)s * 3 * nh + h) * HV];
  }
#pragma unroll
  for (int i = 0; i < kMoveVecs; ++i)
    if (row0 + i * R < rows) dst[(size_t)(row0 + i * R) * HV] = r[i];
}

template <int HV>
__global__ __launch_bounds__(256) void remove_padding_heads_kernel(const uint4* __restrict__ o, uint4* __restrict__ out,
                                                                   const int32_t* __restrict__ cu, int32_t B, int32_t S,
                                                                   int32_t nh) {
  const int64_t p = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // padded position
  if (p >= (int64_t)B * S) return;
  const int lane = threadIdx.x & 63;
  const int32_t b = (int32_t)(p / S), s = (int32_t)(p - (int64_t)b * S);
  const int32_t c0 = cu[b], len = cu[b + 1] - c0;
  if (s >= len) return;
  const int32_t rowv = nh * HV;
  const uint4* src = o + ((size_t)b * nh * S + s) * HV;   // head h: S * HV vectors further on each
  uint4* dst = out + (size_t)(c0 + s) * rowv;
  for (int32_t i0 = lane; i0 < rowv; i0 += 64 * kMoveVecs) {
    uint4 r[kMoveVecs];
#pragma unroll
    for (int j = 0; j < kMoveVecs; ++j) {
      const int32_t i = min(i0 + 64 * j, rowv - 1);       // past the row's end: its last vector, dropped
      r[j] = src[(size_t)(i / HV) * S * HV + i % HV];
    }
#pragma unroll
    for (int j = 0; j < kMoveVecs; ++j)
      if (i0 + 64 * j < rowv) dst[i0 + 64 * j] = r[j];
  }
}

template <int HV>
static hipError_t rebuild(const uint4* qkv, uint4* q, uint4* k, uint4* v, const int32_t* cu, int32_t B, int32_t S, int32_t nh,
                          hipStream_t s) {
  constexpr int32_t positions = kMoveVecs * (64 / HV);   // of one head, moved by a wavefront
  const int32_t groups = (3 * nh + 3) / 4;
  const auto blocks = [&](int32_t per) { return (int64_t)B * ((S + per - 1) / per) * groups; };
  // Fewer than an eighth of them filled in a launch of many workgroups: heads behind one another instead (us, one position
  // per wavefront / this / heads' positions: 2000 x 1 position x 40 x 128 24 / 23 / 56, 3000 x 3 x 12 x 64 15.4 / 13.5 / 24.8,
  // 1000 x 4 x 40 x 128 42 / 38 / 37; but 1 x 3 x 40 x 128 5.8 / 3.4 / 2.2).
  if (8 * S < positions && blocks(positions) > 2048) {
    const int32_t chunks = (nh * S + positions - 1) / positions;
    rebuild_short_kernel<HV><<<dim3((unsigned)(((int64_t)B * 3 * chunks + 3) / 4)), dim3(256), 0, s>>>(qkv, q, k, v, cu, B, S, nh,
                                                                                                     chunks);
    return hipGetLastError();
  }
  // Too few workgroups for the chip: a quarter of the vectors per lane, four times as many wavefronts (1 x 64 positions x 4
  // heads of 64: 3.2 -> 2.4 us)
  if (blocks(positions) < 256)
    rebuild_qkv_kernel<HV, kMoveVecs / 4><<<dim3((unsigned)blocks(positions / 4)), dim3(256), 0, s>>>(qkv, q, k, v, cu, S, nh, groups);
  else
    rebuild_qkv_kernel<HV, kMoveVecs><<<dim3((unsigned)blocks(positions)), dim3(256), 0, s>>>(qkv, q, k, v, cu, S, nh, groups);
  return hipGetLastError();
}

// head_bytes = 128 or 256
hipError_t launch_rebuild_qkv(const void* qkv, void* q, void* k, void* v, const int32_t* cu, int32_t B, int32_t S,
                              int32_t nh, int32_t head_bytes, hipStream_t s) {
  const auto f = head_bytes == 256 ? rebuild<16> : rebuild<8>;
  return f(static_cast<const uint4*>(qkv), static_cast<uint4*>(q), static_cast<uint4*>(k), static_cast<uint4*>(v), cu, B, S, nh, s);
}

hipError_t launch_remove_padding_heads(const void* o, void* out, const int32_t* cu, int32_t B, int32_t S, int32_t nh,
                                       int32_t head_bytes, hipStream_t s) {
  const int64_t blocks = ((int64_t)B * S + 3) / 4;
  const auto kern = head_bytes == 256 ? remove_padding_heads_kernel<16> : remove_padding_heads_kernel<8>;
  kern<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(static_cast<const uint4*>(o), static_cast<uint4*>(out), cu, B, S, nh);
  return hipGetLastError();
}

}  // namespace energon
