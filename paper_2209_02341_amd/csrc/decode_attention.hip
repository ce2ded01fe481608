// Attention of one generation step: one new token per sequence attends the keys / values cached
// for its sequence's earlier tokens plus its own.  The paper (Sec. 2.2) defines the decoder block
// with a causal mask; under that mask earlier tokens' K and V rows never change, so a step needs
// only the cache and the new token's q, k, v.  Every sequence has its own cached length: as in the
// paper's padding elimination (Sec. 4.3), no position beyond a sequence's real length is touched.
//
// The work is one pass over the cached rows (2 * d * e bytes per key and head, each used once):
// bound by HBM, so there is no MFMA here.  One workgroup (4 or 8 wavefronts) per (sequence, head), or per part of its keys
// where there are few of them; a key's head slice (d elements) is spread over d / 8 lanes, 16 bytes each, so a
// wavefront takes 64 / (d / 8) keys per step with fully coalesced loads.  Each lane group runs its own online softmax
// over the keys it sees, one or two steps' loads ahead of its arithmetic; the groups' states are merged by lane
// exchanges, the wavefronts' through LDS, the parts' by the workgroup that finishes last, always in a fixed order.  The new
// token's k and v are read from the qkv row and written to the cache row at the sequence's length.
// About 5.4 TB/s on long caches of many sequences (96 x 40 heads of 200 keys: 74 us).
#include "common.h"
#include <algorithm>

namespace energon {

namespace {

constexpr float kDecLog2e = 1.4426950408889634f;

// sum over the LPK consecutive lanes that hold one key (LPK = 8 or 16, inside one DPP row)
template <int LPK> __device__ __forceinline__ float key_sum(float v) {
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xF, 0xF, true));  // row_half_mirror
  if constexpr (LPK == 16) v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xF, 0xF, true));  // row_mirror
  return v;
}

// the same value of lane ^ off (off = 8, 16 or 32) combined with the own one, on the vector ALU
template <typename F> __device__ __forceinline__ float with_lane_xor(float v, int off, F f) {
  const unsigned u = __float_as_uint(v);
  if (off == 8) return f(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xF, 0xF, true)));   // row_ror 8
  if (off == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return f(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return f(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float add2(float a, float b) { return a + b; }

// A word that workgroups on other XCDs read in the same launch: written through, and read past, the caches that are
// not shared.  (A release and an acquire fence around plain ones write back and drop a whole L2 each: 8 us.)
__device__ __forceinline__ void put_shared(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float get_shared(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Keys of a part, at least: what is cached decides how many of the launch's parts a (sequence, head) uses.
constexpr int kDecPartKeys = 256;

// grid = (B * nh, parts): part y of a (sequence, head) takes the y-th of equal shares of its keys.  A share has
// kDecPartKeys or more, so short sequences use fewer parts than were launched and the rest leaves at once.  With one
// part the result goes straight to out; otherwise each leaves its state (running max, running sum, D sums) in
// part[(y * B * nh + x) * (D + 2)], counts itself in arrived[x] (zero at the start of the launch), and the one that
// counts last adds all of them in their order: no second launch, and nobody waits.
template <typename E, int D, int NW, int U, bool PARTS>
__global__ __launch_bounds__(NW * 64) void decode_attention_kernel(const E* __restrict__ qkv, E* k_cache, E* v_cache,
                                                                  const int32_t* __restrict__ lens, int32_t nh,
                                                                  int32_t S_cap, E* __restrict__ out, float* part,
                                                                  int32_t* arrived) {
  constexpr int LPK = D / 8;          // lanes per key
  constexpr int KPW = 64 / LPK;       // keys per wavefront step
  constexpr int KPB = KPW * NW;       // keys per step of the workgroup
  __shared__ float st_m[NW], st_l[NW];
  __shared__ float st_o[NW][D];

  const int32_t b = blockIdx.x / nh, h = blockIdx.x % nh;
  const int32_t A = nh * D;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sub = lane % LPK, slot = wave * KPW + lane / LPK;   // which 8 elements of d; which key of a step
  int32_t p = lens[b];
  p = p < 0 ? 0 : (p > S_cap ? S_cap : p);     // cached keys; the new token is key p
  const int32_t parts = PARTS ? min((int32_t)gridDim.y, p / kDecPartKeys + 1) : 1, y = PARTS ? (int32_t)blockIdx.y : 0;
  if (y >= parts) return;
  const int32_t share = (p + parts) / parts;   // ceil((p + 1) / parts)
  const int32_t first = y * share, end = min(first + share, p + 1);

  const E* qrow = qkv + (size_t)b * 3 * A + (size_t)h * D + sub * 8;
  const vec8<E> q8 = *reinterpret_cast<const vec8<E>*>(qrow);
  const E* knew = qrow + A;
  const E* vnew = qrow + 2 * A;
  const float sc = rsqrtf((float)D) * kDecLog2e;
  float q[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) q[e] = static_cast<float>(q8[e]) * sc;

  const size_t head_off = (size_t)b * S_cap * A + (size_t)h * D + sub * 8;
  const E* kc = k_cache + head_off;
  const E* vc = v_cache + head_off;

  // append: the new token's k and v become cache row p (one wavefront's first LPK lanes)
  if (y == 0 && wave == 0 && lane < LPK && p < S_cap) {
    *reinterpret_cast<vec8<E>*>(k_cache + head_off + (size_t)p * A) = *reinterpret_cast<const vec8<E>*>(knew);
    *reinterpret_cast<vec8<E>*>(v_cache + head_off + (size_t)p * A) = *reinterpret_cast<const vec8<E>*>(vnew);
  }

  // the running max starts at the lowest finite value: where every score so far is -inf (products that overflow), the
  // weights are 2^-inf = 0 and not 2^(-inf + inf) = NaN
  float m_run = kLowest, l_run = 0.f, o[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = 0.f;

  // U steps' loads are in flight while the U steps before are worked on
  vec8<E> k8[2][U], v8[2][U];
  auto load = [&](int s, int32_t j0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t j = j0 + u * KPB + slot;
      // key p is the new token (read from the qkv row, never from the cache row written above);
      // keys past it are clamped to it and masked below
      const bool cached = j < p;
      k8[s][u] = *reinterpret_cast<const vec8<E>*>(cached ? kc + (size_t)j * A : knew);
      v8[s][u] = *reinterpret_cast<const vec8<E>*>(cached ? vc + (size_t)j * A : vnew);
    }
  };
  auto step = [&](int s, int32_t j0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t j = j0 + u * KPB + slot;
      float x = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) x = fmaf(q[e], static_cast<float>(k8[s][u][e]), x);
      x = key_sum<LPK>(x);                       // the key's score in log2 units, in all its lanes
      if (j < end) {
        const float m_new = fmaxf(m_run, x);
        const float corr = __builtin_amdgcn_exp2f(m_run - m_new);   // first key: 0 (times sums of 0)
        const float pw = __builtin_amdgcn_exp2f(x - m_new);
        l_run = fmaf(l_run, corr, pw);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = fmaf(o[e], corr, pw * static_cast<float>(v8[s][u][e]));
        m_run = m_new;
      }
    }
  };
  constexpr int kTrip = KPB * U;
  const int32_t last = end - wave * KPW;   // a wavefront whose keys of a trip all lie behind the end leaves
  if (first < last) load(0, first);
  for (int32_t j0 = first; j0 < last; j0 += 2 * kTrip) {
    if (j0 + kTrip < last) load(1, j0 + kTrip);
    step(0, j0);
    if (j0 + kTrip < last) {
      if (j0 + 2 * kTrip < last) load(0, j0 + 2 * kTrip);
      step(1, j0 + kTrip);
    }
  }

  // Merge the wavefront's KPW states by lane exchanges, then the wavefronts' through LDS: weights 2^(m_i - M); a
  // state that saw no key of weight has m = kLowest, l = 0, o = 0.
  float M = m_run;
#pragma unroll
  for (int off = LPK; off < 64; off <<= 1) M = with_lane_xor(M, off, fmaxf);
  const float wgt = __builtin_amdgcn_exp2f(m_run - M);
  l_run *= wgt;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] *= wgt;
#pragma unroll
  for (int off = LPK; off < 64; off <<= 1) {
    l_run = with_lane_xor(l_run, off, add2);
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = with_lane_xor(o[e], off, add2);
  }
  if (lane < LPK) {
    if (lane == 0) { st_m[wave] = M; st_l[wave] = l_run; }
#pragma unroll
    for (int e = 0; e < 8; ++e) st_o[wave][sub * 8 + e] = o[e];
  }
  __syncthreads();
  E* const orow = out + (size_t)b * A + (size_t)h * D;
  const size_t stride = (size_t)gridDim.x * (D + 2);   // of a part's states
  if (tid < D) {
    M = st_m[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) M = fmaxf(M, st_m[i]);
    float L = 0.f, acc = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const float w = __builtin_amdgcn_exp2f(st_m[i] - M);
      L = fmaf(st_l[i], w, L);
      acc = fmaf(st_o[i][tid], w, acc);
    }
    if (!PARTS || parts == 1) {
      orow[tid] = static_cast<E>(acc / L);   // key 0 exists: L > 0
    } else {
      float* dst = part + y * stride + (size_t)blockIdx.x * (D + 2);
      put_shared(dst + 2 + tid, acc);
      if (tid == 0) { put_shared(dst, M); put_shared(dst + 1, L); }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // they have arrived before the workgroup is counted
    }
  }
  if (!PARTS || parts == 1) return;
  __shared__ int32_t st_last;
  __syncthreads();
  if (tid == 0) st_last = __hip_atomic_fetch_add(arrived + blockIdx.x, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == parts - 1;
  __syncthreads();
  if (!st_last || tid >= D) return;
  const float* src = part + (size_t)blockIdx.x * (D + 2);
  M = kLowest;
  float L = 0.f, acc = 0.f;
  for (int32_t i0 = 0; i0 < parts; i0 += 8) {   // eight states requested before the first is used
    float m[8], l[8], a[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float* st = src + min(i0 + i, parts - 1) * stride;
      m[i] = get_shared(st);
      l[i] = get_shared(st + 1);
      a[i] = get_shared(st + 2 + tid);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i0 + i >= parts) break;
      const float m_new = fmaxf(M, m[i]);
      const float corr = __builtin_amdgcn_exp2f(M - m_new), w = __builtin_amdgcn_exp2f(m[i] - m_new);
      L = fmaf(L, corr, l[i] * w);
      acc = fmaf(acc, corr, a[i] * w);
      M = m_new;
    }
  }
  orow[tid] = static_cast<E>(acc / L);
}

// Parts that are launched for a (sequence, head)'s keys: as many as bring the launch to about 512 workgroups, each with
// at least 512 of the cache's rows, if the scratch holds their states.  How many of them are used is decided by what is
// cached (kDecPartKeys), so a short conversation in a long cache pays nothing.  Whole steps, us, uncut / cut: 2 of 4000
// keys x 40 heads of 128 227 / 177, 1 of 4000 x 16 x 128 96 / 48; 2 of 100 in a cache of 16384 40.7 / 39.1 (with the parts
// counted from the capacity and added by a second launch: 50.6).  From 256 pairs on nothing is cut.
int32_t dec_parts(int64_t pairs, int32_t S_cap) {
  if (pairs >= 256) return 1;
  return (int32_t)std::max<int64_t>(1, std::min<int64_t>({32, 512 / pairs, S_cap / 512}));
}

template <typename E, int D>
hipError_t launch_dec(const E* qkv, E* kc, E* vc, const int32_t* lens, int32_t B, int32_t S_cap, int32_t nh, E* out,
                      float* scratch, size_t scratch_bytes, int32_t* arrived, hipStream_t s) {
  const int64_t pairs = (int64_t)B * nh;
  const size_t state = (size_t)pairs * (D + 2) * sizeof(float);
  const int32_t fit = scratch != nullptr && arrived != nullptr ? (int32_t)std::min<size_t>(scratch_bytes / state, 32) : 1;
  const int32_t parts = std::max(1, std::min(dec_parts(pairs, S_cap), fit));
  // With a workgroup per CU or less, eight wavefronts and two steps ahead: 40 heads of 4000 keys 60 us with four wavefronts,
  // 43 with eight.  Beyond, four: where the keys are few, eight only take longer to start (us, eight / four: 4096 heads of
  // 50 keys x 64 18.7 / 12.7, 768 of 100 5.4 / 4.6, 3840 x 128 of 500 178 / 181).  From two and a half to eight workgroups per CU
  // their number hides the latency, and one step ahead leaves room for more of them (one / two: 400 x 128 of 2000 keys
  // 112 / 81, 640 128 / 129, 1024 of 1000 94 / 99, 1280 of 300 30.8 / 31.2, 3840 of 500 184 / 181).
  const bool few = pairs <= 256;
  const auto kern = few ? decode_attention_kernel<E, D, 8, 2, true>
                  : pairs >= 640 && pairs <= 2048 ? decode_attention_kernel<E, D, 4, 1, false>
                                                  : decode_attention_kernel<E, D, 4, 2, false>;
  kern<<<dim3((unsigned)pairs, (unsigned)parts), dim3(few ? 8 * 64 : 4 * 64), 0, s>>>(qkv, kc, vc, lens, nh, S_cap, out, scratch,
                                                                                     arrived);
  return hipGetLastError();
}

}  // namespace

size_t decode_attention_scratch_bytes(int64_t B, int32_t nh, int32_t d) {
  const int32_t parts = B > 0 ? dec_parts(B * nh, INT32_MAX) : 1;
  return parts > 1 ? (size_t)(B * nh) * parts * (d + 2) * sizeof(float) : 0;
}

hipError_t launch_decode_attention(const void* qkv, void* k_cache, void* v_cache, const int32_t* lens, int32_t B,
                                   int32_t S_cap, int32_t nh, int32_t d, int dtype, void* out, hipStream_t s,
                                   float* scratch, size_t scratch_bytes, int32_t* arrived) {
  if (B <= 0) return hipSuccess;
#define DEC_CASE(E, D) \
  launch_dec<E, D>((const E*)qkv, (E*)k_cache, (E*)v_cache, lens, B, S_cap, nh, (E*)out, scratch, scratch_bytes, arrived, s)
  return dtype == 1 ? (d == 128 ? DEC_CASE(bf16_t, 128) : DEC_CASE(bf16_t, 64))
                    : (d == 128 ? DEC_CASE(f16_t, 128) : DEC_CASE(f16_t, 64));
#undef DEC_CASE
}

}  // namespace energon
