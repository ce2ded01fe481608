// The two ends of the model around the layer stack, on the packed (padding-free) layout of
// Sec. 4.3; the paper names the embedding layer (Sec. 2.2) without describing it.
//  * embed_packed_kernel: row t of the packed activations = token embedding of ids[t] + learned
//    position embedding of t's position inside its sequence (found from cu_seqlens by bisection);
//    one wavefront per row, 16-byte vectors, one rounding.  HBM-bound: 3 * H * e bytes per token.
//  * cache_fill_kernel: the K and V columns of a prefill's packed QKV rows scattered into the
//    per-sequence cache rows that later generation steps read (the padded positions of the cache
//    are never written and never read).
//  * last_rows_kernel: the row of every sequence's last valid token (what next-token logits are
//    computed from), a zero row for an empty sequence.
#include "common.h"

namespace energon {

namespace {

// U = vectors per lane and source that are requested before the first is stored: a prompt of a few hundred tokens
// gives a CU one workgroup, so its time is the number of memory latencies in a row.  Rows of fewer than four vectors per lane
// go one at a time: batches cost registers there and gain nothing.  Measured (us, embedding, one at a time / five / by the
// row's width): 928 x 4096 5.3 / 5.0 / 4.6, 928 x 8192 10.1 / 7.8 / 7.2, 928 x 5120 6.6 / 4.9 / 4.7, 6000 x 768 4.9 / 5.8 / 4.9.
static int ends_batch(int32_t vecs) {
  const int32_t v = vecs / 64;   // full steps of a row's lanes
  if (v < 4) return 1;
  int best = 4;
  for (const int u : {5, 8})
    if (v >= u && v % u <= v % best) best = u;   // the fewest single steps behind the batches, then the longest batch
  return best;
}

template <typename E, int U>
__global__ __launch_bounds__(256) void embed_packed_kernel(const int32_t* __restrict__ ids,
                                                           const int32_t* __restrict__ cu,
                                                           const int32_t* __restrict__ positions, int32_t B, int64_t T,
                                                           const E* __restrict__ wte, int32_t V,
                                                           const E* __restrict__ wpe, int32_t P, int32_t H,
                                                           E* __restrict__ x) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  int32_t pos;
  if (positions != nullptr) {
    pos = positions[t];                        // a generation step: the position is given per row
  } else {
    // sequence of row t: the last b with cu[b] <= t
    int32_t lo = 0, hi = B;  // invariant: cu[lo] <= t < cu[hi]
    while (hi - lo > 1) {
      const int32_t mid = (lo + hi) >> 1;
      if (cu[mid] <= t) lo = mid; else hi = mid;
    }
    pos = (int32_t)(t - cu[lo]);
  }
  pos = pos < 0 ? 0 : (pos < P ? pos : P - 1);  // out-of-range inputs stay inside the tables
  int32_t id = ids[t];
  id = id < 0 ? 0 : (id < V ? id : V - 1);
  const vec8<E>* a = reinterpret_cast<const vec8<E>*>(wte + (size_t)id * H);
  const vec8<E>* p = reinterpret_cast<const vec8<E>*>(wpe + (size_t)pos * H);
  vec8<E>* o = reinterpret_cast<vec8<E>*>(x + (size_t)t * H);
  const auto put = [&](int32_t v, vec8<E> a8, vec8<E> p8) {
    vec8<E> r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = static_cast<E>(static_cast<float>(a8[e]) + static_cast<float>(p8[e]));
    o[v] = r;
  };
  int32_t v = lane;
  if constexpr (U > 1) {
    for (; v + 64 * (U - 1) < H / 8; v += 64 * U) {
      vec8<E> a8[U], p8[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        a8[u] = a[v + 64 * u];
        p8[u] = p[v + 64 * u];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) put(v + 64 * u, a8[u], p8[u]);
    }
  }
  for (; v < H / 8; v += 64) put(v, a[v], p[v]);
}

__global__ __launch_bounds__(256) void last_rows_kernel(const uint4* __restrict__ x, const int32_t* __restrict__ cu,
                                                        int32_t B, int32_t row_vecs, uint4* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int32_t b = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (b >= B) return;
  const int32_t end = cu[b + 1], len = end - cu[b];
  const uint4* src = x + (size_t)(len > 0 ? end - 1 : 0) * row_vecs;
  for (int32_t v = lane; v < row_vecs; v += 64) out[(size_t)b * row_vecs + v] = len > 0 ? src[v] : make_uint4(0, 0, 0, 0);
}

// K and V thirds of the packed QKV rows of a prefill -> rows 0 .. len-1 of each sequence's cache
// [B, S_cap, A]; one wavefront per packed row, 16-byte vectors.
template <int U>
__global__ __launch_bounds__(256) void cache_fill_kernel(const uint4* __restrict__ qkv, const int32_t* __restrict__ cu,
                                                         int32_t B, int64_t T, int32_t a_vecs, int32_t S_cap,
                                                         uint4* __restrict__ kc, uint4* __restrict__ vc) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  int32_t lo = 0, hi = B;  // invariant: cu[lo] <= t < cu[hi]
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (cu[mid] <= t) lo = mid; else hi = mid;
  }
  const int32_t pos = (int32_t)(t - cu[lo]);
  if (pos >= S_cap) return;   // a sequence longer than the cache: the tail is not stored
  const uint4* src = qkv + (size_t)t * 3 * a_vecs;
  const size_t dst = ((size_t)lo * S_cap + pos) * a_vecs;
  int32_t v = lane;
  if constexpr (U > 1) {
    for (; v + 64 * (U - 1) < a_vecs; v += 64 * U) {
      uint4 k[U], w[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        k[u] = src[a_vecs + v + 64 * u];
        w[u] = src[2 * a_vecs + v + 64 * u];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        kc[dst + v + 64 * u] = k[u];
        vc[dst + v + 64 * u] = w[u];
      }
    }
  }
  for (; v < a_vecs; v += 64) {
    kc[dst + v] = src[a_vecs + v];
    vc[dst + v] = src[2 * a_vecs + v];
  }
}

}  // namespace

hipError_t launch_cache_fill(const void* qkv, const int32_t* cu, int32_t B, int64_t T, int64_t a_bytes, int32_t S_cap,
                             void* kc, void* vc, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  const int u = ends_batch((int32_t)(a_bytes / 16));
  const auto kern = u == 1 ? cache_fill_kernel<1> : u == 4 ? cache_fill_kernel<4> : u == 5 ? cache_fill_kernel<5> : cache_fill_kernel<8>;
  kern<<<dim3((unsigned)((T + 3) / 4)), dim3(256), 0, s>>>((const uint4*)qkv, cu, B, T, (int32_t)(a_bytes / 16), S_cap, (uint4*)kc,
                                                         (uint4*)vc);
  return hipGetLastError();
}

template <typename E>
static hipError_t embed(const int32_t* ids, const int32_t* cu, const int32_t* positions, int32_t B, int64_t T, const void* wte,
                        int32_t V, const void* wpe, int32_t P, int32_t H, void* x, hipStream_t s) {
  const int u = ends_batch(H / 8);
  const auto kern = u == 1 ? embed_packed_kernel<E, 1> : u == 4 ? embed_packed_kernel<E, 4>
                  : u == 5 ? embed_packed_kernel<E, 5> : embed_packed_kernel<E, 8>;
  kern<<<dim3((unsigned)((T + 3) / 4)), dim3(256), 0, s>>>(ids, cu, positions, B, T, (const E*)wte, V, (const E*)wpe, P, H, (E*)x);
  return hipGetLastError();
}

// cu != nullptr: positions from the packed layout; else positions[t] is row t's position
hipError_t launch_embed_packed(const int32_t* ids, const int32_t* cu, const int32_t* positions, int32_t B, int64_t T,
                               const void* wte, int32_t V, const void* wpe, int32_t P, int32_t H, int dtype, void* x,
                               hipStream_t s) {
  if (T <= 0) return hipSuccess;
  return dtype == 1 ? embed<bf16_t>(ids, cu, positions, B, T, wte, V, wpe, P, H, x, s)
                    : embed<f16_t>(ids, cu, positions, B, T, wte, V, wpe, P, H, x, s);
}

hipError_t launch_last_rows(const void* x, const int32_t* cu, int32_t B, int64_t row_bytes, void* out, hipStream_t s) {
  if (B <= 0) return hipSuccess;
  last_rows_kernel<<<dim3((unsigned)((B + 3) / 4)), dim3(256), 0, s>>>((const uint4*)x, cu, B, (int32_t)(row_bytes / 16),
                                                                      (uint4*)out);
  return hipGetLastError();
}

}  // namespace energon
