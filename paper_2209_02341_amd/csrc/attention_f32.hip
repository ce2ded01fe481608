// fp32 storage path of the causal attention over each sequence's real length, on packed rows (the paper,
// Sec. 4.3, keeps attention on the padded layout; here no padding is rebuilt inside a layer), on the
// fp32 matrix instructions.
//
// One workgroup = (sequence, head, 16 queries); its 4 wavefronts (1 where the tiles are few) take the key tiles of 16 in turn, each with
// an online softmax of its own, and merge their four states through LDS at the end.  The path serves short
// sequences of small models, so what bounds it is the chain of dependent loads, not arithmetic: cutting
// the keys over wavefronts shortens the chain and a wavefront requests its next tile before it works on
// this one.  (One wavefront per query on the vector ALU, the former kernel: 8 sequences of up to 128 tokens x
// 16 heads x 64 took 43.9 us.)
//
// Everything is computed transposed, as in the 16-bit kernel, so that a query is a column of every result
// (v_mfma_f32_16x16x4_f32: operands row l % 16, k = l / 16; the lane holds column l % 16, rows 4 (l / 16) + e):
//   S^T[key, query] = K[key, :] . Q[query, :]: k may be walked in any order both operands share, so a lane
//     reads four consecutive elements 16 c + 4 (l / 16) .. + 3 of its key / query row as one vector;
//   O^T[dd, query] += V^T[dd, key] . P^T[key, query]: instruction e takes keys 4 (l / 16) + e, which is where
//     the accumulator of S^T already holds P.  Row r of block j stands for dd = 4 r + j, so a lane's V operands
//     of four blocks are one vector of the key's row, and its results are vectors of the output row.
#include "common.h"

namespace energon {

namespace {

constexpr int kAfQ = 16;

// WK = 4 or 1; ONE: no sequence has more than one tile of keys; WALK: one workgroup takes all blocks of its (sequence, head)
template <int D, int WK, bool ONE, bool WALK>
__global__ __launch_bounds__(WK * 64, 2) void attention_f32_kernel(const float* __restrict__ qkv,
                                                                        float* __restrict__ out,
                                                                        const int32_t* __restrict__ cu, int32_t nh) {
  constexpr int KC = D / 16;   // 16-element chunks of a K / Q row
  constexpr int U = D / 64;    // 64-element parts of a V row: one vector per lane each, four blocks of O^T
  __shared__ float st_m[WK][kAfQ], st_l[WK][kAfQ];
  __shared__ f32x4 st_o[WK][kAfQ][D / 4 + 1];   // rows padded by 16 bytes
  const int32_t b = blockIdx.z, h = blockIdx.y;
  const int32_t c0 = cu[b], len = cu[b + 1] - c0;
  int32_t q0 = ((int32_t)gridDim.x - 1 - (int32_t)blockIdx.x) * kAfQ;   // most keys first
  if (q0 >= len) return;   // the whole workgroup, before any barrier
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, g = lane >> 4;
  const int32_t A = nh * D;
  const size_t ld = (size_t)3 * A;
  const float* base = qkv + (size_t)c0 * ld + (size_t)h * D;   // row 0 of this sequence, Q of this head
  const float scale = rsqrtf((float)D);

  do {
    const int32_t qi = q0 + lr;
    f32x4 q[KC];
    const float* qrow = base + (size_t)min(qi, len - 1) * ld + 4 * g;
#pragma unroll
    for (int c = 0; c < KC; ++c) q[c] = *reinterpret_cast<const f32x4*>(qrow + 16 * c);

    const int32_t n_tiles = ONE ? 1 : q0 / 16 + 1;   // keys 0 .. q0 + 15, the last tile on the diagonal
    f32x4 k4[KC], v4[4][U];
    auto load = [&](int32_t t) {   // keys past the end read the last row: they lie above the diagonal
      const float* kr = base + A + (size_t)min(16 * t + lr, len - 1) * ld + 4 * g;
#pragma unroll
      for (int c = 0; c < KC; ++c) k4[c] = *reinterpret_cast<const f32x4*>(kr + 16 * c);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float* vr = base + 2 * A + (size_t)min(16 * t + 4 * g + e, len - 1) * ld + 4 * lr;
#pragma unroll
        for (int u = 0; u < U; ++u) v4[e][u] = *reinterpret_cast<const f32x4*>(vr + 64 * u);
      }
    };

    // per query (column): running max, this lane's part of the sum.  The max starts at the lowest finite value: where every
    // score so far is -inf (products that overflow), the weights are exp(-inf) = 0 and not exp(-inf + inf) = NaN
    float m_run = kLowest, l_run = 0.f;
    f32x4 o[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) o[u][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (wave < n_tiles) load(wave);
    for (int32_t t = wave; t < n_tiles; t += WK) {
      f32x4 kc[KC], vc[4][U];
#pragma unroll
      for (int c = 0; c < KC; ++c) kc[c] = k4[c];
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int u = 0; u < U; ++u) vc[e][u] = v4[e][u];
      if (t + WK < n_tiles) load(t + WK);
      f32x4 s0 = f32x4{0.f, 0.f, 0.f, 0.f}, s1 = s0;   // two chains
#pragma unroll
      for (int c = 0; c < KC; c += 2)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kc[c][e], q[c][e], s0, 0, 0, 0);
          s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kc[c + 1][e], q[c + 1][e], s1, 0, 0, 0);
        }
      f32x4 s = (s0 + s1) * scale;
      if (t == n_tiles - 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (16 * t + 4 * g + e > qi) s[e] = -INFINITY;
      }
      float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m_run, mx);
      const float corr = expf(m_run - m_new);
      f32x4 p;
#pragma unroll
      for (int e = 0; e < 4; ++e) p[e] = expf(s[e] - m_new);
      l_run = l_run * corr + ((p[0] + p[1]) + (p[2] + p[3]));
      m_run = m_new;
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) o[u][j] *= corr;
      // On the diagonal a masked key's V still meets P = 0 in the product; that is no contribution unless V is
      // infinite or NaN.  Such tiles add their allowed keys one by one, so a bad token reaches later ones only.
      bool finite = true;
      if (t == n_tiles - 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) finite = finite && fabsf(vc[e][u][j]) < INFINITY;
      }
      if (__all(finite)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[u][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vc[e][u][j], p[e], o[u][j], 0, 0, 0);
      } else {
        for (int kk = 0; kk < 16; ++kk) {
          const float pa = __shfl(p[0], 16 * (kk >> 2) + lr, 64), pb = __shfl(p[1], 16 * (kk >> 2) + lr, 64);
          const float pc = __shfl(p[2], 16 * (kk >> 2) + lr, 64), pd = __shfl(p[3], 16 * (kk >> 2) + lr, 64);
          const int32_t key = 16 * t + kk;
          if (key > qi || key >= len) continue;
          const float pk = (kk & 3) == 0 ? pa : (kk & 3) == 1 ? pb : (kk & 3) == 2 ? pc : pd;
          const float* vr = base + 2 * A + (size_t)key * ld + 16 * g;
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const f32x4 vv = *reinterpret_cast<const f32x4*>(vr + 64 * u + 4 * e);
#pragma unroll
              for (int j = 0; j < 4; ++j) o[u][j][e] = fmaf(pk, vv[j], o[u][j][e]);
            }
        }
      }
    }

    // merge the four states: weights exp(m_w - M); a wavefront that saw no key of weight has m = kLowest, l = 0, o = 0
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    if (g == 0) { st_m[wave][lr] = m_run; st_l[wave][lr] = l_run; }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)   // rows 4 g + e of blocks j = dd 64 u + 4 (4 g + e) + j
        st_o[wave][lr][16 * u + 4 * g + e] = f32x4{o[u][0][e], o[u][1][e], o[u][2][e], o[u][3][e]};
    __syncthreads();
    for (int i = tid; i < kAfQ * (D / 4); i += WK * 64) {
      const int r = i / (D / 4), v = i % (D / 4);
      if (q0 + r >= len) break;   // rows ascend with i
      float M = st_m[0][r];
#pragma unroll
      for (int w = 1; w < WK; ++w) M = fmaxf(M, st_m[w][r]);
      float L = 0.f;
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < WK; ++w) {
        const float wgt = expf(st_m[w][r] - M);
        L += st_l[w][r] * wgt;
        acc += st_o[w][r][v] * wgt;
      }
      *reinterpret_cast<f32x4*>(out + (size_t)(c0 + q0 + r) * A + (size_t)h * D + 4 * v) = acc / L;
    }
    if (WALK) {
      __syncthreads();   // the states are read before the next block's are written
      q0 += kAfQ;
    }
  } while (WALK && q0 < len);
}

}  // namespace

hipError_t launch_attention_f32(const float* qkv, float* out, const int32_t* cu, int64_t T, int32_t B, int32_t max_len,
                                int32_t nh, int32_t d, hipStream_t s) {
  if (B <= 0 || max_len <= 0) return hipSuccess;
  const dim3 grid((unsigned)((max_len + kAfQ - 1) / kAfQ), (unsigned)nh, (unsigned)B);
  // Few tiles of keys in many workgroups: three of four wavefronts would mostly take up registers (us, four / one: 5000 x 1
  // token x 4 heads of 64 60 / 23, 1000 x 17 x 12 105 / 64, 64 x 64 x 40 x 128 154 / 121; but 8 of up to 128 tokens x 16 heads
  // 8.0 / 10.9, 4 of up to 32 x 4 3.7 / 4.4, one of 4096 81 / 272).
  const auto launch = [&](auto kernel, int wavefronts, const dim3& grid) {
    kernel<<<grid, dim3((unsigned)wavefronts * 64), 0, s>>>(qkv, out, cu, nh);
    return hipGetLastError();
  };
  if (max_len <= kAfQ)
    return d == 128 ? launch(attention_f32_kernel<128, 1, true, false>, 1, grid) : launch(attention_f32_kernel<64, 1, true, false>, 1, grid);
  const int64_t blocks = (int64_t)grid.x * nh * B;
  if (max_len <= 4 * kAfQ && blocks >= 1024) {
    // most sequences have one block: the others' workgroups would be empty (3001 of 2 and one of 60 x 12 x 128 317 -> 136;
    // but 61 of 1 and one of 17 x 12 x 128 8.0 / 9.0)
    if (T <= (int64_t)kAfQ * B && blocks >= 8192) {
      const dim3 pairs(1, grid.y, grid.z);
      return d == 128 ? launch(attention_f32_kernel<128, 1, false, true>, 1, pairs) : launch(attention_f32_kernel<64, 1, false, true>, 1, pairs);
    }
    return d == 128 ? launch(attention_f32_kernel<128, 1, false, false>, 1, grid) : launch(attention_f32_kernel<64, 1, false, false>, 1, grid);
  }
  return d == 128 ? launch(attention_f32_kernel<128, 4, false, false>, 4, grid) : launch(attention_f32_kernel<64, 4, false, false>, 4, grid);
}

}  // namespace energon
