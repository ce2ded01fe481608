"""fp32 storage: the linear and the attention kernels on the fp32 matrix instructions, at the edges of their
tiles and of the dispatch between tile sizes, against the oracle.

Bound of the linear: any order of summing K products in fp32 is off by at most (K + 2) u sum |x w| with
u = 2^-24 (K - 1 additions, a rounding per product, the bias); the epilogue's few roundings are relative to
the result and its terms (8 u covers them) and GeLU (slope <= 1.13) adds its fit, 1.3e-7 absolute.
Bound of the attention: the logits are off by d u sum |q k| <= eps, which moves every softmax weight by a
factor within exp(+-2 eps) of itself, and the weighted sum of len values adds (len + 8) u of its terms.
"""
import numpy as np
import pytest
import torch

from oracle import energon_oracle as orc
from paper_2209_02341_amd import binding as E
from paper_2209_02341_amd import harness as hz
from paper_2209_02341_amd import workloads as wl

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


# 16 x 16 tiles with four and with eight wavefronts, 32 x 32, 32 x 64, 64 x 64; K with fewer slabs than wavefronts,
# a partial last slab, ragged rows and columns
LINEAR = [(17, 20, 4), (16, 16, 100), (33, 68, 132), (5, 260, 2052), (250, 644, 36), (257, 1028, 64), (387, 1036, 92),
          (1403, 1412, 68),
          # narrow sides take 16 x 16 however long the other is, the next wider 32 x 32, each with one wavefront up to K = 64
          # and with four beyond; 64 x 64 from a longer K on
          (5409, 16, 36), (9, 5412, 64), (5409, 20, 36), (5409, 16, 68), (9, 5412, 100), (5409, 20, 68), (1021, 1020, 1092)]


@pytest.mark.parametrize("M,N,K", LINEAR)
@pytest.mark.parametrize("epi", [E.EPI_BIAS, E.EPI_BIAS_GELU, E.EPI_BIAS_RESIDUAL])
def test_linear_f32(M, N, K, epi):
    rng = np.random.default_rng(M + N + K + epi)
    x, w = rng.standard_normal((M, K)).astype(np.float32), (rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32)
    b, r = rng.standard_normal(N).astype(np.float32), rng.standard_normal((M, N)).astype(np.float32)
    xd, wd, bd, rd = (hz.to_device(a, wl.F32) for a in (x, w, b, r))
    yd = torch.full((M + 1, N), 3.0, device="cuda")
    E.energon_linear(xd, wd, bd, rd if epi == E.EPI_BIAS_RESIDUAL else None, yd, epi)
    x, w, b, r = (a.astype(np.float64) for a in (x, w, b, r))
    ref = orc.linear(x, w, b)
    bound = (K + 2) * U * (np.abs(x) @ np.abs(w).T + np.abs(b))
    if epi == E.EPI_BIAS_GELU:
        bound = 1.13 * bound + 1.3e-7 + 8 * U * np.abs(ref)
        ref = orc.gelu(ref)
    if epi == E.EPI_BIAS_RESIDUAL:
        ref = ref + r
        bound = bound + 8 * U * (np.abs(ref) + np.abs(r))
    out = hz.to_host(yd)
    assert np.all(np.abs(out[:M] - ref) <= bound)
    assert np.all(out[M] == 3.0), "row past M was written"


def _attention(qkv, lens, nh, d):
    lens = np.asarray(lens, np.int32)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    od = torch.full((T + 1, nh * d), 3.0, device="cuda")
    E.energon_attention(hz.to_device(qkv, wl.F32), od[:T], torch.from_numpy(cu).cuda(), len(lens), int(lens.max()), nh, d)
    out = hz.to_host(od)
    assert np.all(out[T] == 3.0), "row past T was written"
    return out[:T], cu


# from the third on one wavefront: one tile of keys at most, up to four of them in many workgroups, the last
# two with a workgroup for all blocks of a (sequence, head)
@pytest.mark.parametrize("lens,nh,d", [([1, 15, 16, 17, 0, 64, 65], 3, 64), ([129, 2, 80], 2, 128), ([1, 15, 0, 16, 3], 3, 64),
                                       ([2] * 70 + [16, 1], 2, 128), ([64, 0, 17, 33, 1] * 60, 1, 64), ([50, 1, 64] * 50, 2, 128),
                                       ([1, 2, 0, 33, 1, 1] * 230, 2, 64), ([1] * 600 + [64, 17], 4, 128)])
def test_attention_f32(lens, nh, d):
    A = nh * d
    qkv = np.random.default_rng(d).standard_normal((sum(lens), 3 * A)).astype(np.float32)
    out, cu = _attention(qkv, lens, nh, d)
    for b, n in enumerate(lens):
        if n == 0:
            continue
        blk = qkv[cu[b]:cu[b + 1]].astype(np.float64)
        ref = orc.masked_causal_attention(blk[:, :A], blk[:, A:2 * A], blk[:, 2 * A:], n, nh, d)
        qa, ka = (np.abs(blk[:, j * A:(j + 1) * A]).reshape(n, nh, d) for j in (0, 1))
        eps = (d + 4) * U * np.einsum("ihc,jhc->hij", qa, ka).max() / np.sqrt(d)
        bound = (2 * eps + (n + 16) * U) * np.abs(blk[:, 2 * A:]).max(axis=0)
        assert np.all(np.abs(out[cu[b]:cu[b + 1]] - ref) <= bound)


@pytest.mark.parametrize("n,bad", [(40, 37), (14, 9)])
def test_attention_f32_bad_token_reaches_later_tokens_only(n, bad):
    nh, d = 2, 64
    A = nh * d
    qkv = np.random.default_rng(0).standard_normal((n, 3 * A)).astype(np.float32)
    clean, _ = _attention(qkv, [n], nh, d)
    qkv[bad, 2 * A:] = np.inf
    out, _ = _attention(qkv, [n], nh, d)
    assert np.allclose(out[:bad], clean[:bad], rtol=0, atol=1e-6)   # same weights, another order of the sums
    assert not np.isfinite(out[bad:]).any()


# scores of -inf (finite q and k whose products overflow) have weight 0 wherever they lie: a whole first tile of one of
# the four wavefronts that share the keys, several, the first keys of all, single ones
@pytest.mark.parametrize("hidden_keys", [range(16, 32), range(16, 64), [*range(16), *range(40, 48)], [0, 17, 33, 63, 64]])
@pytest.mark.parametrize("d", [64, 128])
def test_attention_f32_scores_of_minus_infinity(hidden_keys, d):
    n, nh = 90, 2
    A = nh * d
    qkv = np.random.default_rng(d).standard_normal((n, 3 * A)).astype(np.float32)
    qkv[:, :A] = 1e20
    qkv[:, A:2 * A] *= 1e-22                       # scores of the other keys: around 0
    qkv[list(hidden_keys), A:2 * A] = -1e20
    out, _ = _attention(qkv, [n], nh, d)
    blk = qkv.astype(np.float64)
    ref = orc.masked_causal_attention(blk[:, :A], blk[:, A:2 * A], blk[:, 2 * A:], n, nh, d)
    seen = np.array([any(j not in hidden_keys for j in range(i + 1)) for i in range(n)])
    eps = (d + 4) * U * 1e20 * d * np.abs(np.delete(blk[:, A:2 * A], list(hidden_keys), 0)).max() / np.sqrt(d)
    bound = (2 * eps + (n + 16) * U) * np.abs(blk[:, 2 * A:]).max(axis=0)
    assert np.all(np.abs(out - ref)[seen] <= bound)
