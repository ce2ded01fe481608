"""fp32 storage: the linear kernel on the fp32 matrix instructions, at the edges of its tiles
and of the dispatch between tile sizes, against the oracle.

Bound of the linear: any order of summing K products in fp32 is off by at most (K + 2) u sum |x w| with
u = 2^-24 (K - 1 additions, a rounding per product, the bias); the epilogue's few roundings are relative to
the result and its terms (8 u covers them) and GeLU (slope <= 1.13) adds its fit, 1.3e-7 absolute.
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
          (1403, 1412, 68)]


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
