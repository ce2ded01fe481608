"""fp32 linears on the bf16 matrix instructions (every operand cut into three bf16 numbers), at the edges of their tiles: ragged rows
and columns, a partial last slab, fewer slabs than wavefronts; and what the cut must not change: infinities, NaN, values next
to the largest float, tiny ones.

Bound: any order of summing K products in fp32 is off by at most (K + 2) u sum |x w|, u = 2^-24, and the three products of six that
are left out are below 2^-21 = 8 u of each |x w|.  (Here six roundings per 32 products take the place of 32, so the bound holds
with room.)"""
import numpy as np
import pytest
import torch

from oracle import energon_oracle as orc
from paper_2209_02341_amd import binding as E
from paper_2209_02341_amd import harness as hz
from paper_2209_02341_amd import workloads as wl

pytestmark = pytest.mark.gpu
U = 2.0 ** -24
SHAPES = [
    # M, N, K: the tile that the launch is expected to take (rows x columns, wavefronts along K)
    (650, 1160, 516),                       # 64 x 64, 4
    (867, 164, 96), (871, 164, 68),         # 32 x 32, 4: three slabs on four wavefronts; a last slab of four
    (133, 1072, 160), (129, 1076, 132),     # 32 x 32, 8
    (866, 844, 96), (631, 1176, 68),        # 32 x 48, 4
    (579, 848, 96), (802, 616, 68),         # 48 x 32, 4
    (837, 1188, 96), (855, 1192, 68),       # 32 x 48, 2
    (387, 1036, 2052),                      # an odd number of slabs for some wavefronts, an even one for others
]


def _linear(x, w, b=None, r=None, epi=E.EPI_BIAS):
    yd = torch.full((x.shape[0] + 1, w.shape[0]), 3.0, device="cuda")
    d = lambda a: None if a is None else hz.to_device(a, wl.F32)
    E.energon_linear(d(x), d(w), d(b), d(r), yd, epi)
    out = hz.to_host(yd)
    assert np.all(out[-1] == 3.0), "row past M was written"
    return out[:-1]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("epi", [E.EPI_BIAS, E.EPI_BIAS_GELU, E.EPI_BIAS_RESIDUAL])
def test_split_linear(M, N, K, epi):
    rng = np.random.default_rng(M + N + K + epi)
    x, w = rng.standard_normal((M, K)).astype(np.float32), (rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32)
    b, r = rng.standard_normal(N).astype(np.float32), rng.standard_normal((M, N)).astype(np.float32)
    out = _linear(x, w, b, r if epi == E.EPI_BIAS_RESIDUAL else None, epi)
    x, w, b, r = (a.astype(np.float64) for a in (x, w, b, r))
    ref = orc.linear(x, w, b)
    bound = (K + 10) * U * (np.abs(x) @ np.abs(w).T + np.abs(b))
    if epi == E.EPI_BIAS_GELU:
        bound = 1.13 * bound + 1.3e-7 + 8 * U * np.abs(ref)
        ref = orc.gelu(ref)
    if epi == E.EPI_BIAS_RESIDUAL:
        ref = ref + r
        bound = bound + 8 * U * (np.abs(ref) + np.abs(r))
    assert np.all(np.abs(out - ref) <= bound)


@pytest.mark.parametrize("M,N,K", [(387, 1036, 92), (513, 1028, 260)])
def test_split_keeps_what_fp32_gives_at_the_ends_of_its_range(M, N, K):
    rng = np.random.default_rng(K)
    x, w = rng.standard_normal((M, K)).astype(np.float32), (rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32)
    clean = _linear(x, w)
    big = np.float32(3.4028234e38)
    x[3, 5], x[40, K - 1], x[77, 0] = np.inf, -np.inf, np.nan
    x[100], x[101, 7] = 0.0, big                     # a row of one product with the largest float
    x[100, 9] = big
    x[102] *= np.float32(2.0 ** -90)                 # parts down to 2^-114: still whole
    w[8] = 0.0                                       # inf * 0: NaN
    out = _linear(x, w)
    with np.errstate(all="ignore"):
        ref = x.astype(np.float64) @ w.astype(np.float64).T
        ref32 = ref.astype(np.float32)               # sums beyond the largest float: infinite
    for m in (3, 40, 77):
        assert np.array_equal(np.isnan(out[m]), np.isnan(ref32[m])) and np.array_equal(out[m][np.isinf(ref32[m])], ref32[m][np.isinf(ref32[m])])
    for m in (100, 101):
        assert np.all(np.abs(out[m] - ref[m]) <= (K + 10) * U * (np.abs(x[m]).astype(np.float64) @ np.abs(w).T.astype(np.float64)))
    assert np.all(np.abs(out[102] - ref[102]) <= (K + 10) * U * (np.abs(x[102]).astype(np.float64) @ np.abs(w).T.astype(np.float64)))
    others = [m for m in range(M) if m not in (3, 40, 77, 100, 101, 102)]
    cols = [n for n in range(N) if n != 8]
    assert np.array_equal(out[np.ix_(others, cols)], clean[np.ix_(others, cols)])
