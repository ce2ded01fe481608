"""fp32 linears of ordinary sizes, on every tile that they run on, at the edges of the tiles: ragged rows and columns, a partial last
slab, fewer slabs than wavefronts.  What fp32 arithmetic promises for every input: each product whole, down to the smallest
subnormal operand and up to the largest float; infinities and NaN where they belong and nowhere else, at no one's cost.

Bound of the sums: any order of summing K products in fp32 is off by at most (K + 2) u sum |x w|, u = 2^-24; on random operands
the roundings mostly cancel, sqrt(K) of them instead of K."""
import numpy as np
import pytest
import torch

from oracle import energon_oracle as orc
from paper_2209_02341_amd import binding as E
from paper_2209_02341_amd import harness as hz
from paper_2209_02341_amd import workloads as wl

pytestmark = pytest.mark.gpu
U = 2.0 ** -24
SHAPES = [   # M, N, K
    (650, 1160, 516), (867, 164, 96), (871, 164, 68), (133, 1072, 160), (129, 1076, 132), (866, 844, 96), (631, 1176, 68),
    (579, 848, 96), (802, 616, 68), (837, 1188, 96), (855, 1192, 68),
    (387, 1036, 2052),                      # an odd number of slabs for some wavefronts, an even one for others
    (1030, 2052, 516), (77, 260, 100), (17, 132, 2116),   # the largest and the smallest tiles
]


def _whole(rng, shape, lo, hi):
    """Random floats of all 24 bits, exponents lo .. hi - 1."""
    return ((rng.integers(1 << 23, 1 << 24, shape) | 1) * np.exp2(rng.integers(lo, hi, shape) - 23.0) * rng.choice([-1.0, 1.0], shape)).astype(np.float32)


def _linear(x, w, b=None, r=None, epi=E.EPI_BIAS):
    yd = torch.full((x.shape[0] + 1, w.shape[0]), 3.0, device="cuda")
    d = lambda a: None if a is None else hz.to_device(a, wl.F32)
    E.energon_linear(d(x), d(w), d(b), d(r), yd, epi)
    out = hz.to_host(yd)
    assert np.all(out[-1] == 3.0), "row past M was written"
    return out[:-1]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("epi", [E.EPI_BIAS, E.EPI_BIAS_GELU, E.EPI_BIAS_RESIDUAL])
def test_linear(M, N, K, epi):
    rng = np.random.default_rng(M + N + K + epi)
    x, w = rng.standard_normal((M, K)).astype(np.float32), (rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32)
    b, r = rng.standard_normal(N).astype(np.float32), rng.standard_normal((M, N)).astype(np.float32)
    out = _linear(x, w, b, r if epi == E.EPI_BIAS_RESIDUAL else None, epi)
    x, w, b, r = (a.astype(np.float64) for a in (x, w, b, r))
    ref = orc.linear(x, w, b)
    bound = (K + 10) * U * (np.abs(x) @ np.abs(w).T + np.abs(b))
    if epi == E.EPI_BIAS:   # random roundings, sqrt(K) / 4 u of them at most (K over four wavefronts or more, four products at a time): twice that
        assert np.linalg.norm(out - ref) <= (2.0 + 0.5 * np.sqrt(K)) * U * np.linalg.norm(ref)
    if epi == E.EPI_BIAS_GELU:
        bound = 1.13 * bound + 1.3e-7 + 8 * U * np.abs(ref)
        ref = orc.gelu(ref)
    if epi == E.EPI_BIAS_RESIDUAL:
        ref = ref + r
        bound = bound + 8 * U * (np.abs(ref) + np.abs(r))
    assert np.all(np.abs(out - ref) <= bound)


@pytest.mark.parametrize("M,N,K", [(387, 1036, 92), (513, 1028, 260)])
def test_what_fp32_gives_at_the_ends_of_its_range(M, N, K):
    rng = np.random.default_rng(K)
    x, w = rng.standard_normal((M, K)).astype(np.float32), (rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32)
    clean = _linear(x, w)
    big = np.float32(3.4028234e38)
    x[3, 5], x[40, K - 1], x[77, 0] = np.inf, -np.inf, np.nan
    x[100], x[101, 7] = 0.0, big                     # a row of one product with the largest float
    x[100, 9] = big
    x[102] *= np.float32(2.0 ** -90)
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


def _one_product_rows(M, N, K, lo, hi, w_lo, w_hi, seed):
    """x with one nonzero per row, at changing k: every output is one product, so nothing else can hide what is missing of it."""
    rng = np.random.default_rng(seed)
    x, w = np.zeros((M, K), np.float32), _whole(rng, (N, K), w_lo, w_hi)
    k = (np.arange(M) * 37 + rng.integers(0, K)) % K
    x[np.arange(M), k] = _whole(rng, M, lo, hi)
    return x, w, k


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_every_product_is_whole(M, N, K):
    """One rounding, to the result: u |x w| (and a sixteenth)."""
    x, w, k = _one_product_rows(M, N, K, -3, 4, -3, 4, M + K)
    x[np.arange(M), k] = np.where(np.arange(M) % 3 == 0, np.float32(1 + 2.0 ** -7 - 2.0 ** -23), x[np.arange(M), k])   # all bits but one set
    w[::5] = np.float32(1 + 2.0 ** -7 - 2.0 ** -23)
    ref = x[np.arange(M), k].astype(np.float64)[:, None] * w.astype(np.float64)[:, k].T
    assert np.max(np.abs(_linear(x, w) - ref) / np.abs(ref)) <= U * (1 + 2.0 ** -4)


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("small", ["x", "w"])
def test_small_operands_are_whole(M, N, K, small):
    """Operands down to the smallest subnormal times large ones: as exact as any other product."""
    tiny, large = (-149, -104), (64, 100)
    x, w, k = _one_product_rows(M, N, K, *(tiny + large if small == "x" else large + tiny), M + K)
    ref = x[np.arange(M), k].astype(np.float64)[:, None] * w.astype(np.float64)[:, k].T
    out = _linear(x, w)
    assert np.all(out[ref == 0.0] == 0.0)
    assert np.max(np.abs(out - ref)[ref != 0.0] / np.abs(ref)[ref != 0.0]) <= U * (1 + 2.0 ** -4)


@pytest.mark.parametrize("scale", [-100, -112, -120, -126, -135])
def test_sums_of_small_operands(scale):
    rng = np.random.default_rng(-scale)
    M, N, K = 387, 1036, 516
    x = np.ldexp(rng.standard_normal((M, K)), scale).astype(np.float32)
    w = np.ldexp(rng.standard_normal((N, K)), 60).astype(np.float32)
    bound = (K + 10) * U * (np.abs(x).astype(np.float64) @ np.abs(w).T.astype(np.float64))
    assert np.all(np.abs(_linear(x, w) - x.astype(np.float64) @ w.astype(np.float64).T) <= bound)


@pytest.mark.parametrize("value", [np.nan, np.inf, 2.0 ** -120])
def test_no_value_costs_more(value):
    """A NaN, an infinity or a tiny number in every row: not another kind of walk over K (twice the time leaves room for the clocks)."""
    M, N, K = 1000, 1600, 1600
    x, w = torch.randn((M, K), device="cuda"), torch.randn((N, K), device="cuda") * 0.02
    y = torch.empty((M, N), device="cuda")

    def us(x):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        times = []
        for _ in range(9):
            a.record()
            for _ in range(4):
                E.energon_linear(x, w, None, None, y, E.EPI_BIAS)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 250.0)
        return sorted(times)[4]

    clean = us(x)
    odd = x.clone()
    odd[:, 7] = value * (1.0 + 2.0 ** -23)
    assert us(odd) <= 2.0 * clean
