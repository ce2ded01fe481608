"""16-bit linears too small for whole rounds of the 256x256 kernel, one shape per way they can run: K cut over the
wavefronts of a small tile (three tile sizes), tiles with all of K, K cut over workgroups, the 256x256 kernel in pieces; with and without scratch, ragged rows and columns, all epilogues, the residual also in place (which rules out
overlapping edge tiles).  Against the oracle at the suite's bars; the same bits on a second run over other scratch."""
import numpy as np
import pytest
import torch

from oracle import energon_oracle as orc
from paper_2209_02341_amd import binding as E
from paper_2209_02341_amd import harness as hz
from paper_2209_02341_amd import workloads as wl
from tests.test_gpu_parity import assert_close

pytestmark = pytest.mark.gpu

SHAPES = [
    # M, N, K, dtype, scratch that the plan takes
    (65, 40, 64, wl.BF16, False),          # 32x32, one slab
    (130, 264, 192, wl.BF16, False),       # 32x32, fewer slabs than wavefronts
    (515, 1032, 1024, wl.F16, False),      # 64x64
    (131, 2056, 4096, wl.BF16, False),     # 64x32
    (513, 1032, 2048, wl.BF16, False),     # 64x64
    (1025, 2056, 1024, wl.F16, False),     # 96x96
    (2600, 2056, 192, wl.BF16, False),     # 128x128, with a residual 128x192
    (515, 2056, 4096, wl.BF16, False),     # 64x96
    (900, 5128, 5120, wl.BF16, False),     # 128x192
    (300, 1032, 8192, wl.BF16, True),      # 96x128, K cut seven ways
    (1300, 264, 8192, wl.F16, True),       # 96x128, K cut six ways
    (500, 6584, 7680, wl.BF16, True),      # pieces
]


@pytest.mark.parametrize("M,N,K,dtype,cuts", SHAPES)
@pytest.mark.parametrize("epi", [E.EPI_BIAS, E.EPI_BIAS_GELU, E.EPI_BIAS_RESIDUAL])
def test_linear_plans(M, N, K, dtype, cuts, epi):
    rng = np.random.default_rng(M + N + K + epi)
    x = wl.round_to_dtype(rng.standard_normal((M, K), dtype=np.float32), dtype)
    w = wl.round_to_dtype(rng.standard_normal((N, K), dtype=np.float32) / np.sqrt(K), dtype)
    b = wl.round_to_dtype(rng.standard_normal(N) * 0.5, dtype)
    r = wl.round_to_dtype(rng.standard_normal((M, N), dtype=np.float32), dtype)
    xd, wd, bd, rd = (hz.to_device(a, dtype) for a in (x, w, b, r))
    nbytes = E.energon_linear_scratch_bytes(M, N, K, E.BF16 if dtype == wl.BF16 else E.F16)
    assert (nbytes > 0) == cuts
    ref = orc.linear(x.astype(np.float64), w.astype(np.float64), b.astype(np.float64))
    ref = orc.gelu(ref) if epi == E.EPI_BIAS_GELU else ref + r if epi == E.EPI_BIAS_RESIDUAL else ref
    res = rd if epi == E.EPI_BIAS_RESIDUAL else None
    for scratch_bytes in {0, nbytes}:
        outs = []
        for fill in (0, 255):
            scratch = torch.full((scratch_bytes,), fill, dtype=torch.uint8, device="cuda") if scratch_bytes else None
            yd = torch.full((M + 1, N), 3.0, dtype=xd.dtype, device="cuda")
            E.energon_linear_with_scratch(xd, wd, bd, res, yd, epi, scratch)
            assert torch.all(yd[M] == 3.0), "row past M was written"
            outs.append(yd[:M])
        assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
        assert_close(hz.to_host(outs[0]), ref, dtype, f"linear epi={epi} scratch={scratch_bytes}")
        if res is not None:   # in place
            yd = rd.clone()
            E.energon_linear_with_scratch(xd, wd, bd, yd, yd, epi, scratch)
            assert_close(hz.to_host(yd), ref, dtype, f"linear in place scratch={scratch_bytes}")


def test_scratch_below_the_plans_need_is_not_refused():
    M, N, K = 300, 1032, 8192
    x, w = torch.randn((M, K), device="cuda").bfloat16(), (torch.randn((N, K), device="cuda") * 0.02).bfloat16()
    need = E.energon_linear_scratch_bytes(M, N, K, E.BF16)
    ys = []
    for n in (0, 256, need - 256):
        y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        E.energon_linear_with_scratch(x, w, None, None, y, E.EPI_BIAS, torch.empty(n, dtype=torch.uint8, device="cuda") if n else None)
        ys.append(y)
    ref = x.double() @ w.double().t()
    for y in ys:   # one rounding of the result (2^-9 of it) and of sums of K fp32 products
        assert float((y.double() - ref).abs().max()) <= 2.0 ** -8 * float(ref.abs().max())


# M, N, K, dtype, what runs with bias / bias + GeLU / bias + residual: rows and columns of the tile, last ones ragged
SQUARE, WIDE, SHARED, CUT = (2, 128, 128, 1), (2, 128, 256, 1), (2, 64, 64, 1), (1, 64, 64, 1)
TILES = [
    (650, 5128, 4096, wl.BF16, (SQUARE, SQUARE, SQUARE)),
    (1000, 15368, 192, wl.F16, (SQUARE, SQUARE, SQUARE)),     # three slabs on two buffers
    (2000, 20488, 64, wl.BF16, (SQUARE, SQUARE, SQUARE)),     # one slab
    (515, 12296, 2560, wl.F16, (WIDE, SQUARE, WIDE)),
    (1463, 4920, 1600, wl.BF16, (WIDE, WIDE, WIDE)),
    (650, 1032, 1600, wl.BF16, (SHARED, SHARED, SHARED)),
    (123, 7544, 5696, wl.F16, (CUT, CUT, SHARED)),
    (900, 264, 1600, wl.F16, ((1, 64, 32, 1),) * 3),
]


@pytest.mark.parametrize("M,N,K,dtype,plans", TILES)
@pytest.mark.parametrize("epi", [E.EPI_BIAS, E.EPI_BIAS_GELU, E.EPI_BIAS_RESIDUAL])
def test_linear_tiles(M, N, K, dtype, plans, epi):
    assert E.energon_linear_plan(M, N, K, epi) == plans[epi]
    nbytes = E.energon_linear_scratch_bytes(M, N, K, E.BF16 if dtype == wl.BF16 else E.F16)
    test_linear_plans(M, N, K, dtype, nbytes > 0, epi)
