"""16-bit linears on the tiles of the ring kernel: every tile size, with ragged last rows and columns, fewer slabs of K than
the ring holds and more, K cut over workgroups into parts of unequal length; the plain epilogues (the residual also in
place) and the LayerNorm-folded ones.  Against the oracle at the suite's bars; the same bits on a second run over other
scratch.  The plan names the tile but not which of two kernels runs 128 x 128: up to 256 tiles, one per CU, it is the one with
five slabs in the ring, beyond that and up to 512 the one with two, of which two share a CU."""
import numpy as np
import pytest
import torch

from oracle import energon_oracle as orc
from paper_2209_02341_amd import binding as E
from paper_2209_02341_amd import harness as hz
from paper_2209_02341_amd import workloads as wl
from tests import test_gpu_ln_fold as folded
from tests.test_gpu_parity import assert_close

pytestmark = pytest.mark.gpu

BIAS, GELU, RESIDUAL = E.EPI_BIAS, E.EPI_BIAS_GELU, E.EPI_BIAS_RESIDUAL
SHAPES = [
    # M, N, K, dtype, epilogue, rows and columns of the tile, parts of K
    (129, 3456, 320, wl.BF16, RESIDUAL, (64, 64, 1)),      # as many slabs as the ring holds
    (197, 2816, 64, wl.F16, RESIDUAL, (64, 64, 1)),        # one slab
    (262, 3392, 320, wl.F16, BIAS, (64, 96, 1)),
    (577, 3520, 64, wl.BF16, BIAS, (64, 96, 1)),
    (513, 3712, 320, wl.BF16, BIAS, (96, 96, 1)),
    (513, 3712, 64, wl.F16, GELU, (96, 96, 1)),
    (833, 3520, 320, wl.F16, BIAS, (96, 128, 1)),
    (161, 2752, 4096, wl.BF16, RESIDUAL, (96, 128, 5)),    # 64 slabs in five parts
    (1154, 2624, 320, wl.BF16, RESIDUAL, (128, 128, 1)),
    (780, 5696, 64, wl.BF16, BIAS, (128, 128, 1)),         # 315 tiles
    (97, 10688, 4096, wl.F16, GELU, (128, 128, 3)),
    (1753, 2432, 384, wl.BF16, RESIDUAL, (96, 192, 1)),
    (70, 11584, 4096, wl.F16, BIAS, (96, 192, 4)),
    (1351, 3328, 320, wl.F16, RESIDUAL, (128, 192, 1)),
    (195, 10880, 4096, wl.BF16, GELU, (128, 192, 2)),
    (774, 9472, 320, wl.BF16, RESIDUAL, (160, 192, 1)),
    (780, 9536, 64, wl.F16, BIAS, (160, 192, 1)),
    (1958, 3776, 576, wl.F16, RESIDUAL, (128, 256, 1)),
    (645, 10944, 320, wl.BF16, BIAS, (160, 256, 1)),
    (264, 12480, 4096, wl.F16, GELU, (160, 256, 2)),
    # the ring filled more than twice, an odd number of slabs, widths that are no multiple of any tile's
    (68, 5776, 704, wl.BF16, RESIDUAL, (64, 64, 1)),
    (66, 9800, 576, wl.F16, BIAS, (64, 96, 1)),
    (133, 10912, 448, wl.BF16, BIAS, (96, 96, 1)),
    (197, 9768, 704, wl.F16, BIAS, (96, 128, 1)),
    (195, 12584, 704, wl.BF16, BIAS, (128, 128, 1)),
    (329, 12432, 320, wl.F16, BIAS, (128, 128, 1)),        # 294 tiles
    (789, 4624, 576, wl.BF16, RESIDUAL, (96, 192, 1)),
    (336, 12408, 576, wl.F16, RESIDUAL, (128, 192, 1)),
    (1422, 4408, 448, wl.BF16, RESIDUAL, (160, 192, 1)),
    (1458, 5048, 576, wl.F16, RESIDUAL, (128, 256, 1)),
    (516, 13208, 448, wl.BF16, BIAS, (160, 256, 1)),
    (129, 7016, 6080, wl.F16, BIAS, (160, 192, 6)),        # 95 slabs in six parts
    (1601, 760, 18496, wl.BF16, RESIDUAL, (160, 256, 7)),  # a tall x from memory, 289 slabs in seven parts
    (3001, 248, 14400, wl.F16, GELU, (128, 256, 8)),       # 225 slabs in eight parts
]


@pytest.mark.parametrize("M,N,K,dtype,epi,tile", SHAPES)
def test_ring_tiles(M, N, K, dtype, epi, tile):
    code = E.BF16 if dtype == wl.BF16 else E.F16
    nbytes = E.energon_linear_scratch_bytes(M, N, K, code)
    assert E.energon_linear_plan(M, N, K, epi, scratch_bytes=nbytes) == (2,) + tile
    rng = np.random.default_rng(M + N + K + epi)
    x = wl.round_to_dtype(rng.standard_normal((M, K), dtype=np.float32), dtype)
    w = wl.round_to_dtype(rng.standard_normal((N, K), dtype=np.float32) / np.sqrt(K), dtype)
    b = wl.round_to_dtype(rng.standard_normal(N) * 0.5, dtype)
    r = wl.round_to_dtype(rng.standard_normal((M, N), dtype=np.float32), dtype)
    xd, wd, bd, rd = (hz.to_device(a, dtype) for a in (x, w, b, r))
    ref = orc.linear(x.astype(np.float64), w.astype(np.float64), b.astype(np.float64))
    ref = orc.gelu(ref) if epi == GELU else ref + r if epi == RESIDUAL else ref
    outs = []
    for fill in (0, 255):
        scratch = torch.full((nbytes,), fill, dtype=torch.uint8, device="cuda") if nbytes else None
        yd = torch.full((M + 1, N), 3.0, dtype=xd.dtype, device="cuda")
        E.energon_linear_with_scratch(xd, wd, bd, rd if epi == RESIDUAL else None, yd, epi, scratch)
        assert torch.all(yd[M] == 3.0), "row past M was written"
        outs.append(yd[:M])
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
    assert_close(hz.to_host(outs[0]), ref, dtype, f"ring tile {tile} epi={epi}")
    if epi == RESIDUAL:
        yd = rd.clone()
        E.energon_linear_with_scratch(xd, wd, bd, yd, yd, epi, scratch)
        assert torch.equal(yd.view(torch.int16), outs[0].view(torch.int16))


FOLDED = [(1127, 4160, 64, wl.BF16, True, (128, 128, 1)), (2289, 1024, 128, wl.F16, False, (64, 96, 1)),
          (323, 5504, 192, wl.BF16, False, (96, 96, 1)), (1751, 5248, 64, wl.F16, False, (160, 256, 1)),
          (834, 3520, 448, wl.BF16, True, (96, 128, 1)), (2225, 2240, 1024, wl.F16, False, (128, 192, 1)),
          (102, 480, 704, wl.F16, False, (64, 64, 1)), (67, 8336, 576, wl.BF16, False, (64, 96, 1)),
          (1558, 2440, 2112, wl.BF16, False, (96, 192, 1)), (769, 9504, 448, wl.F16, False, (160, 192, 1)),
          (329, 12432, 320, wl.BF16, False, (128, 128, 1)), (769, 11056, 448, wl.F16, False, (160, 256, 1))]


@pytest.mark.parametrize("M,N,K,dtype,gelu,tile", FOLDED)
def test_ring_tiles_ln_folded(M, N, K, dtype, gelu, tile):
    assert E.energon_linear_plan(M, N, K, GELU if gelu else BIAS, ln_folded=True) == (2,) + tile
    folded.test_linear_ln_folded_matches_layernorm_then_linear(M, N, K, dtype, gelu)


# shapes of 192 and more tiles of 256 x 256 that the ring kernel is expected to finish well before the persistent one
@pytest.mark.parametrize("M,N,K,dtype,epi,tile", [(260, 24832, 256, wl.BF16, BIAS, (96, 96, 1)),
                                                     (303, 24576, 1024, wl.F16, BIAS, (160, 192, 1))])
def test_ring_tiles_instead_of_the_persistent_kernel(M, N, K, dtype, epi, tile):
    assert E.energon_linear_plan(M, N, K, epi, ln_folded=True)[0] == 3   # folded linears stay there
    test_ring_tiles(M, N, K, dtype, epi, tile)
