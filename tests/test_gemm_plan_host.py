"""The work decomposition of the persistent contraction kernel, replayed on the host (no GPU): for the
layer shapes of every workload and for a seeded sweep of shapes and workgroup counts, every tile and every
slab of K must be covered exactly once, pieces must be even and contiguous, and the pieces of a cut tile must
sit in the slots the second kernel reads."""
import numpy as np
import pytest

from paper_2209_02341_amd import binding as E
from paper_2209_02341_amd import harness as hz
from paper_2209_02341_amd import workloads as wl


def layer_shapes(w, T):
    H, A, F = w.hidden, w.attn_width, w.ffn
    return [(T, 3 * A, H), (T, H, A), (T, F, H), (T, H, F)]


@pytest.mark.parametrize("name", ["gpt13b_bf16", "gpt175b_tp8_shard_bf16", "heavy_pad_bf16"])
def test_layer_shapes_are_covered_exactly_once(name):
    w = wl.WORKLOADS[name]
    T = int(wl.sample_lengths(w).sum())
    cut = 0
    for M in (T, w.batch * w.max_len):
        for (m, n, k) in layer_shapes(w, M):
            for scratch in (False, True):
                st, pieces = E.energon_linear_plan_selfcheck(m, n, k, 32, scratch)
                assert st == 0, (name, m, n, k, scratch, st)
                assert pieces == 1 or scratch
                cut += pieces > 1
    assert cut > 0, "no shape of this workload is cut any more"


def test_the_planned_cuts_of_the_benchmark_workloads():
    # (shape, pieces per cut tile) as measured and documented: a change of the cost model must be a decision
    for shape, want in (((8428, 20480, 5120), 3), ((8428, 5120, 20480), 3), ((8428, 15360, 5120), 1), ((8428, 5120, 5120), 1),
                        ((3184, 6144, 12288), 4), ((3184, 12288, 6144), 2), ((3184, 4608, 12288), 1)):
        st, pieces = E.energon_linear_plan_selfcheck(*shape, 32, True)
        assert (st, pieces) == (0, want), (shape, st, pieces)


def test_random_shapes_and_workgroup_counts():
    rng = np.random.default_rng(2209)
    checked = cut = 0
    for _ in range(400):
        M = int(rng.integers(256, 40000))
        N = 8 * int(rng.integers(32, 5000))
        K = 128 * int(rng.integers(1, 200))
        wgs = int(rng.choice([1, 3, 7, 16, 30, 32, 38, 64]))
        for scratch in (False, True):
            st, pieces = E.energon_linear_plan_selfcheck(M, N, K, wgs, scratch)
            assert st in (0, -1), (M, N, K, wgs, scratch, st)
            if st == 0:
                checked += 1
                cut += pieces > 1
    assert checked > 300 and cut > 20, (checked, cut)


def test_shapes_the_kernel_does_not_take():
    assert E.energon_linear_plan_selfcheck(577, 1024, 1024)[0] == -1      # too few tiles
    assert E.energon_linear_plan_selfcheck(8428, 5120, 5184)[0] == -1     # odd number of slabs
    assert E.energon_linear_plan_selfcheck(8428, 5120, 5100)[0] == -1


def test_linear_plan_refusals_and_one_shape_per_kernel():
    for args in ((0, 64, 64), (8, 12, 64), (8, 64, 100), (8, 64, 1 << 24)):
        with pytest.raises(E.EnergonError):
            E.energon_linear_plan(*args)
    with pytest.raises(E.EnergonError):
        E.energon_linear_plan(100, 64, 64, E.EPI_BIAS_RESIDUAL, ln_folded=True)   # no such epilogue
    assert [E.energon_linear_plan(*s)[0] for s in ((4, 512, 512), (100, 512, 512), (658, 5120, 5120), (8428, 5120, 5120))] == [0, 1, 2, 3]


def test_tiles_in_pieces_ask_for_their_pieces_room_only():
    for M, N, K in ((928, 5120, 20480), (404, 8192, 7680), (400, 5120, 20480)):
        need = E.energon_linear_scratch_bytes(M, N, K, E.BF16)
        kernel, rows, columns, pieces = E.energon_linear_plan(M, N, K, E.EPI_BIAS, scratch_bytes=need)
        assert (kernel, rows, columns) == (3, 256, 256) and pieces > 1
        tiles = -(-M // rows) * -(-N // columns)
        per_xcd = -(-tiles // 8)
        assert need == 8 * per_xcd * pieces * rows * columns * 4
        assert E.energon_linear_plan_selfcheck(M, N, K)[0] == 0


@pytest.mark.parametrize("M,N", [(317, 10752), (331, 6528), (268, 6528), (288, 6528), (873, 8704), (865, 8320), (557, 11008), (820, 9344),
                                 (928, 5120)])
def test_square_linears_with_a_bias_only_are_not_held_in_pieces(M, N):
    """Measured 1.15 to 1.38 times as long in pieces of the 256x256 tiles (the last one 1.2): 317 x 10752 x 10752 132 us against 96."""
    need = E.energon_linear_scratch_bytes(M, N, N, E.BF16)
    plans = [E.energon_linear_plan(M, N, N, epi, scratch_bytes=need) for epi in (E.EPI_BIAS, E.EPI_BIAS_GELU, E.EPI_BIAS_RESIDUAL)]
    assert [p[0] for p in plans] == [2, 2, 2]
    assert need == max([4 * p[3] * M * N for p in plans if p[3] > 1], default=0) + 255 & ~255


@pytest.mark.parametrize("M,N,K,epi,plan", [
    # measured on the tiles that these shapes were held on and on these (us): 64x64 38.0 / 23.1, 59.2 / 43.5, 25.8 / 17.1,
    # 29.2 / 20.0, 30.0 / 19.7; K over the wavefronts of small tiles 25.4 / 20.1, 36.5 / 23.5, 55.1 / 27.8; 128x256 in parts 38.6 / 33.6
    (692, 30536, 192, E.EPI_BIAS, (2, 128, 128, 1)), (1033, 30536, 192, E.EPI_BIAS_GELU, (2, 96, 96, 1)),
    (251, 50256, 256, E.EPI_BIAS, (2, 128, 128, 1)), (944, 18016, 192, E.EPI_BIAS, (2, 96, 96, 1)),
    (5239, 2840, 192, E.EPI_BIAS_GELU, (2, 128, 128, 1)),
    (369, 1096, 11456, E.EPI_BIAS_GELU, (2, 96, 128, 7)), (1186, 128, 25024, E.EPI_BIAS_GELU, (2, 96, 128, 8)),
    (720, 72, 40576, E.EPI_BIAS_GELU, (2, 96, 128, 8)), (300, 2048, 16384, E.EPI_BIAS_RESIDUAL, (2, 96, 128, 4)),
])
def test_ragged_widths_and_long_k_run_on_the_tiles_that_every_shape_has(M, N, K, epi, plan):
    assert E.energon_linear_plan(M, N, K, epi, scratch_bytes=E.energon_linear_scratch_bytes(M, N, K, E.BF16)) == plan


@pytest.mark.parametrize("M,N,K,epi,rows", [
    # us on the tiles that W alone chose, in pieces or parts of tall ones before the ring kernel, and on these now
    (3250, 1344, 24832, E.EPI_BIAS_RESIDUAL, 160),   # 257 / 213
    (3054, 1216, 24448, E.EPI_BIAS_RESIDUAL, 256),   # 217 / 174 / 175
    (1659, 2304, 16128, E.EPI_BIAS_GELU, 256),       # 146 / 125 / 128
    (4071, 1216, 16128, E.EPI_BIAS, 256),            # 180 / 156 / 158
    (2857, 1024, 16896, E.EPI_BIAS_RESIDUAL, 160),   # 138 / 108 / 105
    (3736, 768, 24832, E.EPI_BIAS, 160),             # 194 / 142 / 131
    (5536, 512, 18048, E.EPI_BIAS_RESIDUAL, 160),    # 153 / 118 / 111
    (6567, 1792, 19584, E.EPI_BIAS, 256),            # 557 / 450 / 453
    (5462, 512, 22272, E.EPI_BIAS_GELU, 160),        # 179 / 133
    (918, 4864, 8448, E.EPI_BIAS, 160),              # 109 / 95
])
def test_a_tall_x_from_memory_counts_as_a_wide_w_does(M, N, K, epi, rows):
    assert E.energon_linear_plan(M, N, K, epi, scratch_bytes=E.energon_linear_scratch_bytes(M, N, K, E.BF16))[1] == rows


@pytest.mark.parametrize("M,N,K,epi", [
    # us in parts of 128x256 before the ring kernel, on 64x96 tiles, on these now
    (123, 17216, 3456, E.EPI_BIAS_RESIDUAL),   # 35.7 / 45.9 / 37.3
    (119, 17920, 4032, E.EPI_BIAS),            # 38.4 / 51.8 / 40.5
    (124, 18560, 4416, E.EPI_BIAS_RESIDUAL),   # 43.3 / 58.0 / 45.4
    (125, 17088, 3264, E.EPI_BIAS_GELU),       # 33.1 / 43.6 / 35.4
    (107, 16704, 3264, E.EPI_BIAS_GELU),       # 31.7 / 40.9 / 33.3
])
def test_a_wide_w_from_memory_is_read_once_for_few_rows(M, N, K, epi):
    _, rows, _, parts = E.energon_linear_plan(M, N, K, epi, scratch_bytes=E.energon_linear_scratch_bytes(M, N, K, E.BF16))
    assert rows >= M and parts > 1


@pytest.mark.parametrize("M,N,K,epi", [(1350, 768, 256, E.EPI_BIAS), (147, 7168, 64, E.EPI_BIAS_GELU), (353, 2816, 256, E.EPI_BIAS),
                                       (2571, 440, 64, E.EPI_BIAS_GELU), (159, 6560, 192, E.EPI_BIAS)])
def test_short_k_stays_off_the_smallest_tiles_where_they_make_many_rounds(M, N, K, epi):
    """Replayed from a graph 5.3 to 5.8 us with 64x64 tiles before the ring kernel, 6.4 to 6.9 with 32x32."""
    assert E.energon_linear_plan(M, N, K, epi)[0] == 2


@pytest.mark.parametrize("M", [2 ** 31 - 1, 2 ** 31, 2 ** 32 - 100, 2 ** 32, 2 ** 32 + 5, 2 ** 40])
def test_sizes_may_be_asked_for_any_number_of_rows(M):
    """No such call could run, but the sizes are host arithmetic: no plan cuts K for so many rows, so no room for sums."""
    for N, K in ((128, 192), (128, 4096), (4096, 192), (64, 16384), (1032, 4096)):
        assert E.energon_linear_scratch_bytes(M, N, K, E.BF16) == 0
        st, pieces = E.energon_linear_plan_selfcheck(M, N, K)
        assert (st, pieces) in ((-1, 0), (0, 1))
    H, A, F = 256, 256, 1024
    cfg = hz.layer_config(H, 4, 64, F, wl.BF16, 1e-5)
    r256 = lambda n: -(-n // 256) * 256
    assert E.energon_workspace_bytes(cfg, M) == sum(r256(2 * M * n) for n in (H, 3 * A, A, H, H, F))
