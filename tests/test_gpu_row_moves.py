"""Kernels that only move rows, bit for bit: each way its launch can choose, at the edges of the rules."""
import numpy as np
import pytest
import torch

from oracle import energon_oracle as orc
from paper_2209_02341_amd import binding as E
from paper_2209_02341_amd import harness as hz
from paper_2209_02341_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.contiguous().view(torch.int16).cpu().numpy()


# one row per wavefront (rows of 8 KB, or few of them) and two (narrower rows, more than 4096), odd counts, empty sequences,
# lengths in the argument block and in memory
@pytest.mark.parametrize("B,S,H", [(40, 150, 8), (900, 20, 24), (30, 290, 4088), (30, 290, 4096), (7, 13, 40)])
def test_pack_rows(B, S, H):
    rng = np.random.default_rng(B + H)
    lens = rng.integers(0, S + 1, size=B).astype(np.int32)
    lens[B // 2: B // 2 + 2] = 0
    lens[-1] = S - (int(lens[:-1].sum()) + S + 1) % 2          # an odd number of rows
    T = int(lens.sum())
    x = torch.randint(-2 ** 15, 2 ** 15, (B, S, H), dtype=torch.int16, device="cuda").view(torch.bfloat16)
    xp = torch.zeros((T + 1, H), dtype=torch.bfloat16, device="cuda")
    cu, idx = torch.empty(B + 1, dtype=torch.int32, device="cuda"), torch.empty(T, dtype=torch.int32, device="cuda")
    assert E.energon_pack(x, lens, xp[:T], cu, idx) == T
    cu_ref, idx_ref = orc.pack_indices(lens, S)
    assert np.array_equal(cu.cpu().numpy(), cu_ref) and np.array_equal(idx.cpu().numpy(), idx_ref)
    want = x.view(torch.int16).view(B * S, H)[torch.from_numpy(np.asarray(idx_ref, np.int64)).cuda()]
    assert torch.equal(xp[:T].view(torch.int16), want)
    assert not xp[T].view(torch.int16).any(), "row past T was written"


def test_pack_of_more_than_2_to_26_rows():
    """A row per wavefront would be more threads than one launch may have."""
    S, H = 2 ** 25 + 4, 8
    lens = np.asarray([S, S - 3], np.int32)
    T = int(lens.sum())
    x = torch.randint(-2 ** 15, 2 ** 15, (2, S, H), dtype=torch.int16, device="cuda").view(torch.bfloat16)
    xp = torch.empty((T, H), dtype=torch.bfloat16, device="cuda")
    cu, idx = torch.empty(3, dtype=torch.int32, device="cuda"), torch.empty(T, dtype=torch.int32, device="cuda")
    assert E.energon_pack(x, lens, xp, cu, idx) == T
    assert cu.tolist() == [0, S, T]
    assert torch.equal(idx, torch.arange(T, dtype=torch.int32, device="cuda"))
    assert torch.equal(xp.view(torch.int16), x.view(torch.int16).view(2 * S, H)[:T])


# sequences of few positions: heads' positions per wavefront, or (fewer than 4 positions at width 128, 8 at 64, many
# workgroups) heads behind one another; launches of few workgroups with fewer vectors per lane
@pytest.mark.parametrize("B,S,nh,d", [(700, 1, 5, 128), (1100, 3, 7, 128), (700, 4, 5, 128), (2100, 1, 1, 64), (900, 7, 3, 64),
                                      (900, 8, 3, 64), (3, 3, 5, 128), (2, 7, 9, 64), (1, 70, 3, 64), (2, 33, 3, 128),
                                      (90, 65, 5, 64), (90, 33, 5, 128)])
def test_rebuild_of_short_sequences(B, S, nh, d):
    rng = np.random.default_rng(B + S)
    lens = rng.integers(0, S + 1, size=B).astype(np.int32)
    lens[0], lens[-1] = S, S
    T, A = int(lens.sum()), nh * d
    qkv = wl.round_to_dtype(rng.standard_normal((T, 3 * A)), wl.BF16)
    cu_ref, _ = orc.pack_indices(lens, S)
    pads = [torch.full((B + 1, nh, S, d), 9.0, dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    E.energon_rebuild_qkv(hz.to_device(qkv, wl.BF16), torch.from_numpy(cu_ref).cuda(), B, S, nh, d, *(p[:B] for p in pads))
    for got, want in zip(pads, orc.rebuild_qkv_heads(qkv, lens, S, nh, d)):
        assert np.array_equal(_bits(got[:B]), _bits(torch.from_numpy(want.astype(np.float32)).to(torch.bfloat16)))
        assert torch.all(got[B] == 9.0), "past the last sequence was written"


# rows of one step of the lanes, of batches of 4, 5 and 8 vectors with and without single steps behind them, ragged ends
WIDTHS = [2040, 2048, 2056, 2560, 3080, 4096, 4104, 5120, 5128, 12288]


@pytest.mark.parametrize("H", WIDTHS)
@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
def test_embedding_of_wide_rows(H, dtype):
    rng = np.random.default_rng(H)
    V, P, lens = 50, 40, [5, 0, 9]
    T = sum(lens)
    wte, wpe = (wl.round_to_dtype(rng.standard_normal((n, H)), dtype) for n in (V, P))
    ids = rng.integers(0, V, size=T).astype(np.int32)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device="cuda")
    wted, wped = hz.to_device(wte, dtype), hz.to_device(wpe, dtype)
    x = torch.full((T + 1, H), 3.0, dtype=wted.dtype, device="cuda")
    E.energon_embed_packed(torch.from_numpy(ids).cuda(), cu, wted, wped, x[:T])
    pos = np.concatenate([np.arange(n) for n in lens])
    want = (wted[torch.from_numpy(ids.astype(np.int64)).cuda()].float() + wped[torch.from_numpy(pos).cuda()].float()).to(wted.dtype)
    assert torch.equal(x[:T].view(torch.int16), want.view(torch.int16))     # one rounding of an exact fp32 sum
    assert torch.all(x[T] == 3.0), "row past T was written"


@pytest.mark.parametrize("A", WIDTHS)
def test_cache_fill_of_wide_rows(A):
    lens, S_cap = [5, 0, 9], 11
    T = sum(lens)
    qkv = torch.randint(-2 ** 15, 2 ** 15, (T, 3 * A), dtype=torch.int16, device="cuda")
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device="cuda")
    caches = [torch.full((3, S_cap, A), 77, dtype=torch.int16, device="cuda") for _ in range(2)]
    E.energon_cache_fill(qkv.view(torch.bfloat16), cu, *(c.view(torch.bfloat16) for c in caches))
    for c, part in zip(caches, (1, 2)):
        t = 0
        for b, n in enumerate(lens):
            assert torch.equal(c[b, :n], qkv[t:t + n, part * A:(part + 1) * A])
            assert torch.all(c[b, n:] == 77)
            t += n
