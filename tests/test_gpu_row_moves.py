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
