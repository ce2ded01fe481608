"""Which blocks the 16-bit attention kernel computes: batches whose padded length leaves most query blocks empty (the
kernel then counts only the blocks that have queries, from a scan of up to 256 lengths), batches beyond that limit
and dense ones (blocks straight from the workgroup id, longest first, or in groups of (sequence, head) pairs per XCD where
there are many), head counts that the 8 XCDs do not share evenly, sequences at the edges of the 32-key tiles and
128-query blocks.  Against the oracle at the suite's bars."""
import numpy as np
import pytest
import torch

from oracle import energon_oracle as orc
from paper_2209_02341_amd import binding as E
from paper_2209_02341_amd import harness as hz
from paper_2209_02341_amd import workloads as wl
from tests.test_gpu_parity import assert_close

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 160, 193, 256, 257]
CASES = [
    # lengths, max_len, heads, head width, dtype
    ([700] + [1, 0, 33] * 23, 700, 3, 64, wl.BF16),        # 70 sequences: two per lane of the scan
    ([0, 0, 900, 5, 0, 1, 40, 129], 2048, 9, 128, wl.BF16),
    (EDGES, 1024, 8, 128, wl.F16),                          # scan, heads shared evenly
    (EDGES, 257, 5, 128, wl.BF16),                          # no scan
    (EDGES, 257, 2, 64, wl.F16),
    ([2, 17, 0, 140] * 64, 600, 2, 64, wl.BF16),            # 256 sequences: the most the scan takes
    ([3, 20, 0, 130] * 65, 600, 2, 64, wl.BF16),            # 260: beyond it
    ([320], 320, 12, 128, wl.BF16),
]


@pytest.mark.parametrize("lens,S,nh,d,dtype", CASES)
def test_attention_blocks(lens, S, nh, d, dtype):
    lens = np.asarray(lens, np.int32)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, A = int(cu[-1]), nh * d
    qkv = wl.round_to_dtype(np.random.default_rng(S + nh).standard_normal((T, 3 * A)), dtype)
    out = torch.full((T + 1, A), 3.0, dtype=hz.to_device(np.zeros(1), dtype).dtype, device="cuda")
    E.energon_attention(hz.to_device(qkv, dtype), out[:T], torch.from_numpy(cu).cuda(), len(lens), S, nh, d)
    out = hz.to_host(out)
    assert np.all(out[T] == 3.0), "row past T was written"
    for b, n in enumerate(lens):
        if n:
            blk = qkv[cu[b]:cu[b + 1]].astype(np.float64)
            ref = orc.masked_causal_attention(blk[:, :A], blk[:, A:2 * A], blk[:, 2 * A:], int(n), nh, d)
            assert_close(out[cu[b]:cu[b + 1]], ref, dtype, f"attention seq {b}", stages=2)   # P, then the output


# more than 4.5 rounds of workgroups (2304 at width 128, 3456 at 64): pairs in groups per XCD, 4 pairs left over
@pytest.mark.parametrize("B,nh,d,dtype", [(300, 5, 128, wl.BF16), (300, 7, 64, wl.F16)])
@pytest.mark.parametrize("padded", [False, True])
def test_attention_blocks_in_groups(B, nh, d, dtype, padded):
    S, A = 257, nh * d
    kinds = [130, 1, 129, 257, 256]                      # five sequences, over and over
    lens = np.asarray((kinds * B)[:B], np.int32)
    rng = np.random.default_rng(d)
    blocks = [wl.round_to_dtype(rng.standard_normal((n, 3 * A)), dtype) for n in kinds]
    refs = []
    for n, blk in zip(kinds, (b.astype(np.float64) for b in blocks)):
        refs.append(orc.masked_causal_attention(blk[:, :A], blk[:, A:2 * A], blk[:, 2 * A:], n, nh, d))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cud, T = torch.from_numpy(cu).cuda(), int(cu[-1])
    qkv = hz.to_device(np.concatenate([blocks[b % len(kinds)] for b in range(B)]), dtype)
    out = torch.full((T + 1, A), 3.0, dtype=qkv.dtype, device="cuda")
    if padded:
        q, k, v, o = (torch.full((B, nh, S, d), 3.0, dtype=qkv.dtype, device="cuda") for _ in range(4))
        E.energon_rebuild_qkv(qkv, cud, B, S, nh, d, q, k, v)
        E.energon_attention_padded(q, k, v, cud, o)
        E.energon_remove_attn_padding(o, cud, out[:T])
    else:
        E.energon_attention(qkv, out[:T], cud, B, S, nh, d)
    out = hz.to_host(out)
    assert np.all(out[T] == 3.0), "row past T was written"
    for b in range(B):
        assert_close(out[cu[b]:cu[b + 1]], refs[b % len(kinds)], dtype, f"attention seq {b}", stages=2)


# finite q and k whose product is -inf in fp32 (bf16 reaches 1e38) have weight 0 wherever they lie, also as the first tiles of a query
@pytest.mark.parametrize("hidden", [range(64), range(200), [*range(16), *range(32, 160)], range(70, 140)])
@pytest.mark.parametrize("d", [64, 128])
def test_attention_scores_of_minus_infinity(hidden, d):
    n, nh = 300, 2
    A = nh * d
    qkv = wl.round_to_dtype(np.random.default_rng(d).standard_normal((n, 3 * A)), wl.BF16)
    qkv[:, :A], qkv[:, A:2 * A] = 2.0 ** 66, 0.0     # the other keys score 0: equal weights
    qkv[list(hidden), A:2 * A] = -2.0 ** 66
    out = torch.empty((n, A), dtype=torch.bfloat16, device="cuda")
    cu = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    E.energon_attention(hz.to_device(qkv, wl.BF16), out, cu, 1, n, nh, d)
    seen = np.array([any(j not in hidden for j in range(i + 1)) for i in range(n)])
    blk = qkv.astype(np.float64)
    ref = orc.masked_causal_attention(blk[:, :A], blk[:, A:2 * A], blk[:, 2 * A:], n, nh, d)
    assert_close(hz.to_host(out)[seen], ref[seen], wl.BF16, "attention past scores of -inf", stages=2)
