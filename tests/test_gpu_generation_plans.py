"""The ways a generation step can run: the few-row linear at edges of its rules and in every instance (rows, block columns, K
whole or cut over workgroups, ragged last block), asserted to be the one that the plan takes; the cached attention whole or with its keys cut over workgroups, at
cached lengths on both sides of a part's, a trip's and the cache's end; workspaces of the least size that is accepted."""
import numpy as np
import pytest
import torch

from oracle import energon_oracle as orc
from paper_2209_02341_amd import binding as E
from paper_2209_02341_amd import harness as hz
from paper_2209_02341_amd import workloads as wl
from tests.test_gpu_parity import assert_close, layer_noise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,dtype", [
    (1, 8, 64, wl.BF16), (16, 40, 192, wl.F16), (17, 1608, 1600, wl.BF16), (33, 4104, 512, wl.BF16), (64, 264, 3072, wl.F16),
    (3, 20488, 256, wl.BF16), (2, 5128, 5120, wl.BF16), (32, 5120, 5120, wl.F16), (50, 2056, 4096, wl.BF16),
    # both instances (whole and ragged last block) of 64, 32 and 16 columns at K of a few slabs, where the rule of that case decides
    (16, 16384, 768, wl.BF16), (9, 16376, 768, wl.F16), (20, 16384, 256, wl.BF16), (32, 16392, 320, wl.F16), (64, 3072, 768, wl.F16),
    (40, 3080, 768, wl.BF16)])
@pytest.mark.parametrize("epi", [E.EPI_BIAS, E.EPI_BIAS_GELU, E.EPI_BIAS_RESIDUAL])
def test_few_row_linear(M, N, K, dtype, epi):
    rng = np.random.default_rng(M + N + K + epi)
    x = wl.round_to_dtype(rng.standard_normal((M, K), dtype=np.float32), dtype)
    w = wl.round_to_dtype(rng.standard_normal((N, K), dtype=np.float32) / np.sqrt(K), dtype)
    b = wl.round_to_dtype(rng.standard_normal(N) * 0.5, dtype)
    r = wl.round_to_dtype(rng.standard_normal((M, N), dtype=np.float32), dtype)
    xd, wd, bd, rd = (hz.to_device(a, dtype) for a in (x, w, b, r))
    ref = orc.linear(x.astype(np.float64), w.astype(np.float64), b.astype(np.float64))
    ref = orc.gelu(ref) if epi == E.EPI_BIAS_GELU else ref + r if epi == E.EPI_BIAS_RESIDUAL else ref
    for nbytes in (0, 8 * M * N * 4):
        outs = []
        for fill in (0, 255):
            scratch = torch.full((nbytes,), fill, dtype=torch.uint8, device="cuda") if nbytes else None
            yd = torch.full((M + 1, N), 3.0, dtype=xd.dtype, device="cuda")
            E.energon_linear_with_scratch(xd, wd, bd, rd if epi == E.EPI_BIAS_RESIDUAL else None, yd, epi, scratch)
            assert torch.all(yd[M] == 3.0), "row past M was written"
            outs.append(yd[:M])
        assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
        assert_close(hz.to_host(outs[0]), ref, dtype, f"few-row linear epi={epi} scratch={nbytes}")


# every instance of the few-row kernel: rows of the tile x columns of a block x K whole or in parts x whole and ragged last
# block, at the smallest shape whose plan takes it
INSTANCES = [   # M, N, K, tile rows, block columns, parts of K
    (2, 16, 5120, 16, 16, 8), (2, 8, 5120, 16, 16, 8), (2, 16, 64, 16, 16, 1), (2, 8, 64, 16, 16, 1),
    (2, 352, 5120, 16, 32, 8), (2, 344, 5120, 16, 32, 8), (2, 4800, 64, 16, 32, 1), (2, 4104, 64, 16, 32, 1),
    (2, 1280, 8192, 16, 64, 8), (2, 1608, 10240, 16, 64, 8), (2, 10240, 64, 16, 64, 1), (2, 8200, 64, 16, 64, 1),
    (2, 2560, 8192, 16, 80, 8), (2, 2048, 10240, 16, 80, 8), (2, 17600, 64, 16, 80, 1), (2, 16392, 64, 16, 80, 1),
    (17, 16, 4096, 32, 16, 8), (17, 8, 4096, 32, 16, 8), (17, 16, 64, 32, 16, 1), (17, 8, 64, 32, 16, 1),
    (17, 320, 4096, 32, 32, 8), (17, 312, 4096, 32, 32, 8), (17, 4800, 64, 32, 32, 1), (17, 4104, 64, 32, 32, 1),
    (17, 1280, 5120, 32, 64, 8), (17, 1608, 5120, 32, 64, 8), (17, 10240, 64, 32, 64, 1), (17, 8200, 64, 32, 64, 1),
    (17, 2560, 4096, 32, 80, 8), (17, 2048, 5120, 32, 80, 8), (17, 17600, 2048, 32, 80, 1), (17, 16392, 2048, 32, 80, 1),
    (33, 16, 2048, 64, 16, 8), (33, 8, 2048, 64, 16, 8), (33, 16, 64, 64, 16, 1), (33, 8, 64, 64, 16, 1),
    (33, 288, 2048, 64, 32, 8), (33, 280, 2048, 64, 32, 8), (33, 4800, 64, 64, 32, 1), (33, 4104, 64, 64, 32, 1),
    (33, 1280, 2560, 64, 64, 8), (33, 1032, 2560, 64, 64, 8), (33, 10240, 64, 64, 64, 1), (33, 8200, 64, 64, 64, 1),
    (33, 2560, 2048, 64, 80, 8), (33, 2056, 2560, 64, 80, 8), (33, 17600, 64, 64, 80, 1), (33, 16392, 64, 64, 80, 1),
]


@pytest.mark.parametrize("M,N,K,rows,columns,parts", INSTANCES)
def test_few_row_instances(M, N, K, rows, columns, parts):
    room = 8 * M * N * 4 if parts > 1 else 0
    assert E.energon_linear_plan(M, N, K, scratch_bytes=room) == (0, rows, columns, parts)
    for epi in (E.EPI_BIAS, E.EPI_BIAS_GELU, E.EPI_BIAS_RESIDUAL):
        test_few_row_linear(M, N, K, wl.F16 if N % 16 else wl.BF16, epi)


# a part for every 256 cached keys, up to the launched one for every 512 of the cache: 1 and 3, 1 each, 4 each, 1 and 3
@pytest.mark.parametrize("nh,d,lens,S_cap,dtype", [(16, 64, [0, 1599], 1600, wl.BF16), (4, 128, [1, 63, 64], 1600, wl.F16),
                                                    (4, 128, [1000, 1023, 1024], 2048, wl.BF16), (2, 64, [5, 1535], 1536, wl.F16)])
def test_step_with_keys_in_parts(nh, d, lens, S_cap, dtype):
    rng = np.random.default_rng(S_cap + nh)
    H, F, B = 256, 512, len(lens)
    A = nh * d
    p = wl.random_small_layer(rng, H, nh, d, F, dtype, std=0.05)
    kc, vc = (wl.round_to_dtype(rng.standard_normal((B, S_cap, A)), dtype) for _ in range(2))
    x = wl.round_to_dtype(rng.standard_normal((B, H)), dtype)
    cfg, layer = hz.layer_config(H, nh, d, F, dtype), hz.DeviceLayer(p, dtype)
    lens = np.asarray(lens, np.int32)
    caches = [(kc[b, :n].astype(np.float64), vc[b, :n].astype(np.float64)) for b, n in enumerate(lens)]
    ref, k_new, v_new = orc.decode_layer(x, caches, p, nh, d, 1e-5)
    whole = E.energon_decode_workspace_bytes(cfg, B)
    least = E.energon_workspace_bytes(cfg, B)          # these shapes have had no partial sums: the six intermediates
    assert least < whole
    ys = []
    for nbytes in (least, whole, whole + 4096):
        kd, vd, xd = hz.to_device(kc, dtype), hz.to_device(vc, dtype), hz.to_device(x, dtype)
        yd = torch.empty_like(xd)
        args = (cfg, layer.struct, xd, yd, torch.from_numpy(lens).cuda(), lens, kd, vd)
        E.energon_decode_layer_forward(*args, torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda"))
        ys.append(yd)
        # weights of standard deviation 0.05 behind a LayerNorm of 256 features, cached keys of 1: logits of about 0.8
        assert_close(hz.to_host(yd), ref, dtype, f"step, workspace {nbytes}", **layer_noise(1, 1.0))
        for b, n in enumerate(lens):
            assert_close(hz.to_host(kd[b, n]), k_new[b], dtype, "appended key", stages=2)
            assert_close(hz.to_host(vd[b, n]), v_new[b], dtype, "appended value", stages=2)
            assert torch.equal(kd[b, :n].view(torch.int16), hz.to_device(kc[b, :n], dtype).view(torch.int16))
    assert torch.equal(ys[1].view(torch.int16), ys[2].view(torch.int16))
    with pytest.raises(E.EnergonError):
        E.energon_decode_layer_forward(*args, torch.empty(least - 256, dtype=torch.uint8, device="cuda"))


# scores of -inf (finite q and k whose products overflow) have weight 0 wherever they lie in the order the keys are taken:
# the first keys of some wavefronts, whole shares of keys cut over workgroups, the new token
HIDDEN = [range(16, 32), range(4, 60), [*range(3), 70, 200], range(370, 1100)]


def _overflowing(rng, B, S_cap, A, hidden, dtype):
    kc, vc = (rng.standard_normal((B, S_cap, A)) for _ in range(2))
    kc *= 1e-17
    kc[:, [j for j in hidden if j < S_cap]] = -1e25
    return wl.round_to_dtype(kc, dtype), wl.round_to_dtype(vc, dtype)


@pytest.mark.parametrize("hidden", HIDDEN)
@pytest.mark.parametrize("nh,d", [(3, 128), (5, 64)])
def test_cached_attention_scores_of_minus_infinity(hidden, nh, d):
    rng = np.random.default_rng(nh)
    B, S_cap, A = 2, 800, nh * d
    kc, vc = _overflowing(rng, B, S_cap, A, hidden, wl.BF16)
    qkv = rng.standard_normal((B, 3 * A))
    qkv[:, :A] = 1e15
    qkv[:, A:2 * A] *= 1e-17
    qkv[1, A:2 * A] = -1e25                              # sequence 1: its own key too
    qkv = wl.round_to_dtype(qkv, wl.BF16)
    lens = np.asarray([90, 799], np.int32)
    kd, vd = hz.to_device(kc, wl.BF16), hz.to_device(vc, wl.BF16)
    out = torch.empty((B, A), dtype=torch.bfloat16, device="cuda")
    E.energon_decode_attention(hz.to_device(qkv, wl.BF16), kd, vd, torch.from_numpy(lens).cuda(), nh, d, out)
    q = qkv.astype(np.float64)
    ref = np.stack([orc.decode_attention(q[b, :A], q[b, A:2 * A], q[b, 2 * A:], kc[b, :n].astype(np.float64),
                                         vc[b, :n].astype(np.float64), nh, d) for b, n in enumerate(lens)])
    assert_close(hz.to_host(out), ref, wl.BF16, "attention", stages=2)


@pytest.mark.parametrize("hidden", HIDDEN)
def test_step_with_keys_in_parts_and_scores_of_minus_infinity(hidden):
    rng = np.random.default_rng(1)
    H, F, nh, d, B, S_cap = 256, 512, 4, 128, 2, 2048
    A = nh * d
    p = wl.random_small_layer(rng, H, nh, d, F, wl.BF16, std=0.05)
    p["w_qkv"][:2 * A] = 0.0                             # q = 1e15, k = 1e-17 times normal, for every token
    p["b_qkv"] = wl.round_to_dtype(np.concatenate([np.full(A, 1e15), rng.standard_normal(A) * 1e-17,
                                                   rng.standard_normal(A)]), wl.BF16)
    kc, vc = _overflowing(rng, B, S_cap, A, hidden, wl.BF16)
    x = wl.round_to_dtype(rng.standard_normal((B, H)), wl.BF16)
    cfg, layer = hz.layer_config(H, nh, d, F, wl.BF16), hz.DeviceLayer(p, wl.BF16)
    lens = np.asarray([1500, 2047], np.int32)
    ref, _, _ = orc.decode_layer(x, [(kc[b, :n].astype(np.float64), vc[b, :n].astype(np.float64))
                                     for b, n in enumerate(lens)], p, nh, d, 1e-5)
    yd = torch.empty((B, H), dtype=torch.bfloat16, device="cuda")
    ws = torch.full((E.energon_decode_workspace_bytes(cfg, B),), 255, dtype=torch.uint8, device="cuda")
    E.energon_decode_layer_forward(cfg, layer.struct, hz.to_device(x, wl.BF16), yd, torch.from_numpy(lens).cuda(), lens,
                                   hz.to_device(kc, wl.BF16), hz.to_device(vc, wl.BF16), ws)
    assert_close(hz.to_host(yd), ref, wl.BF16, "step", **layer_noise(1, 1.0))


# workgroups of four wavefronts, one step of loads ahead (640 to 2048 heads) and two, of eight (up to 256); lengths around a
# trip of either
@pytest.mark.parametrize("B,nh,d", [(64, 4, 64), (65, 4, 128), (160, 4, 128), (512, 4, 64), (513, 4, 64), (64, 10, 64)])
def test_cached_attention_of_many_heads(B, nh, d):
    rng = np.random.default_rng(B)
    S_cap, A, dtype = 300, nh * d, wl.F16 if d == 64 else wl.BF16
    kinds = [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 127, 128, 299]
    lens = np.asarray((kinds * B)[:B], np.int32)
    n = len(kinds)                                       # distinct sequences, over and over
    kc, vc = (wl.round_to_dtype(rng.standard_normal((n, S_cap, A)), dtype) for _ in range(2))
    qkv = wl.round_to_dtype(rng.standard_normal((n, 3 * A)), dtype)
    at = torch.arange(B, device="cuda") % n
    kd, vd, qd = (hz.to_device(t, dtype)[at].contiguous() for t in (kc, vc, qkv))
    out = torch.empty((B, A), dtype=qd.dtype, device="cuda")
    E.energon_decode_attention(qd, kd, vd, torch.from_numpy(lens).cuda(), nh, d, out)
    q = qkv.astype(np.float64)
    ref = np.stack([orc.decode_attention(q[b, :A], q[b, A:2 * A], q[b, 2 * A:], kc[b, :l].astype(np.float64),
                                         vc[b, :l].astype(np.float64), nh, d) for b, l in enumerate(kinds)])
    assert_close(hz.to_host(out), ref[np.arange(B) % n], dtype, "attention", stages=2)
