"""A small fp32 layer, whose linears normalise their rows themselves: ragged row tiles, one row, the widest and the next wider
hidden size (which takes launches of its own), against the oracle; the normalised rows are left in the workspace as before."""
import numpy as np
import pytest
import torch

from oracle import energon_oracle as orc
from paper_2209_02341_amd import binding as E
from paper_2209_02341_amd import harness as hz
from paper_2209_02341_amd import workloads as wl

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.mark.parametrize("lens,H,nh,F", [([1], 128, 2, 512), ([17, 3, 13], 256, 4, 1024), ([5, 11], 512, 8, 1024), ([16, 33], 68, 1, 260),
                                         ([9, 4], 576, 9, 640), ([40, 31, 1], 256, 4, 300)])
def test_small_f32_layer(lens, H, nh, F):
    w = wl.Workload("small_ln", wl.F32, 1, H, nh, 64, F, len(lens), max(lens), "uniform", 0, max(lens))
    lens = np.asarray(lens, np.int32)
    T, A = int(lens.sum()), nh * 64
    rng = np.random.default_rng(H + T)
    p = wl.random_small_layer(rng, H, nh, 64, F)   # gain around 1, an offset
    x = rng.normal(1.0, 2.0, (T, H)).astype(np.float32)   # a mean far from zero
    cfg = hz.layer_config(H, nh, 64, F, wl.F32, w.ln_eps)
    layer = hz.DeviceLayer(p, wl.F32)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ws = torch.full((E.energon_workspace_bytes(cfg, T),), 255, dtype=torch.uint8, device="cuda")
    y = torch.full((T + 1, H), 3.0, device="cuda")
    E.energon_layer_forward(cfg, layer.struct, hz.to_device(x, wl.F32), y[:T], T, torch.from_numpy(cu).cuda(), lens, int(lens.max()), ws)
    assert torch.all(y[T] == 3.0), "row past T was written"
    off = E.energon_workspace_layout(cfg, T)
    f32 = lambda slot, n: hz.to_host(ws[off[slot]: off[slot] + T * n * 4].view(torch.float32).view(T, n))
    d = {k: None if v is None else np.asarray(v, np.float64) for k, v in p.items()}
    # LayerNorm: sums of H terms, the deviation's root, four roundings; gain and offset of order one
    u = orc.layer_norm(x.astype(np.float64), d["ln1_g"], d["ln1_b"], w.ln_eps)
    assert np.abs(f32(E.WS_U, H) - u).max() <= (H + 16) * U * np.abs(u).max()
    qkv = orc.linear(u, d["w_qkv"], d["b_qkv"])
    bound = (2 * H + 32) * U * (np.abs(u).max() * np.abs(d["w_qkv"]).sum(1).max() + np.abs(d["b_qkv"]).max())
    assert np.abs(f32(E.WS_QKV, 3 * A) - qkv).max() <= bound
    y1 = f32(E.WS_Y1, H).astype(np.float64)
    wn = orc.layer_norm(y1, d["ln2_g"], d["ln2_b"], w.ln_eps)
    assert np.abs(f32(E.WS_W, H) - wn).max() <= (H + 16) * U * np.abs(wn).max()
    m = orc.gelu(orc.linear(wn, d["w_fc1"], d["b_fc1"]))
    bound = 1.13 * (2 * H + 32) * U * (np.abs(wn).max() * np.abs(d["w_fc1"]).sum(1).max() + np.abs(d["b_fc1"]).max()) + 1.3e-7
    assert np.abs(f32(E.WS_M, F) - m).max() <= bound + 8 * U * np.abs(m).max()


@pytest.mark.parametrize("lens,H,nh,F", [([17, 3, 13], 256, 4, 1024), ([9, 4], 576, 9, 640)])
def test_the_timed_layer_is_the_one_that_runs(lens, H, nh, F):
    """energon_layer_forward_profiled makes the same launches: the same bits of everything, in a layer whose linears normalise their
    rows themselves and in one that has launches for it."""
    lens = np.asarray(lens, np.int32)
    T = int(lens.sum())
    rng = np.random.default_rng(H)
    layer = hz.DeviceLayer(wl.random_small_layer(rng, H, nh, 64, F), wl.F32)
    cfg = hz.layer_config(H, nh, 64, F, wl.F32, 1e-5)
    x = hz.to_device(rng.normal(1.0, 2.0, (T, H)).astype(np.float32), wl.F32)
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
    left = []
    for call in (E.energon_layer_forward, E.energon_layer_forward_profiled):
        ws, y = torch.zeros(E.energon_workspace_bytes(cfg, T), dtype=torch.uint8, device="cuda"), torch.empty_like(x)
        ms = call(cfg, layer.struct, x, y, T, cu, lens, int(lens.max()), ws)
        left.append((y, ws))
    assert list(ms) == list(E.STAGE_NAMES) and all(v >= 0.0 for v in ms.values())
    for a, b in zip(*left):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


def _replayed_us(body):
    """us per call of `body`, twenty of them captured into a graph: what the device takes, without the host's time between launches."""
    body()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(20):
            body()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    times = []
    for _ in range(15):
        a.record()
        graph.replay()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 50.0)
    return sorted(times)[7]


@pytest.mark.parametrize("lens,H,nh,F", [([12, 12, 12, 12], 512, 2, 512), ([30, 25, 22], 256, 4, 1024)])
def test_a_replayed_layer_takes_no_longer_than_its_stages_apart(lens, H, nh, F):
    """Normalising in the linear saves launches, also where they cost little.  A tenth is left for the clocks."""
    lens = np.asarray(lens, np.int32)
    T, A = int(lens.sum()), nh * 64
    rng = np.random.default_rng(H)
    layer = hz.DeviceLayer(wl.random_small_layer(rng, H, nh, 64, F), wl.F32)
    p = layer.tensors
    cfg = hz.layer_config(H, nh, 64, F, wl.F32, 1e-5)
    x = hz.to_device(rng.normal(1.0, 2.0, (T, H)).astype(np.float32), wl.F32)
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
    ws = torch.empty(E.energon_workspace_bytes(cfg, T), dtype=torch.uint8, device="cuda")
    new = lambda n: torch.empty((T, n), device="cuda")
    u, qkv, att, y1, wn, m, y, whole = new(H), new(3 * A), new(A), new(H), new(H), new(F), new(H), new(H)

    def apart():
        E.energon_layernorm(x, p["ln1_g"], p["ln1_b"], u, 1e-5)
        E.energon_linear(u, p["w_qkv"], p["b_qkv"], None, qkv, E.EPI_BIAS)
        E.energon_attention(qkv, att, cu, len(lens), int(lens.max()), nh, 64)
        E.energon_linear(att, p["w_o"], p["b_o"], x, y1, E.EPI_BIAS_RESIDUAL)
        E.energon_layernorm(y1, p["ln2_g"], p["ln2_b"], wn, 1e-5)
        E.energon_linear(wn, p["w_fc1"], p["b_fc1"], None, m, E.EPI_BIAS_GELU)
        E.energon_linear(m, p["w_fc2"], p["b_fc2"], y1, y, E.EPI_BIAS_RESIDUAL)

    together = lambda: E.energon_layer_forward(cfg, layer.struct, x, whole, T, cu, lens, int(lens.max()), ws)
    assert _replayed_us(together) <= 1.1 * _replayed_us(apart)
    assert (whole - y).abs().max() <= 1e-5 * y.abs().max()
