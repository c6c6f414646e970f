"""The hot calls only enqueue kernels on the caller's stream (no allocation, no synchronisation, no memset), so a
caller can capture them in a HIP graph: decode attention captured once and replayed with new queries in the same
buffers, every replay compared with the eager call, with eager work and synchronisations between the replays."""
import pytest
import torch

from paper_2507_20030_amd import binding as B
from paper_2507_20030_amd import workload as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("name,cfg", [
    ("fft", wl.Config("g_fft", 2, 2, 2, 4, 128, 1024, 200, 4, "bf16", "mixed", n_sink=3, n_recent=5, seed=21)),
    ("chirp", wl.Config("g_chirp", 1, 2, 2, 2, 128, 1000, 150, 4, "f32", "low", seed=22)),
    # softmax on interpolated grids (a length that is no power of two, a long context of low frequencies)
    ("grid", wl.Config("g_grid", 1, 2, 2, 2, 128, 3000, 700, 4, "f32", "low", n_sink=3, n_recent=5, seed=24)),
    ("low", wl.Config("g_low", 2, 2, 2, 4, 128, 32768, 1000, 4, "bf16", "low", n_sink=3, n_recent=5, seed=25)),
    # long context with many slices: kernels A and B pipelined over groups of slices (10 launches per call)
    ("pipelined", wl.Config("g_pipe", 16, 8, 8, 4, 128, 16384, 1100, 4, "bf16", "mixed", seed=23)),
])
def test_decode_attention_in_a_captured_graph(name, cfg):
    bins = wl.layer_bins(cfg)
    K, V = wl.prefill_tensors(cfg, DEV)
    cache = B.Cache(cfg.n_layers, cfg.batch, cfg.n_kv_heads, cfg.n_q_heads, cfg.head_dim, cfg.torch_dtype,
                    cfg.L, bins, device=DEV, n_sink=cfg.n_sink, n_recent=cfg.n_recent)
    assert B.iwdft_attn_kind(cache.ctx) == ("chirp" if name in ("chirp", "grid") else "fft")
    assert B.iwdft_attn_pipelined(cache.ctx) == (name == "pipelined")
    cache.prefill(K, V)
    for i in range(2):
        tk, tv, _ = wl.decode_step(cfg, i, DEV)
        cache.append(tk, tv)
    qs = [wl.decode_step(cfg, 10 + i, DEV)[2] for i in range(4)]
    q_buf, out_buf = qs[0].clone(), torch.empty_like(qs[0])
    cache.attend(q_buf, out_buf)                      # eager once: one-time kernel attributes are set outside the capture
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        cache.attend(q_buf, out_buf, 0.0, torch.cuda.current_stream())
    for i, q in enumerate(qs):
        ref = cache.attend(q).clone()                 # eager work between the replays
        torch.cuda.synchronize()
        q_buf.copy_(q)
        out_buf.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out_buf, ref), f"{name}: replay {i} differs from the eager call"
    cache.close()


@pytest.mark.parametrize("cfg", [
    wl.Config("p_low", 1, 1, 9, 1, 128, 65536, 4000, 4, "bf16", "low", n_sink=3, n_recent=5, seed=26),  # decimated: three groups of slices
    wl.Config("p_any", 1, 2, 8, 1, 128, 12290, 300, 4, "f32", "low", seed=27),                          # two blocks of 6145 points
])
def test_prefill_in_a_captured_graph(cfg):
    bins = wl.layer_bins(cfg)
    cache = B.Cache(cfg.n_layers, cfg.batch, cfg.n_kv_heads, cfg.n_q_heads, cfg.head_dim, cfg.torch_dtype, cfg.L, bins, device=DEV,
                    n_sink=cfg.n_sink, n_recent=cfg.n_recent)
    gen = torch.Generator(DEV).manual_seed(cfg.seed)
    K, V = wl.prefill_tensors(cfg, DEV)
    cache.prefill(K, V)                               # eager once: one-time kernel attributes are set outside the capture
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        cache.prefill(K, V, torch.cuda.current_stream())
    for i in range(4):
        for x in (K, V):
            x.copy_(torch.randn(x.shape, generator=gen, device=DEV))
        cache.prefill(K, V)                           # eager work between the replays
        ref = cache.export_coeffs(0)
        torch.cuda.synchronize()
        K2, V2 = K.clone(), V.clone()
        for x in (K, V):
            x.zero_()
        cache.prefill(K, V)                           # another state
        K.copy_(K2), V.copy_(V2)
        g.replay()
        for x, y in zip(cache.export_coeffs(0), ref):
            assert torch.equal(x, y), f"replay {i} differs from the eager call"
    cache.close()
