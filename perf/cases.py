"""Timed cases of the K/V-cache path: what a program that keeps its cache in the frequency domain has the library do.

Each case is one pass through the public calls of ``paper_2507_20030_amd.binding``: decode steps (fused, or append and
attention as two calls), the prefill of a context, the reconstruction of a layer, the ablation of one frequency chunk.
Sizes follow the configurations in ``workload.py`` (fewer layers where the inputs would take long to make).
"""
import math

import numpy as np
import torch

from paper_2507_20030_amd import binding

HEAD_DIM = 128
SINK, RECENT = 10, 50  # the exact windows of the paper's own setting


def _case(name, kind, layers, batch, group, M, bins, dtype="bf16", mask="low", windows=False, write_every=0, steps=1,
          outliers=0):
    case = dict(kind=kind, layers=layers, batch=batch, kv_heads=8, group=group, M=M, bins=bins, dtype=dtype, mask=mask,
                windows=windows, write_every=write_every, steps=steps, outliers=outliers)
    return dict(case, name=name) if name else case


def listed():
    return [
        # The smallest decode step: one layer in fp32, one query head per KV head -- a model in a debugger, a unit test,
        # the draft model of a speculative decoder.  Latency and launches count.
        _case("decode-one-layer-1k-f32", "decode", 1, 1, 1, 1024, 64, dtype="f32"),
        # One user of an 8-billion-parameter model at 8192 tokens, a quarter of the bins kept: 16 generated tokens, the
        # coefficients written back once at their end (write_every 16).
        _case("decode-8k", "decode", 32, 1, 4, 8192, 2048, write_every=16, steps=16),
        # The same model with the paper's windows cut out of the 8192-token context: M = 8132 is not a power of two.
        _case("decode-8k-windows", "decode", 32, 1, 4, 8192 - SINK - RECENT, 2033, windows=True, write_every=16, steps=16),
        # One user with a document of 131072 tokens.
        _case("decode-128k", "decode", 32, 1, 4, 131072, 4096, write_every=16, steps=16),
        # A served batch of a model with 8 query heads per KV head, masks per layer, outlier channels in K (20 of its 80
        # layers).
        _case("decode-batch16-16k", "decode", 20, 16, 8, 16384, 1638, mask="mixed", outliers=4, write_every=16, steps=16),
        # Append and attention as two calls (a program that samples or edits in between), batch 8 at 32768 tokens (8 of 32
        # layers).
        _case("append-attend-32k", "split", 8, 8, 4, 32768, 4096, mask="mixed"),
        # The smallest prefill: one layer in fp32, a short prompt.
        _case("prefill-one-layer-1k-f32", "prefill", 1, 1, 1, 1024, 64, dtype="f32"),
        # Prefill of the ordinary 8192-token context ...
        _case("prefill-8k", "prefill", 32, 1, 4, 8192, 2048),
        # ... with the paper's windows cut out of it ...
        _case("prefill-8k-windows", "prefill", 32, 1, 4, 8192 - SINK - RECENT, 2033, windows=True),
        # ... and of the long document (8 of 32 layers).
        _case("prefill-128k", "prefill", 8, 1, 4, 131072, 4096),
        # K~, V~ of one layer in memory for a standard attention kernel: the paper's own decode step, batch 8.
        _case("reconstruct-8k", "reconstruct", 1, 8, 4, 8192, 2048),
        # The offline study of the masks: one of 22 chunks taken out of a layer's K at 8192 tokens, batch 8.
        _case("ablate-8k", "ablate", 1, 8, 4, 8192, 0),
    ]


def _has_short_transform(M):
    """Whether M takes the O(M log M) attention: a power of two, or some divisor brings it down to 8192 points."""
    return M & (M - 1) == 0 or any(M % p == 0 and M // p <= 8192 for p in range(1, 257))


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 5 + ["prefill"] * 4 + ["split", "reconstruct", "ablate"])
    windows = kind in ("decode", "prefill", "split") and rng.random() < 0.4
    pow2 = 2 ** rng.randint(9, 13 if kind == "ablate" else 15 if kind == "reconstruct" else 17)
    M = pow2
    if windows and rng.random() < 0.75:  # windows cut out of a context of any length, else added to a power of two
        while True:
            M = _log_uniform(rng, 512, 32768) - SINK - RECENT
            if _has_short_transform(M):
                break
    bins = max(16, min(4096, int(M * rng.uniform(0.05, 0.25))))
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    group = rng.choice([1, 2, 4, 4, 8])
    mask = "mixed" if bins >= 512 and rng.random() < 0.5 else "low"
    # slices: from one layer of one sequence up to what the largest listed cases hold, in coefficients and in tokens
    most = min(2560, (20 * 128 * 1638) // bins, (256 * 131072 if kind in ("decode", "split") else 64 * 131072) // M)
    if kind in ("reconstruct", "ablate"):
        most = min(most, 64)
    units = _log_uniform(rng, 1, max(1, most // 8))  # of 8 KV heads each
    batch = 1 if kind in ("decode", "prefill", "split") and rng.random() < 0.5 else rng.randint(1, min(16, units))
    layers = 1 if kind in ("reconstruct", "ablate") else max(1, units // batch)
    write_every, steps = rng.choice([(0, 1), (8, 8), (16, 16), (16, 16)]) if kind == "decode" else (0, 1)
    return _case(None, kind, layers, batch, group, M, 0 if kind == "ablate" else bins, dtype, mask, windows, write_every,
                 steps, rng.choice([0, 0, 4]))


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _layer_bins(case, seed):
    """Kept bins per layer: the low band, or (every other layer of "mixed") a low band and 64-bin groups up to M / 2."""
    M, n, out = case["M"], case["bins"], []
    rng = np.random.default_rng(seed)
    for layer in range(case["layers"]):
        n_mid = n // 128 if case["mask"] == "mixed" and layer % 2 else 0
        starts = np.arange(-(-(n - 64 * n_mid) // 64), M // 128) * 64
        n_mid = min(n_mid, len(starts))
        pick = np.sort(rng.choice(starts, size=n_mid, replace=False)) if n_mid else []
        low = np.arange(n - 64 * n_mid)
        out.append(np.concatenate([low, *(np.arange(s, s + 64) for s in pick)]).astype(np.int32))
    return out


def _fill(shape, scale, dtype, gen):
    """[layers, ...] normal values; scale [layers, kv heads, channels] or None."""
    x = torch.empty(shape, dtype=dtype, device="cuda")
    for layer in range(shape[0]):
        v = torch.randn(shape[1:], generator=gen, device="cuda")
        if scale is not None:
            v *= scale[layer][:, None, :] if len(shape) == 5 else scale[layer]
        x[layer] = v
    return x


def _coefficients(case, cache):
    """The cache's complex coefficients (K then V) as stored: the last part of the state but for the exact tokens."""
    slices = case["batch"] * case["kv_heads"]
    rows = sum(-(-len(b) // 32) * 32 for b in cache.desc.bins)  # rows are padded to 32 bins
    exact = (SINK + RECENT if case["windows"] else 0) * 2 * case["layers"] * slices * HEAD_DIM * _dtype(case).itemsize
    end = cache.state_bytes - exact
    return cache.state[end - 2 * 8 * slices * HEAD_DIM * rows:end].view(torch.float32)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    L, B, H, dtype = case["layers"], case["batch"], case["kv_heads"], _dtype(case)
    scale = 10.0 ** (2.0 * torch.rand((L, H, HEAD_DIM), generator=gen, device="cuda") - 1.0)  # K: log-uniform per channel
    if case["outliers"]:
        scale[:, :, torch.randperm(HEAD_DIM, generator=gen, device="cuda")[:case["outliers"]]] *= 20.0
    if case["kind"] == "ablate":
        return dict(case=case, x=_fill((L, B, H, case["M"], HEAD_DIM), scale, dtype, gen))
    sink, recent = (SINK, RECENT) if case["windows"] else (0, 0)
    cache = binding.Cache(L, B, H, H * case["group"], HEAD_DIM, dtype, case["M"], _layer_bins(case, seed), n_sink=sink,
                          n_recent=recent, write_every=case["write_every"])
    tokens = (L, B, H, sink + case["M"] + recent, HEAD_DIM)
    K, V = _fill(tokens, scale, dtype, gen), _fill(tokens, None, dtype, gen)
    state = dict(case=case, cache=cache, coefficients=_coefficients(case, cache))
    if case["kind"] == "prefill":
        return dict(state, K=K, V=V)
    cache.prefill(K, V)
    row = (L, B, H, HEAD_DIM)
    state["tokens"] = [(_fill(row, scale, dtype, gen), _fill(row, None, dtype, gen),
                        _fill((L, B, H * case["group"], HEAD_DIM), None, dtype, gen)) for _ in range(case["steps"])]
    return state


def run(state):
    kind = state["case"]["kind"]
    if kind == "ablate":
        out = torch.empty_like(state["x"])
        binding.iwdft_ablate_chunk(state["x"], out, 22, 3)
        return out
    cache = state["cache"]
    if kind == "prefill":
        cache.prefill(state["K"], state["V"])
        return state["coefficients"]
    if kind == "reconstruct":
        return cache.reconstruct(0, 0, state["case"]["M"])
    outs = []
    for tok_k, tok_v, q in state["tokens"]:
        if kind == "split":
            cache.append(tok_k, tok_v)
            outs.append(cache.attend(q))
        else:
            outs.append(cache.step(tok_k, tok_v, q))
    return outs, state["coefficients"]


def work(case):
    slices = case["layers"] * case["batch"] * case["kv_heads"]
    M, item, heads = case["M"], _dtype(case).itemsize, slices * case["group"]
    tensor = slices * M * HEAD_DIM * item  # K or V over the transformed tokens
    coefs = 2 * 8 * slices * HEAD_DIM * case["bins"]  # both tensors, complex fp32
    exact = 2 * slices * (SINK + RECENT if case["windows"] else 0) * HEAD_DIM * item
    real_transform = 2.5 * M * math.log2(M)  # of M real samples
    if case["kind"] == "ablate":
        return dict(bytes=2 * tensor, flops=2 * slices * HEAD_DIM * real_transform)
    if case["kind"] == "prefill":
        return dict(bytes=2 * tensor + 2 * exact + coefs, flops=2 * slices * HEAD_DIM * real_transform)
    if case["kind"] == "reconstruct":
        return dict(bytes=2 * tensor + coefs, flops=2 * slices * HEAD_DIM * real_transform)
    rows = (2 * slices + 2 * heads) * HEAD_DIM * item  # tokens, queries, outputs
    step_flops = heads * (2 * 4 * HEAD_DIM * case["bins"] + 2 * real_transform)
    return dict(bytes=case["steps"] * (coefs + exact + rows) + coefs,
                flops=case["steps"] * step_flops + coefs / 8 * 4 * case["steps"])


def tolerance(case):
    """Four times what was measured between two correct paths: contraction, transforms and 64-bit sums (prefill, ablation),
    transforms and direct sums (the rest); bf16 outputs differ where a sum lies next to a rounding boundary."""
    if case["kind"] == "prefill":
        return {"rel": 1.6e-5, "max": 2.4e-4}
    if case["dtype"] == "f32":
        return {"rel": 3e-5, "max": 4e-4}
    return {"rel": 6.4e-4, "max": 0.031}
