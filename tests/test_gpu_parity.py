"""GPU parity: every C-ABI call against the float64 oracle on the same seeded inputs.

Tolerances (relative L2 over the compared tensor):
  coefficients (fp32 complex)            1e-4   (stated target)
  attention output, bf16 storage         2e-2   (stated target)
  attention output, fp32 storage         1e-4   (fp32 arithmetic: FFT + exp of scores of
                                                 magnitude <~ 50 gives ~1e-5; one decade of slack)
  reconstruction, fp32 / bf16 storage    1e-4 / 4e-3 (bf16 rounding alone is 2^-9 per element)
Kept-bin masks read back from the device must be bit-exact.
"""
import time

import numpy as np
import pytest
import torch

from oracle import iwdft_oracle as orc
from paper_2507_20030_amd import binding as B
from paper_2507_20030_amd import workload as wl

pytestmark = pytest.mark.gpu

TOL_COEF = 1e-4
TOL_ATTN = {torch.float32: 1e-4, torch.bfloat16: 2e-2}
TOL_REC = {torch.float32: 1e-4, torch.bfloat16: 4e-3}
DEV = "cuda:0"


def rel_l2(a, ref):
    return float(np.linalg.norm(np.asarray(a) - ref) / max(np.linalg.norm(ref), 1e-300))


def f64(t):
    return t.detach().to("cpu").to(torch.float64).numpy()


def c128(t):
    return t.detach().to("cpu").numpy().astype(np.complex128)


def make_cache(cfg, bins, weights=None, flags=0, write_every=0):
    return B.Cache(cfg.n_layers, cfg.batch, cfg.n_kv_heads, cfg.n_q_heads, cfg.head_dim, cfg.torch_dtype,
                   cfg.L, bins, weights, flags, DEV, n_sink=cfg.n_sink, n_recent=cfg.n_recent,
                   write_every=write_every)


class SliceOracle:
    """Float64 state of a few sampled slices, advanced next to the GPU cache: coefficients of the
    transformed middle segment plus the exact sink tokens and the recent window (Sec. 4.2)."""

    def __init__(self, cfg, bins, weights, K, V, slices):
        self.cfg, self.bins, self.weights, self.slices = cfg, bins, weights, slices
        self.M = cfg.L
        self.T = cfg.L
        self.S, self.sink, self.recent = {}, {}, {}
        s0, s1 = cfg.n_sink, cfg.n_sink + cfg.L
        for key in slices:
            l = key[0]
            k, v = f64(K[key]), f64(V[key])
            self.S[key] = [orc.prefill(k[s0:s1], bins[l]), orc.prefill(v[s0:s1], bins[l])]
            self.sink[key] = (k[:s0], v[:s0])
            self.recent[key] = ([r for r in k[s1:]], [r for r in v[s1:]])

    def append(self, tk, tv):
        for key, st in self.S.items():
            l = key[0]
            rk, rv = self.recent[key]
            rk.append(f64(tk[key]))
            rv.append(f64(tv[key]))
            st[0] = orc.append(st[0], rk.pop(0), self.T, self.bins[l], self.M)
            st[1] = orc.append(st[1], rv.pop(0), self.T, self.bins[l], self.M)
        self.T += 1

    def attend(self, q):
        G, d = self.cfg.group, self.cfg.head_dim
        out = {}
        for key, st in self.S.items():
            l, b, h = key
            w = None if self.weights is None else self.weights[l]
            rk, rv = self.recent[key]
            rk = np.stack(rk) if rk else np.zeros((0, d))
            rv = np.stack(rv) if rv else np.zeros((0, d))
            out[key] = orc.windowed_attention(f64(q[l, b, h * G:(h + 1) * G]), self.sink[key][0], self.sink[key][1],
                                              st[0], st[1], self.T, self.M, self.bins[l], rk, rv, w)
        return out

    def reconstruct(self, key, which):
        l = key[0]
        w = None if self.weights is None else self.weights[l]
        return orc.reconstruct(self.S[key][which], self.T, self.M, self.bins[l], w)


def check_coeffs(cache, ora, tag):
    worst = 0.0
    for l in sorted({k[0] for k in ora.S}):
        SK, SV = cache.export_coeffs(l)
        for (ll, b, h), st in ora.S.items():
            if ll != l:
                continue
            worst = max(worst, rel_l2(c128(SK[b, h]), st[0]), rel_l2(c128(SV[b, h]), st[1]))
    assert worst < TOL_COEF, f"{tag}: coefficient rel-L2 {worst:.3e}"
    return worst


def check_attn(cfg, cache, ora, q, tag):
    out = cache.attend(q)
    ref = ora.attend(q)
    G = cfg.group
    worst = 0.0
    for (l, b, h), r in ref.items():
        worst = max(worst, rel_l2(f64(out[l, b, h * G:(h + 1) * G]), r))
    assert worst < TOL_ATTN[cfg.torch_dtype], f"{tag}: attention rel-L2 {worst:.3e}"
    return worst


def check_reconstruct(cfg, cache, ora, a0, n, tag):
    worst = 0.0
    for l in sorted({k[0] for k in ora.S}):
        Kt, Vt = cache.reconstruct(l, a0, n)
        for key in ora.S:
            if key[0] != l:
                continue
            _, b, h = key
            worst = max(worst, rel_l2(f64(Kt[b, h]), ora.reconstruct(key, 0)[a0:a0 + n]),
                        rel_l2(f64(Vt[b, h]), ora.reconstruct(key, 1)[a0:a0 + n]))
    assert worst < TOL_REC[cfg.torch_dtype], f"{tag}: reconstruction rel-L2 {worst:.3e}"
    return worst


def check_masks(cache, bins):
    for l, b in enumerate(bins):
        got = cache.export_bins(l).cpu().numpy()
        assert got.dtype == np.int32 and np.array_equal(got, np.asarray(b, np.int32)), f"mask of layer {l}"


def run_stream(cfg, bins, weights=None, flags=0, steps=None, slices=None, rec=(0, 64), tag="", fused=False,
               write_every=0):
    steps = cfg.steps if steps is None else steps
    slices = wl.sample_slices(cfg) if slices is None else slices
    K, V = wl.prefill_tensors(cfg, DEV)
    cache = make_cache(cfg, bins, weights, flags, write_every)
    check_masks(cache, bins)
    cache.prefill(K, V)
    assert cache.T == cfg.L
    ora = SliceOracle(cfg, bins, weights, K, V, slices)
    del K, V
    stats = {"coef0": check_coeffs(cache, ora, tag + " prefill")}
    stats["rec0"] = check_reconstruct(cfg, cache, ora, rec[0], rec[1], tag + " prefill")
    worst_attn = 0.0
    for i in range(steps):
        tk, tv, q = wl.decode_step(cfg, i, DEV)
        ora.append(tk, tv)
        if fused:  # one call: append, then attend
            out = cache.step(tk, tv, q)
            ref = ora.attend(q)
            G = cfg.group
            w = max(rel_l2(f64(out[l, b, h * G:(h + 1) * G]), r) for (l, b, h), r in ref.items())
            assert w < TOL_ATTN[cfg.torch_dtype], f"{tag} fused step {i}: attention rel-L2 {w:.3e}"
            worst_attn = max(worst_attn, w)
        else:
            cache.append(tk, tv)
            worst_attn = max(worst_attn, check_attn(cfg, cache, ora, q, f"{tag} step {i}"))
    assert cache.T == cfg.L + steps
    stats["attn"] = worst_attn
    stats["coefN"] = check_coeffs(cache, ora, tag + " after appends")
    stats["recN"] = check_reconstruct(cfg, cache, ora, max(0, cfg.L - rec[1]), min(rec[1], cfg.L), tag + " end")
    torch.cuda.synchronize()
    print(f"\n[{tag}] " + " ".join(f"{k}={v:.2e}" for k, v in stats.items()), flush=True)
    cache.close()
    return stats


def small_cfg(**kw):
    base = dict(name="small", n_layers=2, batch=2, n_kv_heads=2, group=2, head_dim=128, L=256, n_bins=40,
                steps=5, dtype="f32", mask="low", seed=3)
    base.update(kw)
    return wl.Config(**base)


def random_bins(cfg, seed):
    rng = np.random.default_rng(seed)
    return [np.sort(rng.choice(cfg.L, size=cfg.n_bins - (l % 2), replace=False)).astype(np.int32)
            for l in range(cfg.n_layers)]


def test_cfg1_full_stream_fft_path():
    cfg = wl.CONFIGS["cfg1"]
    run_stream(cfg, wl.layer_bins(cfg), tag="cfg1")


def test_cfg1_direct_synthesis_path():
    cfg = wl.CONFIGS["cfg1"]
    run_stream(cfg, wl.layer_bins(cfg), flags=B.IWDFT_FLAG_DIRECT_SYNTHESIS, steps=3, tag="cfg1-direct")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,group", [(256, 2), (1024, 3), (96, 1), (160, 2), (2048, 8)])
def test_ragged_random_masks(dtype, L, group):
    # odd bin counts (ragged rows), scattered bins (folding collisions), batch > 1, odd group size,
    # non-power-of-two M (direct synthesis), wrap-around of the slot shift (steps > 0 with small M);
    # 96 and 160 tokens: a ragged last tile and an odd number of 64-token tiles in the dense prefill
    cfg = small_cfg(L=L, group=group, dtype=dtype, n_bins=min(77, L // 2 + 5))
    run_stream(cfg, random_bins(cfg, 11), rec=(3, 50), tag=f"ragged-{dtype}-L{L}-G{group}")


def test_bin_weights_one_sided():
    cfg = small_cfg(L=512, n_bins=257, group=2)
    bins = [np.arange(257, dtype=np.int32) for _ in range(cfg.n_layers)]
    w = [np.where((b == 0) | (b == 256), 1.0, 2.0).astype(np.float32) for b in bins]
    st = run_stream(cfg, bins, weights=w, steps=2, tag="one-sided")
    # the weights also scale the deferred tokens' rank-one terms: fused steps with write-back every 4th
    run_stream(cfg, bins, weights=w, steps=6, fused=True, write_every=4, tag="one-sided-deferred")
    # with every bin of a real signal represented, reconstruction at T = M is the input itself
    K, V = wl.prefill_tensors(cfg, DEV)
    cache = make_cache(cfg, bins, w)
    cache.prefill(K, V)
    Kt, Vt = cache.reconstruct(1, 0, cfg.L)
    assert rel_l2(f64(Kt), f64(K[1])) < 1e-5 and rel_l2(f64(Vt), f64(V[1])) < 1e-5
    cache.close()


@pytest.mark.parametrize("L", [100, 75])
def test_bin_weights_one_sided_any_length(L):
    # the same one-sided synthesis where M is not a power of two (chirp-z attention, dense prefill, direct
    # reconstruction); odd M has no Nyquist bin
    cfg = small_cfg(L=L, n_bins=L // 2 + 1, group=3)
    bins = [np.arange(L // 2 + 1, dtype=np.int32) for _ in range(cfg.n_layers)]
    w = [np.where((b == 0) | (2 * b == L), 1.0, 2.0).astype(np.float32) for b in bins]
    run_stream(cfg, bins, weights=w, steps=3, rec=(0, 32), tag=f"one-sided-{L}")
    run_stream(cfg, bins, weights=w, steps=3, rec=(0, 32), fused=True, tag=f"one-sided-{L}-fused")
    K, V = wl.prefill_tensors(cfg, DEV)
    cache = make_cache(cfg, bins, w)
    assert B.iwdft_attn_kind(cache.ctx) == "chirp"
    cache.prefill(K, V)
    Kt, Vt = cache.reconstruct(1, 0, cfg.L)
    assert rel_l2(f64(Kt), f64(K[1])) < 1e-5 and rel_l2(f64(Vt), f64(V[1])) < 1e-5
    cache.close()


def test_many_wraps_slot_shift():
    # more appends than M: the shift (T - M) mod M wraps several times
    cfg = small_cfg(L=64, n_bins=20, group=1, steps=150, n_layers=1, batch=1)
    run_stream(cfg, random_bins(cfg, 5), rec=(0, 64), tag="wraps")


def test_call_order_and_argument_errors():
    cfg = small_cfg()
    bins = random_bins(cfg, 1)
    cache = make_cache(cfg, bins)
    tk, tv, q = wl.decode_step(cfg, 0, DEV)
    for fn in (lambda: cache.append(tk, tv), lambda: cache.attend(q), lambda: cache.export_coeffs(0),
               lambda: cache.reconstruct(0, 0, 4)):
        with pytest.raises(B.IwdftError) as e:
            fn()
        assert e.value.code == B.IWDFT_ERR_STATE
    K, V = wl.prefill_tensors(cfg, DEV)
    cache.prefill(K, V)
    for fn, code in ((lambda: cache.reconstruct(5, 0, 4), B.IWDFT_ERR_ARG),
                     (lambda: cache.reconstruct(0, cfg.L - 2, 4), B.IWDFT_ERR_ARG),
                     (lambda: cache.export_coeffs(-1), B.IWDFT_ERR_ARG),
                     (lambda: B.iwdft_set_num_tokens(cache.ctx, cfg.L - 1), B.IWDFT_ERR_ARG)):
        with pytest.raises(B.IwdftError) as e:
            fn()
        assert e.value.code == code
    small = torch.empty(256, dtype=torch.uint8, device=DEV)
    with pytest.raises(B.IwdftError) as e:
        B.iwdft_create(cache.desc, small, cache.workspace)
    assert e.value.code == B.IWDFT_ERR_SIZE
    cache.close()


def test_checkpoint_resume_is_bitwise():
    cfg = small_cfg(steps=6)
    bins = random_bins(cfg, 2)
    K, V = wl.prefill_tensors(cfg, DEV)
    cache = make_cache(cfg, bins)
    cache.prefill(K, V)
    steps = [wl.decode_step(cfg, i, DEV) for i in range(6)]
    for tk, tv, _ in steps[:2]:
        cache.append(tk, tv)
    saved, T = cache.state.clone(), cache.T
    for tk, tv, _ in steps[2:]:
        cache.append(tk, tv)
    a = cache.attend(steps[5][2]).clone()
    end = cache.state.clone()
    cache.state.copy_(saved)
    B.iwdft_set_num_tokens(cache.ctx, T)
    for tk, tv, _ in steps[2:]:
        cache.append(tk, tv)
    assert torch.equal(cache.state, end)
    assert torch.equal(cache.attend(steps[5][2]), a)
    cache.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,S,R,group", [(256, 10, 50, 2), (1024, 3, 1, 3), (96, 4, 7, 1), (512, 0, 5, 4),
                                         (512, 6, 0, 8)])
def test_sink_and_recent_windows(dtype, L, S, R, group):
    # exact sink / recent tokens join the softmax; more appends than R so that the ring wraps and every
    # original recent token and several appended ones have aged into the coefficients
    cfg = small_cfg(L=L, group=group, dtype=dtype, n_bins=41, n_sink=S, n_recent=R, steps=max(6, R + 3) if R < 10 else 7)
    run_stream(cfg, random_bins(cfg, 17), rec=(2, 40), tag=f"windows-{dtype}-L{L}-S{S}-R{R}-G{group}")


def test_windows_all_bins_equals_full_attention_over_the_whole_context():
    # every bin kept, nothing appended beyond the recent hand-over: the assembled cache is the complete
    # context, so the library must reproduce plain softmax attention over all S + M + R tokens
    cfg = small_cfg(L=256, n_bins=256, group=2, dtype="f32", n_sink=5, n_recent=9, n_layers=1, batch=1, steps=0)
    bins = [np.arange(256, dtype=np.int32)]
    K, V = wl.prefill_tensors(cfg, DEV)
    cache = make_cache(cfg, bins)
    cache.prefill(K, V)
    _, _, q = wl.decode_step(cfg, 0, DEV)
    out = cache.attend(q)
    G = cfg.group
    for h in range(cfg.n_kv_heads):
        ref = orc.attention(f64(q[0, 0, h * G:(h + 1) * G]), f64(K[0, 0, h]), f64(V[0, 0, h]))
        assert rel_l2(f64(out[0, 0, h * G:(h + 1) * G]), ref) < 1e-5
    cache.close()


def test_cfg2_with_paper_windows_full_size():
    cfg = wl.CONFIGS["cfg2w"]
    run_stream(cfg, wl.layer_bins(cfg), steps=3, tag="cfg2w")


def test_fused_step_cfg1():
    cfg = wl.CONFIGS["cfg1"]
    run_stream(cfg, wl.layer_bins(cfg), fused=True, tag="cfg1-fused")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,S,R,group", [(256, 0, 0, 2), (1024, 3, 5, 3), (96, 4, 7, 1), (2048, 0, 0, 8),
                                         (512, 2, 3, 16)])
def test_fused_step_ragged_and_windows(dtype, L, S, R, group):
    # the fused call must give what append + attend give; group 16 needs two head passes and takes the
    # unfused sequence inside the library
    cfg = small_cfg(L=L, group=group, dtype=dtype, n_bins=min(77, L // 2 + 5), n_sink=S, n_recent=R, steps=9)
    run_stream(cfg, random_bins(cfg, 23), rec=(3, 50), fused=True, tag=f"fused-{dtype}-L{L}-S{S}-R{R}-G{group}")


def test_fused_step_leaves_the_same_state_as_append():
    cfg = small_cfg(L=512, n_bins=100, group=4, dtype="bf16", n_sink=3, n_recent=4, steps=6)
    bins = random_bins(cfg, 29)
    K, V = wl.prefill_tensors(cfg, DEV)
    a, b = make_cache(cfg, bins), make_cache(cfg, bins)
    a.prefill(K, V)
    b.prefill(K, V)
    for i in range(cfg.steps):
        tk, tv, q = wl.decode_step(cfg, i, DEV)
        a.append(tk, tv)
        oa = a.attend(q)
        ob = b.step(tk, tv, q)
        assert rel_l2(f64(ob), f64(oa)) < 5e-3
    assert a.T == b.T
    for l in range(cfg.n_layers):
        (ka, va), (kb, vb) = a.export_coeffs(l), b.export_coeffs(l)
        assert rel_l2(c128(kb), c128(ka)) < 1e-6 and rel_l2(c128(vb), c128(va)) < 1e-6
    a.close()
    b.close()


def test_phase_timing_marks_calls_without_changing_results():
    cfg = small_cfg(L=1024, n_bins=200, group=4, dtype="bf16", n_sink=2, n_recent=3, steps=4)
    bins = random_bins(cfg, 31)
    K, V = wl.prefill_tensors(cfg, DEV)
    a, b = make_cache(cfg, bins), make_cache(cfg, bins)
    a.prefill(K, V)
    b.prefill(K, V)
    B.iwdft_phase_timing(b.ctx, True)
    for i in range(cfg.steps):
        tk, tv, q = wl.decode_step(cfg, i, DEV)
        oa = a.step(tk, tv, q)
        ob = b.step(tk, tv, q)
        assert torch.equal(oa, ob)
        assert torch.equal(a.attend(q), b.attend(q))
    ms, n = B.iwdft_phase_times(b.ctx)
    assert n == 2 * cfg.steps and all(0.0 < m < 1e3 for m in ms)
    ms, n = B.iwdft_phase_times(b.ctx)       # the read-out cleared the list
    assert n == 0 and ms == [0.0, 0.0, 0.0]
    B.iwdft_phase_timing(b.ctx, False)
    tk, tv, q = wl.decode_step(cfg, 0, DEV)
    b.step(tk, tv, q)
    assert B.iwdft_phase_times(b.ctx)[1] == 0
    a.close()
    b.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,S,R,group,J", [(256, 0, 0, 2, 2), (1024, 3, 5, 3, 8), (512, 0, 4, 1, 3), (2048, 0, 0, 8, 8),
                                           (4096, 2, 0, 4, 5), (16384, 0, 3, 4, 8), (512, 2, 3, 16, 8),
                                           (96, 0, 0, 2, 8), (1024, 2, 3, 4, 16), (8192, 0, 0, 2, 13),
                                           (32768, 0, 2, 4, 16)])
def test_deferred_write_back_stream(dtype, L, S, R, group, J):
    # the coefficients are written back every J-th fused step only; every step's attention still has to
    # match the oracle, and so do the coefficients once the deferred tokens are flushed (19 steps: several
    # write-backs and a partial batch at the end).  group 16 and M = 96 cannot defer and run with J = 1.
    big = L > 8192
    cfg = small_cfg(L=L, group=group, dtype=dtype, n_bins=min(77, L // 2 + 5), n_sink=S, n_recent=R,
                    steps=19 if J <= 8 else 37,
                    n_layers=1 if big else 2)
    run_stream(cfg, random_bins(cfg, 47), rec=(3, 50), fused=True, write_every=J,
               tag=f"defer-{dtype}-L{L}-S{S}-R{R}-G{group}-J{J}")


@pytest.mark.parametrize("L,n_bins", [(16384, 1600), (16384, 3000), (8192, 4096), (32768, 900)])
def test_deferred_write_back_every_fft_kernel_variant(L, n_bins):
    # the pending tokens are weighed in the epilogue of attention kernel B, which exists in several
    # register-budget variants (2, 4 or 8 kept bins per thread, one or many transform blocks): all of
    # them with 16 deferred tokens, windows included
    cfg = small_cfg(L=L, group=4, dtype="bf16", n_bins=n_bins, n_sink=2, n_recent=3, steps=18, n_layers=1, batch=1)
    run_stream(cfg, random_bins(cfg, 79), rec=(3, 50), fused=True, write_every=16, tag=f"defer-variants-L{L}-B{n_bins}")


@pytest.mark.parametrize("group,batch,heads,n_bins,J", [
    (1, 1, 1, 1, 0), (3, 1, 2, 129, 0), (8, 3, 2, 300, 4),                         # few blocks: one lane, a lane beyond 128 bins, three blocks a slice
    (1, 32, 16, 100, 0), (1, 32, 16, 100, 4), (2, 19, 27, 128, 4), (2, 27, 19, 127, 0),  # 512 blocks and 513
    (4, 64, 32, 100, 4), (3, 683, 3, 100, 4), (8, 64, 16, 128, 4), (5, 41, 25, 128, 4),   # 2048 and 2049, 1024 and 1025 (read-only steps)
    (16, 2, 4, 40, 0),                                                              # two passes over the heads
])
def test_score_kernel_of_few_and_of_many_blocks(group, batch, heads, n_bins, J):
    cfg = small_cfg(L=512, n_bins=n_bins, dtype="f32", group=group, batch=batch, n_kv_heads=heads, n_layers=1, steps=5, n_sink=2, n_recent=3)
    run_stream(cfg, random_bins(cfg, 71), fused=group <= 8, write_every=J, rec=(0, 16), tag=f"blocks-{group}-{batch}x{heads}",
               slices=wl.sample_slices(cfg, 5))


@pytest.mark.parametrize("L,group,n_bins,dims,S,R,J,dtype,one", [
    (256, 1, 1, (2, 1, 1), 0, 0, 0, "f32", "aw"), (256, 8, 64, (2, 1, 4), 1, 0, 4, "bf16", "ar"),       # one bin; a full quarter, 16 lanes a transform
    (512, 5, 33, (3, 8, 4), 3, 70, 0, "bf16", "aw"), (512, 2, 128, (2, 1, 4), 0, 9, 16, "f32", "arw"),     # more exact tokens than lanes; a last head pair with one head
    (1024, 4, 65, (2, 2, 3), 0, 0, 16, "bf16", "arw"), (1024, 7, 129, (2, 8, 8), 2, 3, 5, "f32", "arw"),    # 64 and 128 lanes a row
    (2048, 1, 250, (1, 1, 3), 4, 0, 3, "bf16", "ar"), (2048, 8, 512, (2, 10, 8), 0, 2, 2, "bf16", "arw"),   # all lanes two rows of a head group
    (4096, 4, 1023, (1, 20, 8), 2, 5, 4, "bf16", "ar"), (4096, 3, 790, (2, 10, 8), 0, 0, 0, "f32", "aw"),  # one row over all lanes
    (1024, 2, 256, (1, 67, 10), 0, 0, 0, "bf16", "aw"), (512, 4, 120, (40, 8, 8), 1, 2, 8, "bf16", "arw"),  # states beyond 160 MiB
])
def test_short_contexts_in_one_launch(L, group, n_bins, dims, S, R, J, dtype, one):
    """One workgroup per slice (attn_slice.hip) against the oracle and against the three kernels, which IWDFT_FLAG_SERIAL_PHASES
    keeps: masks up to M / 2 without shared slots, ragged rows, layers of different lengths.  `one`: what runs as one launch, attention alone, steps that
    read only and steps that write back.  Same sums in another order: fp32 outputs agree to 1e-5 (scores of magnitude 50 times 2^-23), bf16 to one
    rounding (2^-8 of the largest)."""
    cfg = small_cfg(L=L, group=group, dtype=dtype, n_bins=n_bins, n_layers=dims[0], batch=dims[1], n_kv_heads=dims[2], n_sink=S,
                    n_recent=R, steps=6)
    rng = np.random.default_rng(L + n_bins)
    bins = [np.sort(rng.choice(L // 2 + 1, size=max(1, n_bins - 7 * (l % 3)), replace=False)).astype(np.int32) for l in range(dims[0])]
    bins[0][0] = 0
    run_stream(cfg, bins, fused=True, write_every=J, rec=(0, 16), tag=f"slice-L{L}-G{group}-B{n_bins}")
    K, V = wl.prefill_tensors(cfg, DEV)
    a, b = make_cache(cfg, bins, write_every=J), make_cache(cfg, bins, flags=B.IWDFT_FLAG_SERIAL_PHASES, write_every=J)
    calls = dict(a=(0, False), r=(1, False), w=(max(J, 1), True))
    assert "".join(c for c in calls if (c != "r" or J > 1) and B.iwdft_query_attn(a.desc, *calls[c]) == 0) == one
    assert all(B.iwdft_query_attn(b.desc, *x) == 1 for x in calls.values())
    a.prefill(K, V)
    b.prefill(K, V)
    tol = 1e-5 if dtype == "f32" else 2.0 ** -8
    for i in range(cfg.steps):
        tk, tv, q = wl.decode_step(cfg, i, DEV)
        for x, y in ((a.step(tk, tv, q), b.step(tk, tv, q)),) + (((a.attend(q), b.attend(q)),) if i == 4 else ()):
            assert torch.isfinite(x.float()).all()
            assert float((x.float() - y.float()).abs().max()) <= tol * float(y.float().abs().max()), f"step {i}"
    a.flush()
    b.flush()
    for l in range(dims[0]):
        for x, y in zip(a.export_coeffs(l), b.export_coeffs(l)):
            assert float((x - y).abs().max()) <= 1e-6 * float(y.abs().max())
    a.close()
    b.close()


@pytest.mark.parametrize("J", [0, 16])
@pytest.mark.parametrize("L,n_bins,group", [(256, 64, 1), (512, 128, 2), (1024, 160, 1), (1024, 100, 4), (2048, 150, 2), (4096, 160, 1)])
def test_short_contexts_write_back_as_exactly_as_the_three_kernels(L, n_bins, group, J):
    """Token j is one in channel j and zero elsewhere, the state zero before: the coefficients of that channel are e^{j 2 pi k j / M} as the
    step forms it.  Its distance from 64 bits, over all bins and tokens, is no larger than what the three kernels leave (5 % more for the other grouping
    of the products where 16 tokens are written at once); one token at a time both parts of K are right to an ulp below one, 2^-24."""
    cfg = small_cfg(L=L, group=group, dtype="f32", n_bins=n_bins, n_layers=1, batch=1, n_kv_heads=2)
    bins = [np.sort(np.random.default_rng(L + n_bins).choice(L // 2 + 1, size=n_bins, replace=False)).astype(np.int32)]
    zero = torch.zeros((1, 1, 2, L, 128), device=DEV)
    row = torch.zeros((16, 1, 1, 2, 128), device=DEV)
    for j in range(16):
        row[j, ..., j] = 1.0
    q = torch.zeros((1, 1, 2 * group, 128), device=DEV)
    want = np.exp(2j * np.pi * np.outer(np.arange(16), bins[0]) / L)
    errors = {}
    for flags in (0, B.IWDFT_FLAG_SERIAL_PHASES):
        c = make_cache(cfg, bins, flags=flags, write_every=J)
        assert B.iwdft_query_attn(c.desc, J or 1, True) == (1 if flags else 0)
        c.prefill(zero, zero)
        for j in range(16):
            c.step(row[j], row[j], q)
        padded = -(-n_bins // 32) * 32
        held = c.state[-2 * 2 * 128 * padded * 8:].view(torch.complex64).view(2, 2, 128, padded)  # K then V, slices, channels, bins
        for name, F in zip("KV", held):
            F = c128(F)
            assert (F[:, :, n_bins:] == 0).all() and (F[:, 16:] == 0).all()
            errors[name, flags] = np.abs(F[:, :16, :n_bins] - want)
        c.close()
    if J == 0:
        assert errors["K", 0].max() <= 2.0 ** -24 * 2 ** 0.5
    for name in "KV":
        assert np.linalg.norm(errors[name, 0]) <= 1.05 * np.linalg.norm(errors[name, B.IWDFT_FLAG_SERIAL_PHASES]), name


@pytest.mark.parametrize("L,n_bins,group,dims,S,R,J,dtype,low,parts", [
    (16384, 900, 3, (2, 1, 2), 0, 0, 4, "bf16", False, 2), (16384, 2500, 1, (1, 1, 5), 3, 40, 0, "f32", False, 2),   # two blocks; 2 and 8 bins a thread
    (32768, 1500, 8, (1, 2, 3), 0, 0, 16, "bf16", False, 4), (65536, 3100, 2, (1, 1, 9), 1, 2, 3, "bf16", False, 8),  # fewer parts than blocks
    (16384, 4200, 5, (1, 1, 1), 0, 9, 2, "f32", False, 2),                                                          # sums in the rows themselves
    (65536, 4096, 2, (1, 1, 3), 2, 0, 16, "f32", True, 4), (131072, 4000, 3, (1, 1, 5), 0, 5, 4, "bf16", True, 8),     # low frequencies: grids of 16384,
    (65536, 2048, 4, (1, 2, 2), 0, 0, 8, "bf16", True, 8), (65536, 1000, 1, (2, 1, 3), 0, 0, 0, "bf16", True, 16),      # 8192 and 4096 points
    (2 * 8162, 2000, 3, (1, 1, 2), 10, 50, 16, "bf16", False, 2), (37 * 353, 700, 4, (2, 1, 2), 0, 3, 0, "f32", False, 37),  # chirp-z blocks
    (11 * 33 * 32, 300, 2, (1, 1, 3), 0, 0, 4, "bf16", False, 2),
])
def test_softmax_of_few_slices_shared_between_workgroups(L, n_bins, group, dims, S, R, J, dtype, low, parts):
    """attn_parts.hip against the oracle and against one workgroup per pair of heads, which IWDFT_FLAG_SERIAL_PHASES keeps: the same sums in
    another order (tolerances as in test_short_contexts_in_one_launch)."""
    cfg = small_cfg(L=L, group=group, dtype=dtype, n_bins=n_bins, n_layers=dims[0], batch=dims[1], n_kv_heads=dims[2], n_sink=S,
                    n_recent=R, steps=6)
    rng = np.random.default_rng(L + n_bins)
    top = n_bins if low else L // 2 + 1
    bins = [np.sort(rng.choice(top, size=n_bins - 7 * (l % 3), replace=False)).astype(np.int32) for l in range(dims[0])]
    bins[0][0] = 0
    if not low:
        bins[0][-1] = L // 2  # no grid of low frequencies
    run_stream(cfg, bins, fused=True, write_every=J, steps=3, slices=wl.sample_slices(cfg, 2), rec=(0, 4), tag=f"parts-L{L}-G{group}")
    K, V = wl.prefill_tensors(cfg, DEV)
    a, b = make_cache(cfg, bins, write_every=J), make_cache(cfg, bins, flags=B.IWDFT_FLAG_SERIAL_PHASES, write_every=J)
    assert B.iwdft_query_attn(a.desc) == parts and a.ws_bytes > b.ws_bytes and B.iwdft_query_attn(b.desc) == 1
    a.prefill(K, V)
    b.prefill(K, V)
    tol = 1e-5 if dtype == "f32" else 2.0 ** -8
    for i in range(cfg.steps):
        tk, tv, q = wl.decode_step(cfg, i, DEV)
        for x, y in ((a.step(tk, tv, q), b.step(tk, tv, q)),) + (((a.attend(q), b.attend(q)),) if i == 4 else ()):
            assert torch.isfinite(x.float()).all()
            assert float((x.float() - y.float()).abs().max()) <= tol * float(y.float().abs().max()), f"step {i}"
    a.close()
    b.close()


def test_deferred_write_back_mixed_with_other_calls():
    # any call other than the fused step first writes the deferred tokens back: a random mix of calls
    # gives, step for step, what the oracle gives
    cfg = small_cfg(L=1024, n_bins=150, group=4, dtype="bf16", n_sink=2, n_recent=3, steps=40, n_layers=1)
    bins = random_bins(cfg, 53)
    K, V = wl.prefill_tensors(cfg, DEV)
    cache = make_cache(cfg, bins, write_every=8)
    cache.prefill(K, V)
    slices = wl.sample_slices(cfg, 4)
    ora = SliceOracle(cfg, bins, None, K, V, slices)
    rng = np.random.default_rng(5)
    G = cfg.group
    for i in range(cfg.steps):
        tk, tv, q = wl.decode_step(cfg, i, DEV)
        ora.append(tk, tv)
        op = rng.integers(0, 5)
        if op <= 2:
            out = cache.step(tk, tv, q)
            ref = ora.attend(q)
            w = max(rel_l2(f64(out[l, b, h * G:(h + 1) * G]), r) for (l, b, h), r in ref.items())
            assert w < TOL_ATTN[cfg.torch_dtype], f"mixed step {i}: {w:.3e}"
        else:
            cache.append(tk, tv)
            check_attn(cfg, cache, ora, q, f"mixed append/attend {i}")
        if op == 1:
            check_attn(cfg, cache, ora, q, f"mixed attend after step {i}")      # same state, plain attention
        if op == 2 and i % 3 == 0:
            check_coeffs(cache, ora, f"mixed export {i}")
        if op == 0 and i % 4 == 0:
            check_reconstruct(cfg, cache, ora, 7, 40, f"mixed reconstruct {i}")
        assert cache.T == cfg.L + i + 1
    check_coeffs(cache, ora, "mixed end")
    cache.close()


def test_deferred_write_back_equals_immediate_and_checkpoints_after_flush():
    cfg = small_cfg(L=512, n_bins=100, group=4, dtype="bf16", n_sink=3, n_recent=4, steps=13)
    bins = random_bins(cfg, 59)
    K, V = wl.prefill_tensors(cfg, DEV)
    a, b = make_cache(cfg, bins), make_cache(cfg, bins, write_every=8)
    a.prefill(K, V)
    b.prefill(K, V)
    steps = [wl.decode_step(cfg, i, DEV) for i in range(cfg.steps)]
    for tk, tv, q in steps[:11]:                      # 11 steps: one write-back, three tokens deferred
        oa, ob = a.step(tk, tv, q), b.step(tk, tv, q)
        assert rel_l2(f64(ob), f64(oa)) < 5e-3
    b.flush()
    for l in range(cfg.n_layers):
        (ka, va), (kb, vb) = a.export_coeffs(l), b.export_coeffs(l)
        assert rel_l2(c128(kb), c128(ka)) < 1e-6 and rel_l2(c128(vb), c128(va)) < 1e-6
    saved, T = b.state.clone(), b.T                   # complete after the flush
    tail = [b.step(tk, tv, q).clone() for tk, tv, q in steps[11:]]
    b.state.copy_(saved)
    B.iwdft_set_num_tokens(b.ctx, T)
    again = [b.step(tk, tv, q).clone() for tk, tv, q in steps[11:]]
    assert all(torch.equal(x, y) for x, y in zip(tail, again))
    a.close()
    b.close()


@pytest.mark.parametrize("prefill", ["fft", "dense"])
def test_two_runs_are_bitwise_identical(prefill):
    # no kernel uses atomics or data-dependent orders: the same calls on the same inputs leave the same
    # bytes in the state buffer and return the same outputs (whole-buffer comparison, all slices)
    cfg = small_cfg(L=2048, n_bins=333, group=4, dtype="bf16", n_sink=2, n_recent=5, steps=11, n_layers=3, batch=2)
    bins = random_bins(cfg, 67)
    flags = B.IWDFT_FLAG_FFT_PREFILL if prefill == "fft" else B.IWDFT_FLAG_DENSE_PREFILL
    K, V = wl.prefill_tensors(cfg, DEV)
    states, outs = [], []
    for run in range(2):
        c = make_cache(cfg, bins, flags=flags, write_every=4)
        c.prefill(K, V)
        o = []
        for i in range(cfg.steps):
            tk, tv, q = wl.decode_step(cfg, i, DEV)
            if i % 5 == 3:
                c.append(tk, tv)
                o.append(c.attend(q).clone())
            else:
                o.append(c.step(tk, tv, q).clone())
        c.flush()
        torch.cuda.synchronize()
        states.append(c.state.clone())
        outs.append(o)
        c.close()
    assert torch.equal(states[0], states[1])
    assert all(torch.equal(a, b) for a, b in zip(outs[0], outs[1]))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,S,R,group,steps", [(256, 0, 0, 2, 64), (1024, 3, 5, 4, 9), (96, 0, 2, 1, 200)])
def test_shortcut_flag_matches_the_oracle_recursion(dtype, L, S, R, group, steps):
    """IWDFT_FLAG_SHORTCUT: Sec. 4.1's update with (N-1)/N taken as 1, inside the library (the token's scale
    M / (T+1) is applied by the append kernel, the gain T/M by every reader).  Exported coefficients against the
    oracle's shortcut recursion and its closed form, attention and reconstruction against the oracle run on that
    state; both the two calls and iwdft_append_attn (which must fall back to them)."""
    cfg = small_cfg(L=L, n_bins=min(40, L // 2), group=group, dtype=dtype, steps=steps, n_layers=2, batch=1, n_sink=S,
                    n_recent=R)
    bins = random_bins(cfg, 71)
    K, V = wl.prefill_tensors(cfg, DEV)
    cache = B.Cache(cfg.n_layers, cfg.batch, cfg.n_kv_heads, cfg.n_q_heads, cfg.head_dim, cfg.torch_dtype, cfg.L,
                    bins, None, B.IWDFT_FLAG_SHORTCUT, DEV, n_sink=S, n_recent=R, write_every=8)
    cache.prefill(K, V)
    key = (1, 0, 1)
    l = key[0]
    k0, v0 = f64(K[key]), f64(V[key])
    SK, SV, T = orc.prefill(k0[S:S + L], bins[l]), orc.prefill(v0[S:S + L], bins[l]), L
    sink = (k0[:S], v0[:S])
    rk, rv = [r for r in k0[S + L:]], [r for r in v0[S + L:]]
    absorbed = [k0[S:S + L]]
    worst = 0.0
    G = cfg.group
    for i in range(cfg.steps):
        tk, tv, q = wl.decode_step(cfg, i, DEV)
        if i % 3 == 2:
            out = cache.step(tk, tv, q)
        else:
            cache.append(tk, tv)
            out = cache.attend(q)
        rk.append(f64(tk[key]))
        rv.append(f64(tv[key]))
        xk, xv = rk.pop(0), rv.pop(0)
        SK, SV = orc.append_shortcut(SK, xk, T, bins[l], L), orc.append_shortcut(SV, xv, T, bins[l], L)
        absorbed.append(xk[None, :])
        T += 1
        ref = orc.windowed_attention(f64(q[l, 0, G:2 * G]), sink[0], sink[1], SK, SV, T, L, bins[l],
                                     np.stack(rk) if rk else np.zeros((0, 128)), np.stack(rv) if rv else np.zeros((0, 128)))
        worst = max(worst, rel_l2(f64(out[l, 0, G:2 * G]), ref))
    assert worst < TOL_ATTN[cfg.torch_dtype], f"shortcut attention rel-L2 {worst:.3e}"
    assert cache.T == T
    gk, gv = cache.export_coeffs(l)
    e_rec = max(rel_l2(c128(gk[0, 1]), SK), rel_l2(c128(gv[0, 1]), SV))
    e_closed = rel_l2(c128(gk[0, 1]), orc.closed_form_shortcut(np.vstack(absorbed), L, bins[l]))
    assert e_rec < TOL_COEF and e_closed < TOL_COEF, f"shortcut coefficients {e_rec:.2e} / {e_closed:.2e}"
    Kt, Vt = cache.reconstruct(l, 0, L)
    e_k = rel_l2(f64(Kt[0, 1]), orc.reconstruct(SK, T, L, bins[l]))
    e_v = rel_l2(f64(Vt[0, 1]), orc.reconstruct(SV, T, L, bins[l]))
    assert max(e_k, e_v) < TOL_REC[cfg.torch_dtype]
    drift = rel_l2(SK, orc.closed_form(np.vstack(absorbed), L, bins[l]))
    print(f"\n[shortcut {dtype} M={L}] coefficients {e_rec:.2e} attention {worst:.2e} reconstruction {max(e_k, e_v):.2e}; "
          f"drift of the shortcut from the exact rule after {steps} appends: {drift:.2e}", flush=True)
    cache.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,n_bins,steps,grid", [(256, 100, 7, (3, 4, 60)), (1000, 77, 3, (0, 7, 143)), (4096, 300, 2, (5, 64, 64)),
                                                 (8192, 600, 9, (8191, 1, 1)), (96, 96, 100, (1, 5, 19))])
def test_reconstruct_on_a_strided_grid(dtype, L, n_bins, steps, grid):
    """iwdft_reconstruct_grid against the oracle's strided reconstruction (slots a0 + j * stride)."""
    cfg = small_cfg(L=L, n_bins=n_bins, group=1, dtype=dtype, steps=steps, n_layers=2, batch=2)
    bins = random_bins(cfg, 73)
    K, V = wl.prefill_tensors(cfg, DEV)
    cache = make_cache(cfg, bins)
    cache.prefill(K, V)
    slices = [(0, 0, 0), (1, 1, 1)]
    ora = SliceOracle(cfg, bins, None, K, V, slices)
    for i in range(steps):
        tk, tv, _ = wl.decode_step(cfg, i, DEV)
        cache.append(tk, tv)
        ora.append(tk, tv)
    a0, stride, n = grid
    worst = 0.0
    for (l, b, h) in slices:
        Kt, Vt = cache.reconstruct(l, a0, n, stride=stride)
        for which, got in ((0, Kt), (1, Vt)):
            ref = orc.reconstruct_grid(ora.S[(l, b, h)][which], ora.T, L, bins[l], a0, stride, n)
            worst = max(worst, rel_l2(f64(got[b, h]), ref))
    assert worst < TOL_REC[cfg.torch_dtype], f"grid reconstruction rel-L2 {worst:.3e}"
    with pytest.raises(B.IwdftError):
        cache.reconstruct(0, a0, n + 1 + (L - 1 - a0 - (n - 1) * stride) // stride, stride=stride)   # one row past M
    with pytest.raises(B.IwdftError):
        B.iwdft_reconstruct_grid(cache.ctx, 0, 0, 0, 1, None, None)
    cache.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,n_bins,steps", [(256, 100, 7), (512, 77, 3), (1024, 300, 1030), (2048, 77, 5), (4096, 1500, 2),
                                            (8192, 600, 9), (16384, 900, 4), (32768, 2100, 3)])
def test_reconstruct_long_ranges_through_ffts(dtype, L, n_bins, steps):
    # long slot ranges take the inverse-FFT kernel (all transform lengths, the decimated form beyond 8192,
    # a non-zero slot shift after appends, wrap-around of the shift); ranges: everything, an offset half,
    # and a short one that stays with the direct contraction -- all against the oracle
    big = L > 8192
    cfg = small_cfg(L=L, dtype=dtype, n_bins=n_bins, steps=steps, group=1, n_layers=1 if big else 2,
                    batch=1 if big else 2)
    bins = random_bins(cfg, 73)
    w = [np.random.default_rng(l).uniform(0.5, 2.0, size=len(b)).astype(np.float32) for l, b in enumerate(bins)]
    K, V = wl.prefill_tensors(cfg, DEV)
    cache = make_cache(cfg, bins, w)
    cache.prefill(K, V)
    ora = SliceOracle(cfg, bins, w, K, V, wl.sample_slices(cfg, 4))
    for i in range(steps):
        tk, tv, _ = wl.decode_step(cfg, i % 32, DEV)
        cache.append(tk, tv)
        ora.append(tk, tv)
    for a0, n in [(0, L), (L // 4 + 3, L // 2), (5, 16)]:
        check_reconstruct(cfg, cache, ora, a0, n, f"rec-fft-{dtype}-L{L} [{a0}, {a0 + n})")
    # and the same numbers as the direct contraction (forced by the flag) to a few ulps of the output
    direct = make_cache(cfg, bins, w, flags=B.IWDFT_FLAG_DIRECT_SYNTHESIS)
    direct.prefill(K, V)
    for i in range(steps):
        tk, tv, _ = wl.decode_step(cfg, i % 32, DEV)
        direct.append(tk, tv)
    Ka, Va = cache.reconstruct(0, 0, L)
    Kb, Vb = direct.reconstruct(0, 0, L)
    assert rel_l2(f64(Ka), f64(Kb)) < TOL_REC[cfg.torch_dtype] and rel_l2(f64(Va), f64(Vb)) < TOL_REC[cfg.torch_dtype]
    cache.close()
    direct.close()


def test_deferred_write_back_many_wraps():
    # more steps than M: the slot shifts of the deferred tokens wrap around inside a batch
    cfg = small_cfg(L=256, n_bins=60, group=2, steps=530, n_layers=1, batch=1, dtype="f32")
    run_stream(cfg, random_bins(cfg, 61), fused=True, write_every=8, tag="defer-wraps")


def test_fused_step_cfg2_windows_full_size():
    cfg = wl.CONFIGS["cfg2w"]
    run_stream(cfg, wl.layer_bins(cfg), steps=3, fused=True, tag="cfg2w-fused")


@pytest.mark.parametrize("prefill,fused,J,steps", [("fft", True, 16, 18), ("fft", True, 8, 10), ("fft", True, 1, 3),
                                                   ("fft", False, 0, 3),
                                                   ("dense", False, 0, 3)])
def test_cfg2_full_size_sampled_slices(prefill, fused, J, steps):
    # ("fft", True, 16) is the launch configuration the benchmark times: FFT prefill, fused decode step,
    # coefficients written back every 16th step (18 steps: one write-back, two tokens left deferred)
    cfg = wl.CONFIGS["cfg2"]
    flags = B.IWDFT_FLAG_FFT_PREFILL if prefill == "fft" else B.IWDFT_FLAG_DENSE_PREFILL
    run_stream(cfg, wl.layer_bins(cfg), flags=flags, steps=steps, fused=fused, write_every=J,
               tag=f"cfg2-{prefill}-fused{int(fused)}-J{J}")


@pytest.mark.parametrize("L,n_bins", [(1, 1), (2, 1), (2, 2), (3, 2), (64, 1), (64, 64)])
def test_degenerate_sizes(L, n_bins):
    # one-token caches, a single kept bin, every bin kept; alternating two-call / fused steps
    cfg = small_cfg(L=L, n_bins=n_bins, group=2, steps=4, n_layers=1, batch=2)
    bins = [np.arange(n_bins, dtype=np.int32)]
    for fused in (False, True):
        run_stream(cfg, bins, rec=(0, L), fused=fused, tag=f"degenerate-L{L}-B{n_bins}-f{int(fused)}")


def test_dc_only_mask_outputs_the_mean_value_row():
    # |B| = {0}: every reconstructed slot is the same vector, so attention returns exactly the
    # reconstructed V row whatever the query: (1/M) * sum of all tokens seen
    cfg = small_cfg(L=1024, n_bins=1, group=2, steps=3, n_layers=1, batch=1, dtype="f32")
    bins = [np.zeros(1, np.int32)]
    K, V = wl.prefill_tensors(cfg, DEV)
    cache = make_cache(cfg, bins)
    cache.prefill(K, V)
    tot = f64(V[0, 0]).sum(axis=1)                    # [kv heads, d]
    for i in range(cfg.steps):
        tk, tv, q = wl.decode_step(cfg, i, DEV)
        out = cache.step(tk, tv, q)
        tot = tot + f64(tv[0, 0])
        ref = np.repeat(tot / cfg.L, cfg.group, axis=0)
        assert rel_l2(f64(out[0, 0]), ref) < 1e-5
    cache.close()


@pytest.mark.parametrize("L,n_bins,group,dtype,S,R", [
    (8192, 4096, 2, "bf16", 0, 0),     # the most bins the register-resident kernels take
    (8192, 4100, 2, "bf16", 0, 0),     # one step beyond: the bin-strided kernels, single transform
    (8192, 8192, 3, "f32", 2, 6),      # every bin kept; a last head pair with one head; windows
    (16384, 5000, 4, "bf16", 0, 0),    # two decimated blocks, running sums kept in the output rows
    (32768, 9000, 2, "f32", 4, 4),     # four blocks, fp32 tokens, windows
    (32768, 16384, 1, "bf16", 0, 0),   # half of all bins (mirror-closed sets collide in every slot), one query head
])
def test_more_than_4096_kept_bins_per_layer(L, n_bins, group, dtype, S, R):
    """Up to 4096 kept bins per layer the FFT kernels hold per-bin values in registers; beyond that the prefill and the
    decode attention walk the bin list in strides of the workgroup (and keep running sums in their output rows), still
    O(M log M).  Every step against the oracle, two calls and fused; the deferred write-back is taken as 1 there."""
    cfg = small_cfg(L=L, n_bins=n_bins, group=group, steps=3, n_layers=1, batch=1, n_kv_heads=2, dtype=dtype,
                    n_sink=S, n_recent=R)
    bins = [np.sort(np.random.default_rng(3).choice(cfg.L, size=n_bins, replace=False)).astype(np.int32)]
    cache = make_cache(cfg, bins, write_every=8)
    assert B.iwdft_prefill_kind(cache.ctx) == "fft" and B.iwdft_attn_kind(cache.ctx) == "fft"
    cache.close()
    run_stream(cfg, bins, rec=(5, 40), tag=f"bins-{L}-{n_bins}")
    run_stream(cfg, bins, rec=(5, 40), fused=True, write_every=8, tag=f"bins-{L}-{n_bins}-fused")
    if n_bins > 4096:   # and against the direct sums of the same library
        K, V = wl.prefill_tensors(cfg, DEV)
        a, d = make_cache(cfg, bins), make_cache(cfg, bins, flags=B.IWDFT_FLAG_DIRECT_SYNTHESIS | B.IWDFT_FLAG_DENSE_PREFILL)
        assert B.iwdft_attn_kind(d.ctx) == "direct" and B.iwdft_prefill_kind(d.ctx) == "dense"
        a.prefill(K, V)
        d.prefill(K, V)
        (ka, va), (kd, vd) = a.export_coeffs(0), d.export_coeffs(0)
        assert rel_l2(c128(ka), c128(kd)) < 2e-5 and rel_l2(c128(va), c128(vd)) < 2e-5
        _, _, q = wl.decode_step(cfg, 0, DEV)
        assert rel_l2(f64(a.attend(q)), f64(d.attend(q))) < (2e-5 if dtype == "f32" else 8e-3)
        a.close()
        d.close()


@pytest.mark.parametrize("L,dtype", [(16384, "f32"), (32768, "f32"), (32768, "bf16"), (131072, "bf16")])
def test_prefill_of_layers_with_few_and_with_more_than_4096_bins(L, dtype):
    """Beyond 8192 tokens and 4096 bins the prefill either keeps its sums in the output rows or runs 4096 bins a launch, where
    layers with fewer have nothing left to do: both sides of the rule, layer by layer against the oracle (2^-24 times ~log2 of the
    points and the sums over the residues: 2e-6), and bit for bit on tensors that are 8 bytes off alignment."""
    rng = np.random.default_rng(L)
    counts = [100, 4097, 4096, 8200, 33]
    bins = [np.sort(rng.choice(L, size=n, replace=False)).astype(np.int32) for n in counts]
    cfg = small_cfg(L=L, n_bins=100, dtype=dtype, n_layers=5, batch=1, n_kv_heads=1, group=1)
    K, V = wl.prefill_tensors(cfg, DEV)
    flat = torch.empty(2 * K.numel() + 32, dtype=K.dtype, device=DEV)
    off = 8 // K.element_size()
    Ku, Vu = flat[off:off + K.numel()].view(K.shape), flat[2 * off + K.numel():2 * off + 2 * K.numel()].view(K.shape)
    Ku.copy_(K)
    Vu.copy_(V)
    a, u = make_cache(cfg, bins), make_cache(cfg, bins)
    assert B.iwdft_prefill_kind(a.ctx) == "fft"
    a.prefill(K, V)
    u.prefill(Ku, Vu)
    for layer in range(5):
        (ka, va), (ku, vu) = a.export_coeffs(layer), u.export_coeffs(layer)
        assert torch.equal(ka, ku) and torch.equal(va, vu)
        for X, got in ((K, ka), (V, va)):
            assert rel_l2(c128(got[0, 0]), orc.prefill(f64(X[layer, 0, 0]), bins[layer])) < 2e-6, (layer, counts[layer])
    a.close()
    u.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,S,R,group,n_bins", [(33, 0, 0, 1, 9), (100, 2, 3, 2, 100), (129, 0, 0, 3, 40), (1000, 10, 50, 4, 250),
                                                (2049, 0, 4, 2, 300), (3000, 0, 0, 8, 1500), (8191, 1, 1, 1, 700)])
def test_any_length_attention_through_chirp_transforms(dtype, L, S, R, group, n_bins):
    """M that is not a power of two (M = context - sink - recent in general): the attention runs O(M log M)
    chirp-z transforms, all convolution lengths; every step against the oracle (two calls and the fused step,
    deferred with one and two heads), and against the direct synthesis of the same library."""
    cfg = small_cfg(L=L, n_bins=n_bins, group=group, dtype=dtype, steps=4, n_layers=2, batch=1, n_sink=S, n_recent=R)
    bins = random_bins(cfg, 83)
    c = make_cache(cfg, bins, write_every=8)
    assert B.iwdft_attn_kind(c.ctx) == "chirp"
    c.close()
    run_stream(cfg, bins, tag=f"chirp-{L}", write_every=8, rec=(0, min(64, L)))
    run_stream(cfg, bins, tag=f"chirp-{L}-fused", fused=True, write_every=8, rec=(0, min(64, L)))
    K, V = wl.prefill_tensors(cfg, DEV)
    a, d = make_cache(cfg, bins), make_cache(cfg, bins, flags=B.IWDFT_FLAG_DIRECT_SYNTHESIS)
    assert B.iwdft_attn_kind(d.ctx) == "direct"
    a.prefill(K, V)
    d.prefill(K, V)
    _, _, q = wl.decode_step(cfg, 0, DEV)
    assert rel_l2(f64(a.attend(q)), f64(d.attend(q))) < (2e-5 if dtype == "f32" else 8e-3)
    a.close()
    d.close()


@pytest.mark.parametrize("L,S,R,group,n_bins,J,heads", [
    (255, 0, 0, 2, 60, 4, 2),       # below 256 slots every step writes back
    (256 + 1, 0, 3, 1, 90, 4, 2),   # 513 -> 1024 points
    (500, 10, 50, 4, 120, 8, 192), (513, 0, 0, 3, 300, 16, 77), (1025, 1, 0, 8, 200, 4, 110), (2048 - 1, 0, 2, 2, 500, 8, 2),
    (4096 + 1, 0, 0, 1, 1000, 8, 2), (2 * 4099, 10, 50, 5, 2000, 4, 13), (3 * 8191, 0, 1, 2, 4500, 4, 2),
])
def test_chirp_attention_defers_the_write_back(L, S, R, group, n_bins, J, heads):
    """Both sides of every convolution length (2 M - 1 against 2^m), one block and several, more bins than 4096, an odd
    number of heads (with more than two, enough slices to defer): fused steps across two write-backs against the oracle, and with
    every step written back."""
    cfg = small_cfg(L=L, n_bins=n_bins, group=group, dtype="f32", steps=J + 3, n_layers=2, batch=1, n_sink=S, n_recent=R,
                    n_kv_heads=heads)
    bins = random_bins(cfg, 57)
    run_stream(cfg, bins, rec=(0, min(64, L)), fused=True, write_every=J, slices=wl.sample_slices(cfg, 4), tag=f"chirp-defer-{L}")
    K, V = wl.prefill_tensors(cfg, DEV)
    a, d = make_cache(cfg, bins, write_every=J), make_cache(cfg, bins)
    assert B.iwdft_attn_kind(a.ctx) == "chirp" and a.ws_bytes - d.ws_bytes >= (L > 255) * 2 * heads * (J - 1) * 128 * 4
    a.prefill(K, V)
    d.prefill(K, V)
    for i in range(J + 3):
        k, v, q = wl.decode_step(cfg, i, DEV)
        assert rel_l2(f64(a.step(k, v, q)), f64(d.step(k, v, q))) < 2e-5
    for layer in range(2):
        for x, y in zip(a.export_coeffs(layer), d.export_coeffs(layer)):
            assert rel_l2(c128(x), c128(y)) < 2e-6
    a.close()
    d.close()


@pytest.mark.parametrize("L,n_bins,heads,low", [(1000, 250, 260, False), (8132, 2033, 32, False), (3 * 8191, 4100, 16, False), (3000, 700, 96, True),
                                                (8132, 2033, 32, True)])
def test_chirp_attention_weighs_pending_tokens_as_exactly_as_absorbed_ones(L, n_bins, heads, low):
    """V is zero but for the pending tokens, whose rows are unit vectors: the output holds their weights, one per channel.
    Bins from the whole circle (high ones turn fastest) or the low ones (interpolated transforms) and no constant term, which would hide the
    others.  On top of what the step that writes every token back shows: up to 15 rotations, 2 roundings of 2^-24 each, adding up at random:
    sqrt(30) 2^-24 = 3.3e-7 at the last tokens (mean over the last four steps), half of it and a fluctuation in the mean over all steps:
    2e-7.  The worst output is where the roundings of the scores, 2^-24 of |score| <= 32 in either form, differ most: 2e-6 of a weight."""
    cfg = small_cfg(L=L, n_bins=n_bins, group=2, dtype="f32", steps=15, n_layers=1, batch=1, n_kv_heads=heads)
    bins = [np.sort(np.random.default_rng(5).choice(np.arange(L // 2, L), size=n_bins, replace=False)).astype(np.int32)]
    if low:
        bins = [np.arange(1, n_bins + 1, dtype=np.int32)]
    K, V = wl.prefill_tensors(cfg, DEV)
    V.zero_()
    a, d = make_cache(cfg, bins, write_every=16), make_cache(cfg, bins)
    assert B.iwdft_attn_kind(a.ctx) == "chirp" and a.ws_bytes > d.ws_bytes
    a.prefill(K, V)
    d.prefill(K, V)
    slices = [(0, 0, h) for h in range(0, heads, heads // 8)]
    ora = SliceOracle(cfg, bins, None, K, V, slices)
    err = {"deferred": [], "written": []}
    for i in range(cfg.steps):
        tk, tv, q = wl.decode_step(cfg, i, DEV)
        tv = torch.zeros_like(tv)
        tv[..., i] = 1.0
        ora.append(tk, tv)
        ref = ora.attend(q)
        for name, c in (("deferred", a), ("written", d)):
            out = c.step(tk, tv, q)
            err[name].append([rel_l2(f64(out[l, b, 2 * h:2 * h + 2]), r) for (l, b, h), r in ref.items()])
    x, y = (np.array(err[n]) for n in ("deferred", "written"))
    print(f"\n[pending-{L}-{low}] deferred {x.mean():.2e} {x[-4:].mean():.2e} {x.max():.2e} written {y.mean():.2e} {y[-4:].mean():.2e} {y.max():.2e}", flush=True)
    assert x.mean() < y.mean() + 2e-7 and x[-4:].mean() < y[-4:].mean() + 3.3e-7 and x.max() < y.max() + 2e-6
    a.close()
    d.close()


@pytest.mark.parametrize("L,S,R,group,n_bins,heads", [
    (3000, 10, 50, 4, 700, 36), (3000, 0, 3, 2, 700, 3), (8132, 10, 50, 4, 2033, 13), (8132, 3, 0, 3, 2000, 13), (5000, 2, 7, 8, 1000, 25),
    (16384, 10, 50, 4, 1000, 3), (16384, 1, 2, 3, 256, 2), (65536, 3, 40, 2, 1000, 2), (65536, 10, 50, 4, 4000, 1), (131072, 0, 5, 8, 4096, 1),
])
def test_attention_on_a_grid_with_windows_defers_the_write_back(L, S, R, group, n_bins, heads):
    """Low bins, softmax on the interpolated grid (test_abi.py has the rule): exact tokens, pending tokens and grid in one softmax, fused
    steps across two write-backs against the oracle, and with every step written back."""
    J = 8
    cfg = small_cfg(L=L, n_bins=n_bins, group=group, dtype="f32", steps=J + 3, n_layers=2, batch=1, n_sink=S, n_recent=R, n_kv_heads=heads)
    bins = [np.arange(n_bins - l, dtype=np.int32) for l in range(2)]
    run_stream(cfg, bins, rec=(0, 64), fused=True, write_every=J, slices=wl.sample_slices(cfg, 4), tag=f"grid-defer-{L}")
    K, V = wl.prefill_tensors(cfg, DEV)
    a, d = make_cache(cfg, bins, write_every=J), make_cache(cfg, bins)
    assert a.ws_bytes > d.ws_bytes or L >= 16384
    a.prefill(K, V)
    d.prefill(K, V)
    for i in range(J + 3):
        k, v, q = wl.decode_step(cfg, i, DEV)
        assert rel_l2(f64(a.step(k, v, q)), f64(d.step(k, v, q))) < 2e-5
    a.close()
    d.close()


@pytest.mark.parametrize("flags", [0, B.IWDFT_FLAG_SHORTCUT])
@pytest.mark.parametrize("L,n_bins", [(3000, 300), (8132, 200), (16384, 256)])
def test_attention_on_a_grid_takes_bin_weights_and_the_shortcut(L, n_bins, flags):
    """One-sided weights and the update with (N-1)/N taken as 1, whose gain every reader of the coefficients applies: the grid against the
    direct sums of the same library, after five tokens.  Both are fp32 sums of scores below 8: 1e-5."""
    cfg = small_cfg(L=L, n_bins=n_bins, group=3, n_sink=2, n_recent=3, n_layers=1)
    bins = [np.arange(n_bins, dtype=np.int32)]
    w = [np.where(bins[0] > 0, 2.0, 1.0) * np.random.default_rng(L).uniform(0.5, 1.5, n_bins)]
    K, V = wl.prefill_tensors(cfg, DEV)
    a, d = make_cache(cfg, bins, w, flags), make_cache(cfg, bins, w, flags | B.IWDFT_FLAG_DIRECT_SYNTHESIS)
    assert B.iwdft_attn_kind(a.ctx) != "direct" and B.iwdft_attn_kind(d.ctx) == "direct"
    for c in (a, d):
        c.prefill(K, V)
    for i in range(5):
        k, v, q = wl.decode_step(cfg, i, DEV)
        x, y = (f64(c.step(k, v, q)) for c in (a, d))
        assert rel_l2(x, y) < 1e-5, i
    a.close()
    d.close()


@pytest.mark.parametrize("L,S,R,group,n_bins,dtype", [
    (16324, 10, 50, 4, 1600, "bf16"),    # 16384 - 60 = 2 * 8162: the paper's windows cut out of a 16K context
    (32708, 10, 50, 2, 3000, "f32"),     # 32768 - 60 = 4 * 8177
    (24570, 0, 0, 3, 5000, "bf16"),      # 3 * 8190, more than 4096 bins, a last head pair with one head
    (8198, 0, 3, 1, 700, "f32"),         # 2 * 4099 (a prime block length), one query head
])
def test_long_contexts_that_are_not_a_power_of_two_through_decimated_chirp_transforms(L, S, R, group, n_bins, dtype):
    """M > 8192 that is not a power of two: Pb = M / Q decimated blocks of Q <= 8192 points, each through the chirp-z
    transforms, softmax online across the blocks.  Every step against the oracle (two calls and fused), and against the
    direct sums of the same library."""
    cfg = small_cfg(L=L, n_bins=n_bins, group=group, dtype=dtype, steps=3, n_layers=1, batch=1, n_sink=S, n_recent=R)
    bins = random_bins(cfg, 29)
    c = make_cache(cfg, bins)
    assert B.iwdft_attn_kind(c.ctx) == "chirp"
    c.close()
    run_stream(cfg, bins, tag=f"chirp-{L}", rec=(0, 64))
    run_stream(cfg, bins, tag=f"chirp-{L}-fused", fused=True, rec=(0, 64))
    K, V = wl.prefill_tensors(cfg, DEV)
    a, d = make_cache(cfg, bins), make_cache(cfg, bins, flags=B.IWDFT_FLAG_DIRECT_SYNTHESIS)
    a.prefill(K, V)
    d.prefill(K, V)
    _, _, q = wl.decode_step(cfg, 0, DEV)
    assert rel_l2(f64(a.attend(q)), f64(d.attend(q))) < (2e-5 if dtype == "f32" else 8e-3)
    a.close()
    d.close()


def test_long_prime_context_takes_the_direct_sums():
    cfg = small_cfg(L=10007, n_bins=300, group=2, dtype="f32", steps=2, n_layers=1, batch=1)
    bins = random_bins(cfg, 5)
    c = make_cache(cfg, bins)
    assert B.iwdft_attn_kind(c.ctx) == "direct"
    c.close()
    run_stream(cfg, bins, tag="direct-10007", rec=(0, 64))


def test_paper_windows_on_a_context_that_is_a_power_of_two_full_size():
    """cfg2's shape with the paper's windows cut out of an 8192-token context (Sec. 5.1: 10 sink + 50 recent tokens,
    M = 8192 - 60 = 8132): the realistic setting, chirp-z attention at full size."""
    cfg = wl.CONFIGS["cfg2x"]
    assert cfg.n_prefill == 8192
    bins = wl.layer_bins(cfg)
    c = make_cache(cfg, bins)
    assert B.iwdft_attn_kind(c.ctx) == "chirp" and B.iwdft_prefill_kind(c.ctx) == "chirp"
    c.close()
    d = make_cache(cfg, bins, flags=B.IWDFT_FLAG_DENSE_PREFILL)
    assert B.iwdft_attn_kind(d.ctx) == "chirp" and B.iwdft_prefill_kind(d.ctx) == "dense"
    d.close()
    run_stream(cfg, bins, steps=3, tag="cfg2w-8132")
    run_stream(cfg, bins, flags=B.IWDFT_FLAG_DENSE_PREFILL, steps=1, tag="cfg2w-8132-dense")
    run_stream(cfg, bins, steps=3, fused=True, tag="cfg2w-8132-fused")


@pytest.mark.parametrize("scale", [2.0 ** -6, 2.0 ** 9])
def test_dense_and_fft_prefill_agree_across_the_dense_path_input_range(scale):
    # the dense contraction works on fp16 operand pairs (documented range +-65504, full precision above 2^-14):
    # inside that range a K/V scale of 2^-6 ... 2^9 (values to ~2^-10 and ~2^14 with the 0.1-10 channel scales)
    # leaves both prefills within the coefficient tolerance of the oracle and of each other
    cfg = small_cfg(L=2048, n_bins=500, dtype="bf16", n_layers=1, batch=1, n_kv_heads=2)
    bins = random_bins(cfg, 91)
    K, V = wl.prefill_tensors(cfg, DEV)
    K, V = (K.float() * scale).to(K.dtype), (V.float() * scale).to(V.dtype)
    got = {}
    for name, flag in (("fft", B.IWDFT_FLAG_FFT_PREFILL), ("dense", B.IWDFT_FLAG_DENSE_PREFILL)):
        c = make_cache(cfg, bins, flags=flag)
        c.prefill(K, V)
        got[name] = c.export_coeffs(0)
        ref = orc.prefill(f64(K[0, 0, 1]), bins[0])
        assert rel_l2(c128(got[name][0][0, 1]), ref) < TOL_COEF, name
        c.close()
    assert rel_l2(c128(got["dense"][0]), c128(got["fft"][0])) < 2e-5 and rel_l2(c128(got["dense"][1]), c128(got["fft"][1])) < 2e-5


def test_most_exact_tokens():
    # S + R = 1024 is the most the library takes
    cfg = small_cfg(L=512, n_bins=60, group=2, steps=3, n_layers=1, batch=1, n_sink=500, n_recent=524, dtype="bf16")
    run_stream(cfg, random_bins(cfg, 43), fused=True, tag="max-exact")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,S,R,n_bins", [(256, 0, 0, 129), (512, 2, 3, 77), (1024, 0, 0, 300), (2048, 0, 5, 77),
                                          (4096, 0, 0, 1500), (8192, 4, 0, 600), (16384, 0, 0, 900),
                                          (32768, 3, 2, 2100)])
def test_fft_prefill_all_transform_lengths(dtype, L, S, R, n_bins):
    # every transform length of the in-LDS FFT (2^8 .. 2^13) and the decimated form beyond it, ragged
    # scattered bins (both halves of the spectrum, so k and M - k both occur), with and without windows;
    # slices enough for the form that takes several channel pairs per load (8 x 8192 / L; 256 points have one)
    big = L > 8192
    cfg = small_cfg(L=L, dtype=dtype, n_bins=n_bins, n_sink=S, n_recent=R, steps=2,
                    n_layers=1 if big else 2, batch=1 if big else 2, n_kv_heads=2 if big else 2 * 8192 // L)
    bins = random_bins(cfg, 37)
    st = run_stream(cfg, bins, flags=B.IWDFT_FLAG_FFT_PREFILL, rec=(3, 50), tag=f"fftpf-{dtype}-L{L}")
    assert st["coef0"] < 2e-5


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_bins", [300, 2048])
def test_two_transforms_of_8192_points_in_a_workgroup_give_the_same_bits(dtype, n_bins):
    """Prefill, reconstruction and, in fp32, ablation of as many slices as fill whole rounds of workgroups of 1024 threads (two_transforms in
    pair_io.h) against the same slices a few at a time, which run one transform per workgroup: the same arithmetic."""
    cfg = small_cfg(L=8192, group=2, dtype=dtype, n_bins=n_bins, n_layers=1, batch=4, n_kv_heads=8)
    bins = [np.sort(np.random.default_rng(n_bins).choice(8192, size=n_bins, replace=False)).astype(np.int32)]
    K, V = wl.prefill_tensors(cfg, DEV)
    a = make_cache(cfg, bins)
    a.prefill(K, V)
    ka, va = a.reconstruct(0, 0, 8192)
    oa = torch.empty_like(K)
    B.iwdft_ablate_chunk(K, oa, 22, 3)
    few = small_cfg(L=8192, group=2, dtype=dtype, n_bins=n_bins, n_layers=1, batch=1, n_kv_heads=3)
    b = make_cache(few, bins)
    for row, h in ((0, 0), (1, 5), (3, 4)):
        Kb, Vb = (x[:, row:row + 1, h:h + 3].contiguous() for x in (K, V))
        b.prefill(Kb, Vb)
        for x, y in zip(a.export_coeffs(0), b.export_coeffs(0)):
            assert torch.equal(x[row:row + 1, h:h + 3], y)
        kb, vb = b.reconstruct(0, 0, 8192)
        assert torch.equal(ka[row:row + 1, h:h + 3], kb) and torch.equal(va[row:row + 1, h:h + 3], vb)
        ob = torch.empty_like(Kb)
        B.iwdft_ablate_chunk(Kb, ob, 22, 3)
        assert torch.equal(oa[:, row:row + 1, h:h + 3], ob)
    a.close()
    b.close()


@pytest.mark.parametrize("dtype,batch", [("bf16", 2), ("f32", 1), ("bf16", 4)])
@pytest.mark.parametrize("n_bins", [1024, 1025, 4000])
def test_reconstruction_of_two_blocks_with_two_transforms_gives_the_same_bits(dtype, batch, n_bins):
    """16384 slots, one round of workgroups at both sides of the row length up to which bf16 takes two transforms a workgroup, and two rounds:
    K and V of all slices against two slices at a time, which run one transform per workgroup."""
    cfg = small_cfg(L=16384, group=2, dtype=dtype, n_bins=n_bins, n_layers=1, batch=batch, n_kv_heads=8)
    bins = [np.sort(np.random.default_rng(n_bins).choice(8193, size=n_bins, replace=False)).astype(np.int32)]
    K, V = wl.prefill_tensors(cfg, DEV)
    a = make_cache(cfg, bins)
    a.prefill(K, V)
    ka, va = a.reconstruct(0, 0, 16384)
    b = make_cache(small_cfg(L=16384, group=2, dtype=dtype, n_bins=n_bins, n_layers=1, batch=1, n_kv_heads=2), bins)
    rows = 2 * 2 * 128 * (-(-n_bins // 32) * 32)  # floats of one slice pair's coefficients, K or V
    for row, h in ((0, 0), (batch - 1, 6)):
        b.prefill(*(x[:, row:row + 1, h:h + 2].contiguous() for x in (K, V)))
        for which in (0, 1):  # the same coefficients, so that the prefill's own rules do not matter
            src, dst = (c.state[c.state_bytes - 8 * 128 * (-(-n_bins // 32) * 32) * 2 * n:].view(torch.float32)
                        for c, n in ((a, batch * 8), (b, 2)))
            at = which * src.numel() // 2 + (row * 8 + h) * (rows // 2)
            dst[which * rows:(which + 1) * rows] = src[at:at + rows]
        kb, vb = b.reconstruct(0, 0, 16384)
        assert torch.equal(ka[row:row + 1, h:h + 2], kb) and torch.equal(va[row:row + 1, h:h + 2], vb)
    a.close()
    b.close()


def test_fft_and_dense_prefill_give_the_same_state():
    cfg = small_cfg(L=4096, dtype="bf16", n_bins=500, n_sink=2, n_recent=3)
    bins = random_bins(cfg, 41)
    K, V = wl.prefill_tensors(cfg, DEV)
    a, b = make_cache(cfg, bins, flags=B.IWDFT_FLAG_FFT_PREFILL), make_cache(cfg, bins, flags=B.IWDFT_FLAG_DENSE_PREFILL)
    assert B.iwdft_prefill_kind(a.ctx) == "fft" and B.iwdft_prefill_kind(b.ctx) == "dense"
    c = make_cache(cfg, bins)                      # no flag: 500 kept bins -> FFT
    d = make_cache(small_cfg(L=4096, n_bins=100), [np.arange(100, dtype=np.int32)] * 2)   # few bins -> dense
    assert B.iwdft_prefill_kind(c.ctx) == "fft" and B.iwdft_prefill_kind(d.ctx) == "dense"
    c.close()
    d.close()
    a.prefill(K, V)
    b.prefill(K, V)
    for l in range(cfg.n_layers):
        (ka, va), (kb, vb) = a.export_coeffs(l), b.export_coeffs(l)
        assert rel_l2(c128(ka), c128(kb)) < 1e-5 and rel_l2(c128(va), c128(vb)) < 1e-5
    a.close()
    b.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,n_bins,heads,flag", [
    (512, 400, 128, True), (1024, 400, 64, True), (2048, 500, 33, True), (4096, 600, 17, True), (8192, 5000, 9, True),
    (16384, 1100, 2, True), (32768, 2100, 2, True), (16384, 5000, 2, True),
    (512, 100, 128, False), (1024, 200, 64, False), (2048, 300, 33, False), (4096, 200, 17, False), (8192, 300, 9, False),
    (16384, 200, 2, False),  # channels of a pair scaled to one size
])
def test_fft_prefill_of_tensors_that_are_not_16_byte_aligned(dtype, L, n_bins, heads, flag):
    """The FFT prefill fetches several channel pairs with one 8- or 16-byte load when K and V allow it and the slices fill the
    device (8 x 8192 / L of them); tensors that start 8 bytes off take one pair per load instead.  Every pair's transform is
    the same arithmetic either way: the two states agree bit for bit."""
    cfg = small_cfg(L=L, n_bins=n_bins, n_layers=1, batch=1, n_kv_heads=heads, dtype=dtype, mask="low")
    bins = wl.layer_bins(cfg)
    K, V = wl.prefill_tensors(cfg, DEV)
    pad = 8 // K.element_size()
    Ku = torch.empty(K.numel() + pad, dtype=K.dtype, device=DEV)[pad:].view_as(K)
    Vu = torch.empty(V.numel() + pad, dtype=V.dtype, device=DEV)[pad:].view_as(V)
    Ku.copy_(K)
    Vu.copy_(V)
    assert K.data_ptr() % 16 == 0 and Ku.data_ptr() % 16 == 8 and Vu.data_ptr() % 16 == 8
    a = make_cache(cfg, bins, flags=B.IWDFT_FLAG_FFT_PREFILL if flag else 0)
    b = make_cache(cfg, bins, flags=B.IWDFT_FLAG_FFT_PREFILL if flag else 0)
    assert B.iwdft_prefill_kind(a.ctx) == "fft"
    a.prefill(K, V)
    b.prefill(Ku, Vu)
    (ka, va), (kb, vb) = a.export_coeffs(0), b.export_coeffs(0)
    assert torch.equal(ka, kb) and torch.equal(va, vb)
    a.close()
    b.close()


def test_misaligned_tensors_are_refused_before_any_launch():
    """Token, query, output and prefill tensors are accessed 16 bytes at a time: a tensor that starts elsewhere is an
    IWDFT_ERR_ARG (only the FFT prefill without windows takes K, V aligned to a channel pair, tested above)."""
    def off(t, pad=4):
        u = torch.empty(t.numel() + pad, dtype=t.dtype, device=DEV)[pad:].view_as(t)
        u.copy_(t)
        return u

    for S, R, flags in ((0, 0, B.IWDFT_FLAG_DENSE_PREFILL), (2, 3, B.IWDFT_FLAG_FFT_PREFILL)):
        cfg = small_cfg(L=1024, n_bins=400, n_layers=1, batch=1, n_kv_heads=2, dtype="bf16", n_sink=S, n_recent=R)
        bins = wl.layer_bins(cfg)
        K, V = wl.prefill_tensors(cfg, DEV)
        c = make_cache(cfg, bins, flags=flags)
        for args in ((off(K), V), (K, off(V))):
            with pytest.raises(B.IwdftError) as e:
                c.prefill(*args)
            assert e.value.code == B.IWDFT_ERR_ARG
        c.prefill(K, V)
        tk, tv, q = wl.decode_step(cfg, 0, DEV)
        out = torch.empty_like(q)
        for call in (lambda: c.append(off(tk), tv), lambda: c.append(tk, off(tv)), lambda: c.attend(off(q), out),
                     lambda: c.attend(q, off(out)), lambda: c.step(off(tk), tv, q, out), lambda: c.step(tk, tv, off(q), out),
                     lambda: c.step(tk, tv, q, off(out))):
            with pytest.raises(B.IwdftError) as e:
                call()
            assert e.value.code == B.IWDFT_ERR_ARG
        assert c.T == cfg.L                      # nothing was absorbed by the refused calls
        c.append(tk, tv)
        c.attend(q, out)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(out.float()).all())
        c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,S,R,n_bins,n_layers", [
    (257, 0, 0, 257, 2),      # prime, every bin kept: convolutions of 1024 points
    (1000, 3, 5, 333, 2),     # 2048
    (1001, 0, 0, 1001, 4),    # ... enough slices for several channel pairs per load
    (2047, 0, 0, 700, 2),     # 4096, one point short of the limit
    (2047, 2, 2, 1100, 3),
    (4095, 0, 3, 1500, 2),    # 8192
    (4095, 0, 0, 1500, 3),
    (8191, 0, 0, 2100, 3),    # 16384
    (8191, 1, 0, 900, 1),
    (16324, 10, 50, 1500, 1),  # two blocks of 8162 points, the paper's windows
    (12003, 0, 0, 1500, 3),    # three blocks of 4001 points
])
def test_chirp_prefill_all_convolution_lengths(dtype, L, S, R, n_bins, n_layers):
    cfg = small_cfg(L=L, dtype=dtype, n_bins=n_bins, n_sink=S, n_recent=R, steps=1, n_layers=n_layers,
                    batch=2 if n_layers > 1 else 1, n_kv_heads=8 if n_layers > 2 else 2)
    c = make_cache(cfg, random_bins(cfg, 53))
    assert B.iwdft_prefill_kind(c.ctx) == "chirp"
    c.close()
    st = run_stream(cfg, random_bins(cfg, 53), rec=(3, 20), tag=f"chirppf-{dtype}-L{L}")
    assert st["coef0"] < 2e-5


@pytest.mark.parametrize("L", [259, 511, 513, 1000, 2047, 2049, 4095, 4097, 8191, 2 * 6144, 3 * 8192, 3 * 8191, 9 * 931, 5 * 8191,
                               41 * 353, 37 * 687, 11 * 2971, 13 * 5039,  # 2, 7, 4 and 8 blocks that do not divide L, last ones one sample shorter
                               24582, 65541, 63012])  # ... 4, 9 and 8, which have 2, 3 and 4 in common with L: taps for a part of the frequencies
def test_interpolated_prefill_against_64_bit_transforms(L):
    """Every grid length at both ends of its range (L / 2 up to a power of two: the widest and the closest spacing of the taps; 24576
    = 3 x 8192: taps on grid points), a layer of low bins and one of bins anywhere.  Bar: aliasing 2e-8 + fp32 rounding, which grows
    by at most 2^-24 per radix-2 stage in the 2-norm (16 stages with the two ends): 1e-6."""
    rng = np.random.default_rng(L)
    low = np.arange(min(L // 4, 700), dtype=np.int32)
    wide = np.unique(np.r_[0, 1, 2, 3, L // 2 - 1, L // 2, L // 2 + 1, L - 3, L - 2, L - 1, rng.integers(0, L, 500)]).astype(np.int32)
    K, V = torch.randn((2, 2, 1, 8, L, 128), device=DEV, generator=torch.Generator(DEV).manual_seed(L))
    c = B.Cache(2, 1, 8, 8, 128, torch.float32, L, [low, wide])
    assert B.iwdft_prefill_kind(c.ctx) == "chirp"
    c.prefill(K, V)
    for layer, bins in enumerate((low, wide)):
        for X, got in zip((K, V), c.export_coeffs(layer)):
            ref = torch.fft.fft(X[layer, 0, ::7].cpu().double(), dim=1)[:, bins.astype(np.int64)] / L
            got = got[0, ::7].cpu().to(torch.complex128)
            assert float((got - ref).norm() / ref.norm()) < 1e-6
            assert float((got - ref).abs().max() / ref.abs().pow(2).mean().sqrt()) < 1e-5
    c.close()


@pytest.mark.parametrize("blocks,Q,heads", [(2, 8162, 16), (3, 8191, 16), (5, 6005, 16), (8, 8191, 8), (16, 8191, 8), (64, 8191, 8)])
def test_interpolated_prefill_of_several_blocks_is_as_exact_beside_an_offset(blocks, Q, heads):
    """Noise of size 1 beside an offset of 30.  Near the offset's own bin, 0, the interpolation sums values of its size, whose taps and
    twiddles are rounded to 2^-25; that is the same in every block and adds up.  Bar in units of the offset and of the noise's sums:
    2^-20 for the roundings of one block (at most 2^-24 per radix-2 stage, 16 with the two ends), 2^-21 sqrt(blocks) for what adds up.  The
    first 64 bins without 0, and the rest, which roundings alone reach."""
    L = blocks * Q
    assert next(p for p in range(1, L) if L % p == 0 and L // p <= 8192) == blocks
    K = 30 + torch.randn((1, 1, heads, L, 128), device=DEV, generator=torch.Generator(DEV).manual_seed(L))
    n_bins = 2000
    c = B.Cache(1, 1, heads, heads, 128, torch.float32, L, [np.arange(n_bins, dtype=np.int32)])
    assert B.iwdft_prefill_kind(c.ctx) == "chirp"
    c.prefill(K, K)
    got = c.export_coeffs(0)[1][0, heads - 1].cpu().to(torch.complex128)
    ref = torch.fft.fft(K[0, 0, heads - 1].cpu().double().T.contiguous(), dim=1)[:, :n_bins] / L
    err = (got if got.shape == ref.shape else got.T) - ref
    for rest, bar in ((slice(1, 64), 2.0 ** -20 + 2.0 ** -21 * blocks ** 0.5), (slice(64, n_bins), 2.0 ** -20)):
        assert float(err[:, rest].abs().pow(2).mean().sqrt()) * L ** 0.5 < 30 * bar, rest
    c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,reach,heads,S,R,off", [
    (16384, 256, 64, 0, 0, 0), (16384, 257, 35, 2, 3, 0), (16384, 1024, 32, 0, 0, 8),    # a grid of 4096 points (fp32, 32 slices)
    (32768, 512, 32, 0, 0, 8), (32768, 2048, 17, 0, 5, 0), (32768, 4096, 17, 0, 0, 0),   # ... 4096 (two groups of slices); the tokens themselves
    (65536, 1000, 9, 10, 50, 0), (131072, 4096, 9, 0, 0, 8), (262144, 4096, 4, 1, 0, 0),  # ... 16384: three groups
])
def test_prefill_of_low_frequencies_against_64_bit_transforms(dtype, L, reach, heads, S, R, off):
    """Tokens themselves and four to sixteen per grid point, bins up to a quarter of the grid and their mirrors; 8-byte aligned tensors.  Bar: aliasing
    2e-9 + fp32 rounding of at most 2^-24 per radix-2 stage (14, window and gain): 1e-6.  Channel 5 carries a tone of 30 at the
    frequency that aliases onto the last bin: 2e-9 of it there, and the rounding of its samples, which may repeat with it, 2^-25."""
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    rng = np.random.default_rng(L + reach)
    N = 1024
    while N < 4 * reach or 16 * N < L:
        N *= 2
    low = np.arange(reach + 1) if reach <= 512 or reach >= 4096 else rng.integers(0, reach, reach // 2)
    bins = np.unique(np.r_[0, 1, low, reach, L - reach, L - reach + 1, L - 1]).astype(np.int32)
    X = [torch.randn((1, 1, heads, S + L + R, 128), device=DEV, generator=torch.Generator(DEV).manual_seed(L + i)) for i in range(2)]
    n = torch.arange(L, device=DEV, dtype=torch.float64)
    for x in X:
        x[..., S:S + L, 5] += (30 * torch.cos(2 * np.pi / L * torch.remainder(n * (N - reach), L))).float()
    pad = off // td.itemsize
    K, V = (torch.empty(x.numel() + pad, dtype=td, device=DEV)[pad:].view(x.shape).copy_(x) for x in X)
    c = B.Cache(1, 1, heads, heads, 128, td, L, [bins], n_sink=S, n_recent=R)
    assert B.iwdft_prefill_kind(c.ctx) == "fft"
    c.prefill(K, V)
    for x, got in zip((K, V), c.export_coeffs(0)):
        for h in (0, heads - 1):
            ref = torch.fft.fft(x[0, 0, h, S:S + L].cpu().double().T.contiguous(), dim=1)[:, bins.astype(np.int64)] / L
            err = got[0, h].cpu().to(torch.complex128)
            err = (err if err.shape == ref.shape else err.T) - ref
            rest = [i for i in range(128) if i not in (4, 5)]  # the tone's transform also holds channel 4
            assert float(err[rest].norm() / ref[rest].norm()) < 1e-6
            assert float(err[rest].abs().max() / ref[rest].abs().pow(2).mean().sqrt()) < 1e-5
            assert float(err[4:6].abs().max()) < 30 * (2e-9 + 2.0 ** -25)
    c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,n_bins,heads", [(16384, 1024, 32), (32768, 1000, 17), (32768, 4096, 16), (65536, 1000, 16), (65536, 4096, 2), (131072, 2048, 3),
                                             (131072, 4096, 4), (262144, 4096, 2)])
def test_prefill_is_as_exact_beside_an_offset_or_a_strong_tone(dtype, L, n_bins, heads):
    """Channels 0 .. 31: noise of size 1 beside an offset of 30, 32 .. 63 beside a tone of 30 at three periods, 64 .. 95 at six tenths of the
    kept band, the rest noise alone; every eighth of the kept bins is judged by itself, without the tone and its neighbours.  Bar: roundings of
    2^-24 of the signal, white over all L bins and growing by at most one per radix-2 stage: below 2^-20 of its root mean square.  bf16
    samples with an offset: their sums over the first butterflies are exact (24 bits hold 256 sums of 8-bit values of one size), so that
    nothing of the offset is left, and the noise alone has 1e-6."""
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(DEV).manual_seed(L + n_bins)
    n = torch.arange(L, device=DEV, dtype=torch.float64)[:, None]
    mid = n_bins * 6 // 10
    X = [torch.randn((1, 1, heads, L, 128), device=DEV, generator=gen) for _ in range(2)]
    for x in X:
        x[..., :32] += 30
        for c, k in ((slice(32, 64), 3), (slice(64, 96), mid)):
            phase = 6.28 * torch.rand(32, device=DEV, generator=gen, dtype=torch.float64)
            x[..., c] += (30 * torch.cos(2 * np.pi / L * torch.remainder(n * k, L) + phase)).float()
    K, V = (x.to(td) for x in X)
    c = B.Cache(1, 1, heads, heads, 128, td, L, [np.arange(n_bins, dtype=np.int32)])
    assert B.iwdft_prefill_kind(c.ctx) == "fft"
    c.prefill(K, V)
    exact_sums = 1e-6 if dtype == "bf16" else 30 * 2.0 ** -20
    for x, got in zip((K, V), c.export_coeffs(0)):
        for h in (0, heads - 1):
            ref = torch.fft.fft(x[0, 0, h].cpu().double().T.contiguous(), dim=1)[:, :n_bins] / L
            err = got[0, h].cpu().to(torch.complex128)
            err = (err if err.shape == ref.shape else err.T) - ref
            for chans, tone, bar in ((slice(0, 32), 0, exact_sums), (slice(32, 64), 3, 21.2 * 2.0 ** -20),
                                     (slice(64, 96), mid, 21.2 * 2.0 ** -20), (slice(96, 128), 0, 1e-6)):
                for e in range(8):
                    rest = [k for k in range(e * n_bins // 8, (e + 1) * n_bins // 8) if abs(k - tone) > 2]
                    got_rel = float(err[chans][:, rest].abs().pow(2).mean().sqrt()) * L ** 0.5
                    assert got_rel < bar, (chans, e, got_rel, bar)
    c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,n_bins,group,heads,gain", [
    (16384, 256, 1, 2, 1), (16384, 1025, 3, 2, 1), (32768, 2049, 4, 2, 1),  # 4 tokens per grid point of 4096 points (two cases), of 8192
    (32768, 500, 2, 3, 1), (65536, 1025, 8, 1, 1), (65536, 4097, 2, 1, 1),  # 8 of 4096, 16 of 4096, 4 of 16384 points
    (262144, 4096, 2, 1, 1),                                               # 16 of 16384
    (16384, 256, 2, 2, 300), (65536, 4096, 2, 1, 300),                      # scores whose maximum needs a look at every token
])
def test_attention_of_low_frequencies_against_64_bit_transforms(dtype, L, n_bins, group, heads, gain):
    """Scores carry 2^-24 of their size per radix-2 stage and tap (about 4 x 2^-24 in the 2-norm, 2^-21 with the worst token), the same
    as weights; outputs in bf16 are rounded to 2^-9."""
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(DEV).manual_seed(L + n_bins)
    K, V = (torch.randn((1, 1, heads, L, 128), device=DEV, generator=gen).to(td) for _ in range(2))
    q = (gain * torch.randn((1, 1, heads * group, 128), device=DEV, generator=gen) * (L / n_bins) ** 0.5).to(td)
    c = B.Cache(1, 1, heads, heads * group, 128, td, L, [np.arange(n_bins, dtype=np.int32)])
    c.prefill(K, V)
    out = c.attend(q)
    keep = torch.zeros(L, dtype=torch.float64)
    keep[:n_bins] = 1
    largest = 0.0
    for h in range(heads):
        k, v = (torch.fft.ifft(torch.fft.fft(x[0, 0, h].cpu().double().T.contiguous()) * keep).real for x in (K, V))
        s = q[0, 0, h * group:(h + 1) * group].cpu().double() @ k / 128 ** 0.5
        ref = torch.softmax(s, 1) @ v.T
        err = float((out[0, 0, h * group:(h + 1) * group].cpu().double() - ref).norm() / ref.norm())
        big = float(s.abs().max())
        largest = max(largest, big)
        assert err < 1e-5 + 2.0 ** -21 * big + (2.0 ** -9 if dtype == "bf16" else 0), (err, big)
    assert (largest > 64 / 0.083 / 1.4427) == (gain > 1), largest
    c.close()


@pytest.mark.parametrize("L,n_bins", [(65536, 1000), (131072, 4096), (262144, 4096)])
def test_attention_of_low_frequencies_is_as_exact_beside_a_mean_score(L, n_bins):
    """Scores of size 2 beside a mean of 13 to 19, which softmax does not see: it must not cost precision either.  Reference in 64 bits from the
    stored coefficients.  Bar: what is left are roundings of scores of size 2, of exponentials and of the transforms' values, 2^-24
    each and independent from token to token: 2e-7 (seen 1.0e-7 .. 1.4e-7; 2.2e-7 .. 3.0e-7 with the mean inside the transforms)."""
    heads, group = 4, 4
    gen = torch.Generator().manual_seed(L + n_bins)
    K, V = (torch.randn((heads, L, 128), generator=gen) for _ in range(2))
    K[..., ::3] += 30
    q = torch.randn((1, 1, heads * group, 128), generator=gen) * (L / n_bins) ** 0.5 / 16
    c = B.Cache(1, 1, heads, heads * group, 128, torch.float32, L, [np.arange(n_bins, dtype=np.int32)])
    c.prefill(K.to(DEV)[None, None], V.to(DEV)[None, None])
    out = c.attend(q.to(DEV)).cpu().double()
    Bp = -(-n_bins // 32) * 32
    U = c.state[c.state_bytes - 16 * heads * 128 * Bp:].view(torch.float32).view(2, heads, 128, Bp, 2).cpu().double()
    U = torch.view_as_complex(U.contiguous())
    errs = []
    for h in range(heads):
        full = torch.zeros((2, 128, L), dtype=torch.complex128)
        full[:, :, :n_bins] = U[:, h, :, :n_bins]
        k, v = torch.fft.ifft(full, dim=-1).real
        ref = torch.softmax(q[0, 0, h * group:(h + 1) * group].double() @ k / 128 ** 0.5, 1) @ v.T
        errs.append(float((out[0, 0, h * group:(h + 1) * group] - ref).norm() / ref.norm()))
    assert np.mean(errs) < 2e-7, errs
    c.close()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("L", [2047, 2049, 2050, 3001, 4095, 4097, 6000, 8132, 8191])
def test_attention_of_any_length_against_64_bit_transforms(L, wide):
    """Low bins up to the last one that a grid of the next power of two carries (interpolation; chirp-z transforms up to 2048 tokens), and
    bins anywhere, L / 2 and mirrors among them (chirp-z).  Bar as above: 2^-21 of the scores."""
    gen = torch.Generator(DEV).manual_seed(L)
    rng = np.random.default_rng(L)
    N = 1 << (L - 1).bit_length()
    low = np.r_[np.arange(3, L // 6), L - 1, L - 2, (N // 4 - 1) if 2 * N > 4 * (N // 4 - 1) and N // 4 - 1 < L // 2 else 7]
    bins = np.unique(low) if not wide else np.unique(np.r_[0, 1, 2, L // 2 - 1, L // 2, L // 2 + 1, L - 2, L - 1, rng.integers(0, L, L // 5)])
    heads, group = 3, 3
    K, V = (torch.randn((1, 1, heads, L, 128), device=DEV, generator=gen) for _ in range(2))
    q = torch.randn((1, 1, heads * group, 128), device=DEV, generator=gen) * (L / len(bins)) ** 0.5
    c = B.Cache(1, 1, heads, heads * group, 128, torch.float32, L, [bins.astype(np.int32)])
    c.prefill(K, V)
    out = c.attend(q)
    keep = torch.zeros(L, dtype=torch.float64)
    keep[torch.from_numpy(bins).long()] = 1
    for h in range(heads):
        k, v = (torch.fft.ifft(torch.fft.fft(x[0, 0, h].cpu().double().T.contiguous()) * keep).real for x in (K, V))
        s = q[0, 0, h * group:(h + 1) * group].cpu().double() @ k / 128 ** 0.5
        ref = torch.softmax(s, 1) @ v.T
        err = float((out[0, 0, h * group:(h + 1) * group].cpu().double() - ref).norm() / ref.norm())
        assert err < 2e-6 + 2.0 ** -21 * float(s.abs().max()), err
    c.close()


def test_create_of_a_length_that_is_no_power_of_two_costs_what_another_does():
    """A context's tables (taps, 1 / W, chirp) are made on the device: with the same bins and slices M = 8132 differs from M = 8192 by a few
    launches and one wait, where tables of 8132 entries each made on the host took 15 times as long (best of 20 calls each)."""
    best = {}
    for L in (8192, 8132):
        d = B.Descriptor(1, 1, 8, 32, 128, B.IWDFT_BF16, L, [np.arange(2033, dtype=np.int32)], write_every=16)
        state, ws = (torch.empty(n, dtype=torch.uint8, device=DEV) for n in B.iwdft_query_bytes(d))
        times = []
        for _ in range(20):
            torch.cuda.synchronize()
            t = time.perf_counter()
            ctx = B.iwdft_create(d, state, ws)
            times.append(time.perf_counter() - t)
            B.iwdft_destroy(ctx)
        best[L] = min(times)
    assert best[8132] < 4 * best[8192], best


def test_chirp_prefill_keeps_the_precision_of_a_small_channel_next_to_a_large_one():
    # neighbouring channels share a transform; every channel has to be as accurate as alone (fp32 rounding, 2^-24, times
    # ~log2 of the 16384 points of each of two transforms and the tables: below 1e-5)
    cfg = small_cfg(L=8132, n_bins=2033, dtype="f32", n_layers=1, batch=1, n_kv_heads=1)
    bins = [np.arange(cfg.n_bins, dtype=np.int32)]
    K, V = wl.prefill_tensors(cfg, DEV)
    K[..., 0::4] *= 2.0 ** 20
    K[..., 3::4] *= 2.0 ** -20
    V[..., 1] = 0.0
    V[..., 100, 6] = float("inf")
    c = make_cache(cfg, bins)
    assert B.iwdft_prefill_kind(c.ctx) == "chirp"
    c.prefill(K, V)
    for name, X, got in zip("KV", (K, V), c.export_coeffs(0)):
        X = X.nan_to_num(0.0, 0.0, 0.0)
        ref = orc.prefill(f64(X[0, 0, 0]), bins[0])
        got = c128(got[0, 0]).reshape(ref.shape)
        for ch in range(128):
            g, r = np.take(got, ch, axis=ref.shape.index(128)), np.take(ref, ch, axis=ref.shape.index(128))
            if name == "V" and ch == 6:  # its transform partner, channel 7, is as it would be without it
                assert not np.isfinite(g).any()
            else:
                assert np.linalg.norm(g - r) <= 1e-5 * np.linalg.norm(r), ch
    c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,n_bins,heads", [
    (256, 40, 1), (512, 128, 1), (1024, 300, 1), (2048, 128, 1), (4096, 200, 1), (8192, 300, 1),  # one pair per load
    (256, 256, 257), (512, 100, 129), (1024, 256, 65), (2048, 383, 33), (4096, 128, 17), (8192, 383, 9),  # several
    (16384, 128, 2), (65536, 383, 1),  # residues
])
def test_fft_prefill_keeps_the_precision_of_a_small_channel_next_to_a_large_one(dtype, L, n_bins, heads):
    """Fewer than 384 kept bins: neighbouring channels share a transform, each is as accurate as alone (fp32 rounding, 2^-24, times ~log2 of the 8192
    points and the residue sums: below 4e-6 relative per channel over the kept bins), zero stays zero, and a channel that is not
    finite does not reach its partner -- in every residue, and where it is not finite in one of them only."""
    cfg = small_cfg(L=L, n_bins=n_bins, dtype=dtype, n_layers=1, batch=1, n_kv_heads=heads)
    bins = random_bins(cfg, 23)
    K, V = wl.prefill_tensors(cfg, DEV)
    K[..., 0::4] *= 2.0 ** 20
    K[..., 3::4] *= 2.0 ** -20
    K[..., L // 2:, 9] = 0.0
    K[..., L // 2:, 8] *= 2.0 ** 10
    V[..., 1] = 0.0
    V[..., 64] = 0.0
    V[..., 100, 6] = float("inf")
    V[..., 7, 11] = float("nan")
    V[..., 8, 20:22] = float("-inf")
    c = make_cache(cfg, bins)
    assert B.iwdft_prefill_kind(c.ctx) == "fft"
    c.prefill(K, V)
    for name, X, got in zip("KV", (K, V), c.export_coeffs(0)):
        for h in sorted({0, heads // 2, heads - 1}):
            ref = orc.prefill(f64(X[0, 0, h].nan_to_num(0.0, 0.0, 0.0)), bins[0])
            g = c128(got[0, h])
            assert g.shape == ref.shape == (n_bins, 128)
            for ch in range(128):
                if name == "V" and ch in (6, 11, 20, 21):
                    assert not np.isfinite(g[:, ch]).any(), ch
                else:
                    assert np.linalg.norm(g[:, ch] - ref[:, ch]) <= 4e-6 * np.linalg.norm(ref[:, ch]), (name, h, ch)
    c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,n_bins,heads", [(32768, 800, 16), (65536, 4000, 1), (65536, 2048, 2), (131072, 1000, 1)])
def test_decimated_prefill_keeps_every_channel_alone(dtype, L, n_bins, heads):
    """Low bins of long contexts, grids of 4096 to 16384 points: every channel goes through transforms of its own in 64 bits, however large or
    small its neighbours are, zero stays zero, and one that is not finite reaches no other.  Bar: rounding of the result, 2^-25 per part."""
    cfg = small_cfg(L=L, n_bins=n_bins, dtype=dtype, n_layers=1, batch=1, n_kv_heads=heads)
    bins = [np.arange(n_bins, dtype=np.int32)]
    K, V = wl.prefill_tensors(cfg, DEV)
    K[..., 0::4] *= 2.0 ** 40
    K[..., 3::4] *= 2.0 ** -40
    K[..., L // 2:, 9] = 0.0
    V[..., 1] = 0.0
    V[..., 100, 6] = float("inf")
    V[..., L - 1, 11] = float("nan")
    V[..., 8, 20:22] = float("-inf")
    c = make_cache(cfg, bins)
    assert B.iwdft_prefill_kind(c.ctx) == "fft"
    c.prefill(K, V)
    for name, X, got in zip("KV", (K, V), c.export_coeffs(0)):
        ref = torch.fft.fft(X[0, 0, -1].cpu().double().nan_to_num(0.0, 0.0, 0.0).T.contiguous(), dim=1)[:, :n_bins] / L
        g = got[0, -1].cpu().to(torch.complex128)
        g = g if g.shape == ref.shape else g.T
        for ch in range(128):
            if name == "V" and ch in (6, 11, 20, 21):
                assert not torch.isfinite(g[ch].abs()).any(), ch
            else:
                assert float((g[ch] - ref[ch]).norm()) <= 2.0 ** -24 * float(ref[ch].norm()), (name, ch)
    c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,n_bins,batch", [(256, 100, 34), (512, 300, 17), (1024, 600, 25), (2048, 700, 5), (4096, 2100, 3),
                                            (8192, 900, 2), (16384, 2000, 2)])
def test_reconstruct_several_channel_pairs_per_store(dtype, L, n_bins, batch):
    """Enough slices for the form that stores several channel pairs at once (bf16 from 2048 points on, fp32 from 1024 on; shorter
    ones have the one-pair form only), a range that starts and ends inside the rows and wraps: against the oracle on three slices,
    and bit for bit against the one-pair form that outputs 8 bytes off take."""
    cfg = small_cfg(L=L, dtype=dtype, n_bins=n_bins, steps=3, group=1, n_layers=1, batch=batch, n_kv_heads=8)
    bins = random_bins(cfg, 79)
    K, V = wl.prefill_tensors(cfg, DEV)
    cache = make_cache(cfg, bins)
    cache.prefill(K, V)
    ora = SliceOracle(cfg, bins, None, K, V, wl.sample_slices(cfg, 3))
    for i in range(3):
        tk, tv, _ = wl.decode_step(cfg, i, DEV)
        cache.append(tk, tv)
        ora.append(tk, tv)
    a0, n = L // 4 + 3, L // 2 + 1
    check_reconstruct(cfg, cache, ora, a0, n, f"rec-wide-{dtype}-L{L}")
    Ka, Va = cache.reconstruct(0, a0, n)
    flat = torch.empty(2 * Ka.numel() + 64, dtype=Ka.dtype, device=DEV)
    off = 8 // Ka.element_size()
    Kb = flat[off:off + Ka.numel()].view(Ka.shape)
    Vb = flat[off + Ka.numel():off + 2 * Ka.numel()].view(Va.shape)
    B.iwdft_reconstruct(cache.ctx, 0, a0, n, Kb, Vb)
    torch.cuda.synchronize()
    assert torch.equal(Ka, Kb) and torch.equal(Va, Vb)
    cache.close()
