"""Boundary checks that need no GPU: the library loads, exports every symbol the
header declares, and rejects bad descriptors with the documented error codes."""
import ctypes
import os
import re

import numpy as np
import pytest

from paper_2507_20030_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_functions():
    src = open(os.path.join(ROOT, "include", "iwdft.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b((?:iwdft_|compressed_)\w+)\s*\(", src)))


def test_library_exports_every_declared_symbol():
    lib = B.load_library()
    names = header_functions()
    assert set(names) == set(B.EXPORTED)
    for n in names:
        assert hasattr(lib, n), n


def desc(**kw):
    args = dict(n_layers=2, batch=1, n_kv_heads=2, n_q_heads=4, head_dim=128, kv_dtype=B.IWDFT_BF16,
                M=64, bins=[np.arange(8), np.array([0, 3, 9, 63])])
    args.update(kw)
    return B.Descriptor(**args)


def test_query_bytes_accounts_for_padded_rows():
    d = desc()
    state, ws = B.iwdft_query_bytes(d)
    # rows are padded to 32 bins: 2 layers * 2 slices * 128 channels * 32 * 8 B per tensor
    coef = 2 * 2 * 128 * 32 * 8
    assert state >= 2 * coef and state < 2 * coef + 4096
    assert ws >= 2 * (2 * 2 * 2 * 32 * 8)
    assert state % 256 == 0 and ws % 256 == 0


def padded(*sizes):
    return sum(-(-n // 256) * 256 for n in sizes)


@pytest.mark.parametrize("M,reach,points", [
    (2047, 400, 0), (2049, 1023, 4096), (2049, 1024, 0), (2050, 1023, 4096), (2050, 1024, 0), (4095, 1023, 4096), (4095, 1024, 0), (4097, 2047, 8192),
    (5000, 700, 8192), (8132, 2032, 8192), (8132, 2047, 8192), (8132, 2048, 0), (8191, 2047, 8192), (8194, 100, 0),
])
def test_attention_of_other_lengths_takes_the_grid_by_rule(M, reach, points):
    """2049 .. 8191 tokens and all frequencies below a quarter of the next power of two: the workspace then holds that grid's 1 / W and
    the taps of the tokens and of the grid's points, ten floats each."""
    low, high = (B.iwdft_query_bytes(desc(M=M, bins=[np.array([0, reach]), np.array([k])], flags=B.IWDFT_FLAG_DENSE_PREFILL))[1]
                 for k in (3, M // 2))
    assert low - high == (padded(4 * (points // 4 + 1), 40 * (M // 2 + 1), 40 * (points // 2 + 1)) if points else 0)
    mirrored = B.iwdft_query_bytes(desc(M=M, bins=[np.array([0, reach]), np.array([M - 1])], flags=B.IWDFT_FLAG_DENSE_PREFILL))[1]
    assert mirrored == low


@pytest.mark.parametrize("M,reach,points", [
    (8192, 100, 0), (16384, 1024, 4096), (16384, 1025, 0), (32768, 1024, 4096), (32768, 1025, 8192), (32768, 2049, 0), (65536, 4096, 16384),
    (65536, 10, 4096), (131072, 10, 8192), (262144, 4096, 16384), (262144, 4097, 0), (524288, 10, 0),
])
def test_attention_of_long_contexts_takes_the_grid_by_rule(M, reach, points):
    """M = 2^m, four to sixteen tokens per point of a grid of 4096 to 16384 points that is four times as long as the highest kept frequency, no
    bin beyond M / 2: the workspace then holds 1 / W and eight taps per token between two points."""
    low, high = (B.iwdft_query_bytes(desc(M=M, bins=[np.array([0, reach]), np.array([k])], flags=B.IWDFT_FLAG_DENSE_PREFILL))[1]
                 for k in (3, M - 1))
    assert low - high == (padded(4 * (points // 4 + 1), 32 * (M // points)) if points else 0)


@pytest.mark.parametrize("M,n_bins,heads,dtype,points", [
    (131072, 4097, 1, B.IWDFT_BF16, 16384), (131072, 4098, 1, B.IWDFT_BF16, 0), (65536, 4096, 1, B.IWDFT_BF16, 16384),
    (65536, 2048, 2, B.IWDFT_BF16, 8192), (32768, 4096, 64, B.IWDFT_BF16, 0), (32768, 1024, 15, B.IWDFT_F32, 0), (32768, 1024, 16, B.IWDFT_F32, 4096),
    (16384, 1024, 64, B.IWDFT_BF16, 0), (16384, 1024, 31, B.IWDFT_F32, 0), (16384, 1024, 32, B.IWDFT_F32, 4096), (262144, 4096, 3, B.IWDFT_F32, 16384),
    (131072, 127, 1, B.IWDFT_BF16, 0),
])
def test_prefill_of_long_contexts_takes_the_grid_by_rule(M, n_bins, heads, dtype, points):
    """Low bins: grids of 8192 points and more from eight tokens per point on, of 4096 from 16 slices on, four tokens per point with 16384
    points, or with 4096 in fp32 from 32 slices on; never where the contraction runs.  The workspace then holds up to 128 MiB of grids
    (64-bit, 2 tensors x 128 channels), their transforms' twiddles and 1 / W, and ten taps per token between two points."""
    kw = dict(M=M, n_layers=1, n_kv_heads=heads, n_q_heads=heads, kv_dtype=dtype, bins=[np.arange(n_bins)])
    ws = B.iwdft_query_bytes(desc(**kw))[1]
    dense = B.iwdft_query_bytes(desc(**kw, flags=B.IWDFT_FLAG_DENSE_PREFILL))[1]
    if not points:
        assert ws == dense
        return
    rows = -(-n_bins // 32) * 32
    arrays = 2 * padded(8 * heads * rows)
    grids = min(heads, 2 ** 27 // (2048 * points)) * 2048 * points
    tables = padded(80 * (M // points), 16 * (points // 4 + 1), 8 * (points // 4 + 1))
    assert ws - dense == max(grids, arrays) + tables - arrays


def test_query_attn_checks_its_arguments():
    d = desc(M=1024)
    assert B.iwdft_query_attn(d) == B.iwdft_query_attn(d, 16, True) == 0 and B.iwdft_query_attn(desc()) == 1
    for pending in (-1, 17):
        with pytest.raises(B.IwdftError) as e:
            B.iwdft_query_attn(d, pending)
        assert e.value.code == B.IWDFT_ERR_ARG
    lib = B.load_library()
    assert lib.iwdft_query_attn(ctypes.byref(d.c), 0, 0, None) == B.IWDFT_ERR_ARG
    n = ctypes.c_int32()
    assert lib.iwdft_query_attn(None, 0, 0, ctypes.byref(n)) == B.IWDFT_ERR_ARG


@pytest.mark.parametrize("slices,row,group,attend,read,write", [
    (95, 160, 1, 1, 1, 1), (95, 192, 1, 1, 1, 0), (95, 256, 4, 1, 1, 0), (95, 288, 1, 0, 0, 0), (95, 128, 4, 1, 1, 1), (95, 160, 4, 1, 1, 0),  # few
    (95, 128, 8, 1, 1, 0), (95, 160, 8, 0, 0, 0), (96, 256, 8, 1, 1, 1), (96, 256, 1, 1, 1, 1), (513, 256, 1, 1, 0, 0), (513, 160, 1, 1, 1, 1),
    (159, 288, 2, 1, 1, 0), (160, 288, 2, 1, 1, 1), (160, 800, 4, 1, 1, 1), (160, 832, 4, 1, 1, 0), (513, 256, 4, 1, 1, 1),       # written back
    (143, 416, 4, 0, 1, 0), (143, 384, 4, 1, 1, 0), (144, 416, 4, 1, 1, 0), (127, 800, 1, 0, 0, 0), (128, 800, 1, 0, 1, 0),     # read only, long rows
    (256, 1024, 4, 1, 1, 0), (257, 1024, 4, 0, 0, 0), (435, 1024, 4, 0, 0, 0), (436, 1024, 4, 1, 1, 0), (512, 1024, 4, 1, 1, 0),  # by rounds of 512
    (513, 1024, 1, 0, 0, 0), (871, 1024, 1, 1, 1, 0), (307, 768, 2, 0, 0, 0), (308, 768, 2, 1, 1, 0), (614, 544, 4, 0, 0, 0), (615, 544, 4, 1, 1, 0),
    (716, 224, 2, 1, 0, 1), (717, 224, 2, 1, 1, 1), (716, 224, 4, 1, 1, 1), (716, 192, 2, 1, 1, 1), (819, 224, 1, 1, 0, 0), (820, 224, 1, 1, 1, 0), (96, 512, 9, 0, 0, 0),
])
def test_short_contexts_take_one_launch_by_rule(slices, row, group, attend, read, write):
    """Attention alone, a step that only reads with three tokens pending, and one that writes back: one launch (attn_slice_fits) on both sides of every
    line, M = 2048 or, for longer rows, 4096."""
    kw = dict(M=2048 if row <= 512 else 4096, n_layers=1, batch=slices, n_kv_heads=1, n_q_heads=group, bins=[np.arange(row)])
    got = [B.iwdft_query_attn(desc(**kw), *x) == 0 for x in ((0, False), (3, False), (1, True))]
    assert got == [attend, read, write]
    assert B.iwdft_query_attn(desc(**kw, flags=B.IWDFT_FLAG_SERIAL_PHASES)) == 1


@pytest.mark.parametrize("M,n_bins,heads,dtype,logn,period", [
    (62811, 4096, 96, B.IWDFT_BF16, 14, 6979), (62811, 512, 96, B.IWDFT_BF16, 14, 62811),   # 9 even blocks; 8 uneven ones
    (24582, 2048, 8, B.IWDFT_BF16, 14, 12291), (65541, 2048, 8, B.IWDFT_F32, 14, 21847),    # 4 and 9 blocks: two and three of them in common with M
    (14473, 64, 32, B.IWDFT_F32, 11, 14473), (14473, 2000, 96, B.IWDFT_BF16, 14, 14473),    # more blocks on a shorter grid; two
    (37492, 92, 64, B.IWDFT_BF16, 0, 0), (13827, 87, 64, B.IWDFT_BF16, 0, 0), (31870, 200, 64, B.IWDFT_BF16, 14, 15935),  # the contraction; four blocks
])
def test_prefill_of_other_lengths_takes_the_blocks_by_rule(M, n_bins, heads, dtype, logn, period):
    """The workspace holds 1 / W of the grid and ten taps for every frequency up to half a period."""
    kw = dict(M=M, n_layers=1, n_kv_heads=heads, n_q_heads=heads, kv_dtype=dtype, bins=[np.arange(n_bins)])
    ws, dense = (B.iwdft_query_bytes(desc(**kw, flags=f))[1] for f in (0, B.IWDFT_FLAG_DENSE_PREFILL))
    assert ws - dense == (padded(4 * 2 ** logn // 2, 48 * (period // 2 + 1)) if logn else 0)


@pytest.mark.parametrize("M,n_bins,heads,group,low,mixed", [
    (131072, 4096, 8, 4, 8, 16), (131072, 1000, 8, 4, 8, 16), (131072, 4096, 64, 4, 1, 2), (65536, 4096, 8, 4, 4, 8), (65536, 1024, 2, 1, 16, 8),
    (32768, 2048, 8, 4, 1, 4), (32768, 1000, 2, 4, 8, 4), (16384, 1000, 8, 4, 1, 2), (16384, 1000, 128, 2, 1, 1), (262144, 4096, 4, 1, 16, 32),
    (524288, 4096, 4, 1, 64, 64), (3 * 8191, 2000, 8, 4, 3, 3), (8192, 2000, 8, 4, 1, 1),
])
def test_workspace_holds_the_parts_of_a_softmax_and_no_more(M, n_bins, heads, group, low, mixed):
    """Rows and statistics of as many parts as low bins or bins up to M / 2 take, whichever are more (the room does not depend on which bins a
    row of that length holds); IWDFT_FLAG_SERIAL_PHASES, with one part, needs none."""
    kw = dict(M=M, n_layers=1, n_kv_heads=heads, n_q_heads=heads * group)
    for bins, parts in ((np.arange(n_bins), low), (np.r_[np.arange(n_bins - 1), M // 2], mixed)):
        d, serial = desc(bins=[bins], **kw), desc(bins=[bins], **kw, flags=B.IWDFT_FLAG_SERIAL_PHASES)
        assert B.iwdft_query_attn(d) == parts and B.iwdft_query_attn(serial) == 1
        room = max(low, mixed)
        rows = 8 * heads * group * (-(-n_bins // 32) * 32)
        want = padded(rows * room, 16 * heads * ((group + 1) // 2) * room) if room > 1 else 0
        assert B.iwdft_query_bytes(d)[1] - B.iwdft_query_bytes(serial)[1] == want


@pytest.mark.parametrize("kw,code", [
    (dict(n_layers=0, bins=[]), B.IWDFT_ERR_ARG),
    (dict(n_q_heads=3), B.IWDFT_ERR_ARG),
    (dict(kv_dtype=7), B.IWDFT_ERR_ARG),
    (dict(M=0), B.IWDFT_ERR_ARG),
    (dict(M=(1 << 30) + 1), B.IWDFT_ERR_ARG),
    (dict(flags=1 << 20), B.IWDFT_ERR_ARG),
    (dict(write_every=17), B.IWDFT_ERR_ARG),
    (dict(flags=B.IWDFT_FLAG_DENSE_PREFILL | B.IWDFT_FLAG_FFT_PREFILL), B.IWDFT_ERR_ARG),
    (dict(flags=B.IWDFT_FLAG_FFT_PREFILL), B.IWDFT_ERR_UNSUPPORTED),   # M = 64: below the FFT's smallest length
    (dict(flags=B.IWDFT_FLAG_FFT_PREFILL, M=768), B.IWDFT_ERR_UNSUPPORTED),  # not a power of two
    (dict(head_dim=64), B.IWDFT_ERR_UNSUPPORTED),
    (dict(n_sink=-1), B.IWDFT_ERR_ARG),
    (dict(n_recent=-3), B.IWDFT_ERR_ARG),
    (dict(n_sink=1000, n_recent=25), B.IWDFT_ERR_UNSUPPORTED),
    # a long prime M: no O(M log M) attention, too many terms for the direct sums chosen unasked
    (dict(M=1048583, bins=[np.arange(2048), np.arange(8)]), B.IWDFT_ERR_UNSUPPORTED),
    (dict(bins=[np.arange(8), np.array([0, 3, 3, 9])]), B.IWDFT_ERR_BINS),
    (dict(bins=[np.arange(8), np.array([5, 3])]), B.IWDFT_ERR_BINS),
    (dict(bins=[np.arange(8), np.array([0, 64])]), B.IWDFT_ERR_BINS),
    (dict(bins=[np.arange(8), np.array([-1, 2])]), B.IWDFT_ERR_BINS),
    (dict(bins=[np.arange(8), np.zeros(0, np.int32)]), B.IWDFT_ERR_BINS),
    (dict(bins=[np.arange(8), np.arange(4)], bin_weights=[np.ones(8), np.array([1, np.nan, 1, 1])]),
     B.IWDFT_ERR_BINS),
])
def test_bad_descriptors_are_rejected(kw, code):
    with pytest.raises(B.IwdftError) as e:
        B.iwdft_query_bytes(desc(**kw))
    assert e.value.code == code
    assert B.iwdft_last_error()


def test_null_pointers_and_null_ctx():
    lib = B.load_library()
    assert lib.iwdft_query_bytes(None, None, None) == B.IWDFT_ERR_ARG
    s = ctypes.c_size_t()
    assert lib.iwdft_query_bytes(None, ctypes.byref(s), ctypes.byref(s)) == B.IWDFT_ERR_ARG
    assert lib.iwdft_num_tokens(None) == -1
    assert lib.iwdft_destroy(None) == B.IWDFT_OK
    assert lib.iwdft_set_num_tokens(None, 5) == B.IWDFT_ERR_ARG
    assert lib.iwdft_prefill_kind(None) == -1
    assert lib.iwdft_attn_kind(None) == -1
    assert lib.iwdft_attn_pipelined(None) == -1
    assert lib.iwdft_flush(None, None) == B.IWDFT_ERR_ARG
    assert lib.iwdft_phase_timing(None, 1) == B.IWDFT_ERR_ARG
    ms, n = (ctypes.c_double * 3)(), ctypes.c_int64()
    assert lib.iwdft_phase_times(None, ms, ctypes.byref(n)) == B.IWDFT_ERR_ARG
    d = desc()
    out = ctypes.c_void_p()
    assert lib.iwdft_create(ctypes.byref(d.c), None, 0, None, 0, ctypes.byref(out)) == B.IWDFT_ERR_ARG
    assert lib.iwdft_create(ctypes.byref(d.c), None, 0, None, 0, None) == B.IWDFT_ERR_ARG


def test_workspace_holds_the_deferred_tokens():
    bins = [np.arange(40), np.arange(40)]
    ws1 = B.iwdft_query_bytes(desc(M=1024, bins=bins))[1]
    ws8 = B.iwdft_query_bytes(desc(M=1024, bins=bins, write_every=8))[1]
    # 8 rows of 128 bf16 for K and for V per slice, and 16 floats per (slice, query head)
    assert ws8 - ws1 >= 2 * (4 * 8 * 128 * 2) + 4 * 2 * 16 * 4
    # M = 64 has no FFT attention path, so nothing is deferred and nothing is reserved
    assert B.iwdft_query_bytes(desc(write_every=8))[1] == B.iwdft_query_bytes(desc())[1]


@pytest.mark.parametrize("heads,layers,n_bins,deferred", [
    (2, 2, 250, True), (3, 2, 250, False), (8, 2, 250, False),    # 2 x 2 slices x 256 rows
    (3, 96, 250, True), (8, 96, 250, True), (4, 95, 250, False),  # 49152 rows; one layer fewer
])
def test_chirp_contexts_defer_where_it_is_faster(heads, layers, n_bins, deferred):
    """M = 1000: up to two query heads per KV head always, more from 49152 coefficient rows on (the workspace tells)."""
    kw = dict(M=1000, n_layers=layers, n_q_heads=2 * heads, bins=[np.arange(n_bins)] * layers)
    ws1, ws8 = B.iwdft_query_bytes(desc(**kw))[1], B.iwdft_query_bytes(desc(write_every=8, **kw))[1]
    assert (ws8 - ws1 >= 2 * (2 * layers * 8 * 128 * 2)) == deferred and (ws8 == ws1) == (not deferred)


def test_query_bytes_grows_with_exact_windows():
    s0, w0 = B.iwdft_query_bytes(desc())
    s1, w1 = B.iwdft_query_bytes(desc(n_sink=10, n_recent=50))
    # 4 slices x (10 + 50) tokens x 128 channels x 2 B (bf16), K and V
    assert s1 - s0 >= 2 * 4 * 60 * 128 * 2 and s1 - s0 < 2 * 4 * 60 * 128 * 2 + 2048
    assert w1 > w0


def test_static_scratch_symbol_is_visible_to_the_hip_runtime(tmp_path):
    """The HIP runtime finds a registered device variable by name in the code object and aborts the process
    when it is missing, so the library's file-scope scratch array must be a GLOBAL symbol of the device code."""
    import shutil
    import subprocess
    obj = os.path.join(os.path.dirname(B.LIB_PATH), "_build", "api.o")
    tools = "/opt/rocm/llvm/bin"
    if not (os.path.exists(obj) and os.path.exists(f"{tools}/clang-offload-bundler") and shutil.which("objcopy")):
        pytest.skip("object file or LLVM tools not available")
    fat, co = str(tmp_path / "fat.bin"), str(tmp_path / "dev.co")
    subprocess.run(["objcopy", "-O", "binary", "--only-section=.hip_fatbin", obj, fat], check=True)
    subprocess.run([f"{tools}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--output={co}"], check=True)
    syms = subprocess.run([f"{tools}/llvm-readelf", "-s", co], check=True, capture_output=True, text=True).stdout
    rows = [ln.split() for ln in syms.splitlines() if ln.strip().endswith("scratch")]
    assert rows, "no scratch symbol in the device code object"
    assert all(r[4] == "GLOBAL" and int(r[2]) == B.IWDFT_STATIC_SCRATCH_BYTES for r in rows), rows


def test_plan_accepts_long_contexts_with_a_small_divisor_and_the_direct_sums_on_request():
    # 2^20 - 64 = 129 * 8128: 129 decimated blocks of 8128 points (chirp-z); a long prime is accepted when the caller
    # insists on the direct sums
    big = [np.arange(2048), np.arange(8)]
    assert B.iwdft_query_bytes(desc(M=(1 << 20) - 64 * 1, bins=big))[0] > 0
    assert B.iwdft_query_bytes(desc(M=1048583, bins=big, flags=B.IWDFT_FLAG_DIRECT_SYNTHESIS))[0] > 0
    assert B.iwdft_query_bytes(desc(M=10007, bins=big))[0] > 0      # 10007 * 2048 terms: the direct sums are fine


def test_dynamic_lds_is_declared_for_16_byte_accesses():
    """Static arrays are placed in front of dynamic LDS: without the attribute its start is only as aligned as its element."""
    csrc = os.path.join(ROOT, "paper_2507_20030_amd", "csrc")
    found = 0
    for name in sorted(os.listdir(csrc)):
        for line in open(os.path.join(csrc, name)):
            if "extern __shared__" in line:
                found += 1
                assert "__attribute__((aligned(16)))" in line, (name, line.strip())
    assert found >= 8
