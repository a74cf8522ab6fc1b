"""Host-only checks of the C-ABI library: it loads without a GPU, exports every symbol the
header declares, and rejects bad arguments before touching the device."""
import ctypes
import os
import re
import shutil
import subprocess

import pytest
import torch

from paper_2508_20407_amd import binding as b

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(not os.path.exists(b.LIB_PATH), reason="libtlinattn.so not built")


def header_symbols():
    syms = set()
    for name in sorted(os.listdir(os.path.join(ROOT, "include"))):
        if not name.endswith(".h"):
            continue
        text = open(os.path.join(ROOT, "include", name)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        syms |= set(re.findall(r"\b(tlin_[a-z_]+)\s*\(", text))
    return sorted(syms)


def test_library_exports_every_declared_symbol():
    syms = header_symbols()
    assert set(syms) == set(b.EXPORTS)
    L = b.lib()
    for s in syms:
        assert getattr(L, s) is not None


def test_version_and_status_strings():
    assert b.version() >= 100
    seen = {b.status_string(i) for i in range(5)}
    assert len(seen) == 5 and b.status_string(0) == "ok"
    assert b.status_string(99) == "unknown status"


def test_params_struct_matches_header_layout():
    # 10 four-byte fields, then six int64[3] arrays aligned to 8
    assert ctypes.sizeof(b.TlinParams) == 40 + 6 * 24
    assert b.TlinParams.q_stride.offset == 40 and b.TlinParams.o_stride.offset == 40 + 5 * 24


def P(**kw):
    d = dict(B=1, H=2, W=64, N=1024, D=64, in_dtype=b.TLIN_BF16, out_dtype=b.TLIN_BF16, scale=0.125)
    d.update(kw)
    return b.make_params(**d)


def test_workspace_and_split_planning_is_pure_host_arithmetic():
    p = P(B=1, H=32, W=512, N=131072, D=128)
    s = b.num_splits(p)
    assert s >= 1
    need = b.workspace_bytes(p)
    rows = 32 * (s + 1) * 512
    assert need == rows * 128 * 4 + 2 * rows * 4
    assert b.num_splits(P(num_splits=4)) == 4
    assert b.num_splits(P(num_splits=5)) == 4      # 16 tiles: 4 per partition, none empty
    assert b.num_splits(P(num_splits=10 ** 6)) == 1024 // 64   # one 64-key tile per partition at most
    assert b.num_splits(P(N=1)) == 1
    assert b.workspace_bytes(P(W=0)) == 0 and b.num_splits(P(D=30)) == 0


A = 1 << 20   # a fake, suitably aligned device address: validation must fail before it is used


@pytest.mark.parametrize("kw,status", [
    (dict(B=0), b.TLIN_ERR_INVALID_ARG), (dict(H=-1), b.TLIN_ERR_INVALID_ARG), (dict(W=0), b.TLIN_ERR_INVALID_ARG),
    (dict(N=0), b.TLIN_ERR_INVALID_ARG), (dict(D=30), b.TLIN_ERR_UNSUPPORTED), (dict(D=256), b.TLIN_ERR_UNSUPPORTED), (dict(D=0), b.TLIN_ERR_UNSUPPORTED), (dict(D=4), b.TLIN_ERR_UNSUPPORTED),
    (dict(D=36), b.TLIN_ERR_INVALID_ARG),                                      # dense bf16 rows of 72 bytes
    (dict(in_dtype=7), b.TLIN_ERR_INVALID_ARG), (dict(out_dtype=-1), b.TLIN_ERR_INVALID_ARG),
    (dict(scale=0.0), b.TLIN_ERR_INVALID_ARG), (dict(scale=float("nan")), b.TLIN_ERR_INVALID_ARG),
    (dict(scale=float("inf")), b.TLIN_ERR_INVALID_ARG), (dict(num_splits=-2), b.TLIN_ERR_INVALID_ARG),
    (dict(N=(1 << 30) + 1), b.TLIN_ERR_INVALID_ARG), (dict(W=(1 << 30) + 64), b.TLIN_ERR_INVALID_ARG),   # beyond 32-bit tile arithmetic
    (dict(kh_stride=(0, 0, 1 << 24)), b.TLIN_ERR_INVALID_ARG),                 # row stride of 32 MiB
    (dict(q_stride=(64 * 64 * 2, 64 * 64, 60)), b.TLIN_ERR_INVALID_ARG),       # row stride < D
    (dict(kh_stride=(1024 * 68 * 2, 1024 * 68, 68)), b.TLIN_ERR_INVALID_ARG),  # rows not 16-byte aligned
])
def test_history_rejects_bad_params(kw, status):
    assert b.history_attn_raw(P(**kw), A, A, A, A, None, A, 1 << 30, None) == status


def test_other_head_dimensions_run_in_the_next_native_size():
    # rows padded to whole 16-byte pieces are accepted; the workspace is sized for the kernel's 64 / 128 columns
    st40 = lambda rows: (2 * rows * 40, rows * 40, 40)
    p36 = P(D=36, q_stride=st40(64), kh_stride=st40(1024), vh_stride=st40(1024), kw_stride=st40(64), vw_stride=st40(64),
            o_stride=st40(64))
    assert b.num_splits(p36) == b.num_splits(P()) and b.workspace_bytes(p36) == b.workspace_bytes(P())
    p96 = P(D=96)
    assert b.workspace_bytes(p96) == b.workspace_bytes(P(D=128))
    # fp32 rows of 36 floats are whole pieces already
    assert b.num_splits(P(D=36, in_dtype=b.TLIN_F32, out_dtype=b.TLIN_F32)) >= 1
    # a row stride that cannot hold the last piece
    bad = P(D=36, q_stride=(2 * 64 * 36, 64 * 36, 36))
    assert b.history_attn_raw(bad, A, A, A, A, None, A, 1 << 30, None) == b.TLIN_ERR_INVALID_ARG


def test_null_and_misaligned_pointers_and_workspace():
    p = P()
    assert b.num_splits(p) > 1
    big = 1 << 30
    assert b.history_attn_raw(p, None, A, A, A, None, A, big, None) == b.TLIN_ERR_INVALID_ARG
    assert b.history_attn_raw(p, A, A, None, A, None, A, big, None) == b.TLIN_ERR_INVALID_ARG
    assert b.history_attn_raw(p, A, A, A, None, None, A, big, None) == b.TLIN_ERR_INVALID_ARG
    assert b.history_attn_raw(p, A + 2, A, A, A, None, A, big, None) == b.TLIN_ERR_INVALID_ARG
    assert b.history_attn_raw(p, A, A, A, A, None, None, 0, None) == b.TLIN_ERR_WORKSPACE
    assert b.history_attn_raw(p, A, A, A, A, None, A, 16, None) == b.TLIN_ERR_WORKSPACE
    assert b.history_attn_raw(p, A, A, A, A, None, A + 16, big, None) == b.TLIN_ERR_WORKSPACE
    assert b.window_causal_attn_raw(p, A, None, A, A, None, None, 0, None) == b.TLIN_ERR_INVALID_ARG
    assert b.layer_attn_raw(p, A, A, A, A, A, A, None, 0, None) == b.TLIN_ERR_WORKSPACE
    assert b.layer_attn_raw(p, A, None, A, A, A, A, A, big, None) == b.TLIN_ERR_INVALID_ARG
    assert b.layer_attn_raw(P(combine=3), A, A, A, A, A, A, A, big, None) == b.TLIN_ERR_INVALID_ARG
    assert b.layer_attn_raw(P(N=-1), A, A, A, A, A, A, A, big, None) == b.TLIN_ERR_INVALID_ARG


@pytest.mark.skipif(torch.cuda.is_available(), reason="the accepted calls would run on fake addresses")
@pytest.mark.parametrize("kw,bytes_for", [
    (dict(H=8, W=1, N=4096, num_splits=1), 0),             # one partition, asked for
    (dict(H=8, W=2, N=4096, D=96, num_splits=1), 0),
    (dict(B=25, H=32, W=1, N=4096), 0), (dict(B=25, H=32, W=1, N=1100, D=96), 0),   # one partition: the heads alone fill the chip
    (dict(H=12, W=1, N=100000), 63),                       # the matrix-core path's partitions and no more
])
def test_history_calls_of_few_rows_keep_to_the_workspace_of_the_matrix_core_path(kw, bytes_for):
    """One or two bf16 rows at head dimensions below 128: what the matrix-core path needs is enough (nothing
    for a single partition), whichever kernel runs when the whole of tlin_workspace_bytes is there."""
    p = P(**kw)
    need = p.B * p.H * bytes_for * p.W * ((64 if p.D <= 64 else 128) * 4 + 8)
    assert need < b.workspace_bytes(p)
    ws = A if need else None
    # every argument check is passed: the first thing that fails is the missing device
    assert b.history_attn_raw(p, A, A, A, A, None, ws, need, None) == b.TLIN_ERR_HIP
    if not need:                # a workspace that is not used is not looked at
        assert b.history_attn_raw(p, A, A, A, A, None, None, 1 << 30, None) == b.TLIN_ERR_HIP
        assert b.history_attn_raw(p, A, A, A, A, None, A + 16, 1 << 30, None) == b.TLIN_ERR_HIP
    if need:
        assert b.history_attn_raw(p, A, A, A, A, None, ws, need - 1, None) == b.TLIN_ERR_WORKSPACE
        assert b.history_attn_raw(p, A, A, A, A, None, None, need, None) == b.TLIN_ERR_WORKSPACE
        assert b.history_attn_raw(p, A, A, A, A, None, A + 16, need, None) == b.TLIN_ERR_WORKSPACE
    # where the streaming kernel is the only path its workspace is still asked for
    assert b.history_attn_raw(P(D=128, W=1, N=4096, num_splits=1), A, A, A, A, None, None, 0, None) == b.TLIN_ERR_WORKSPACE


@pytest.mark.parametrize("H,W,N,D,matrix,stream,streams", [
    (12, 1, 99991, 36, 63, 83, True), (12, 2, 99991, 36, 63, 83, False),           # one row, two rows
    (32, 1, 300001, 48, 24, 32, False), (32, 1, 65000, 48, 24, 32, True),          # 1.8 GB, 0.4 GB
    (32, 1, 300001, 32, 24, 32, True), (12, 2, 300001, 32, 64, 85, False),         # 64 bytes of columns
    (100, 1, 19737, 68, 6, 10, True), (100, 2, 75005, 68, 6, 10, True),            # 600 workgroups on 512 places
    (100, 2, 75005, 36, 8, 10, True), (100, 2, 75005, 32, 8, 10, False),           # 800 on 768
    (128, 1, 30000, 68, 4, 8, False),                                              # 512 on 512
])
def test_streaming_kernel_of_short_bf16_rows_runs_where_it_is_ahead(H, W, N, D, matrix, stream, streams):
    """Both sides of the lines between the two paths, seen by the number of partitions each cuts."""
    row = -(-D // 8) * 8
    st = lambda rows: (H * rows * row, rows * row, row)
    p = P(H=H, W=W, N=N, D=D, q_stride=st(W), kh_stride=st(N), vh_stride=st(N), o_stride=st(W))
    assert b.num_splits(p) == (stream if streams else matrix)
    # layer calls never stream: their workspace holds the matrix-core path's partitions and the window's
    assert b.workspace_bytes(p) == H * max(matrix + 1, stream if streams else 0) * W * ((64 if D <= 64 else 128) * 4 + 8)


def test_static_workspace_entry_point_checks_arguments_and_its_limit_on_the_host():
    p = P()
    assert b.layer_attn_static_ws_raw(p, None, A, A, A, A, A, None) == b.TLIN_ERR_INVALID_ARG
    assert b.layer_attn_static_ws_raw(P(combine=3), A, A, A, A, A, A, None) == b.TLIN_ERR_INVALID_ARG
    assert b.layer_attn_static_ws_raw(P(W=0), A, A, A, A, A, A, None) == b.TLIN_ERR_INVALID_ARG
    # a workspace need beyond the array's size is refused before any device call
    big = P(B=4, H=32, W=512, N=131072, D=128)
    assert b.workspace_bytes(big) > b.STATIC_WS_BYTES
    assert b.layer_attn_static_ws_raw(big, A, A, A, A, A, A, None) == b.TLIN_ERR_WORKSPACE
    # the largest fixed workload fits
    assert b.workspace_bytes(P(B=1, H=32, W=512, N=131072, D=128)) <= b.STATIC_WS_BYTES
    text = open(os.path.join(ROOT, "include", "tlinattn.h")).read()
    assert "#define TLIN_STATIC_WS_BYTES ((size_t)64 << 20)" in text and b.STATIC_WS_BYTES == 64 << 20


@pytest.mark.parametrize("W", [65, 100, 128, 200])
@pytest.mark.parametrize("D", [16, 64])
def test_calls_of_many_heads_are_not_cut_out_of_the_static_workspace(W, D):
    """fp32 layer calls that fit the library's own array in one partition are not refused for their second one."""
    seen = 0
    for H in range(8, 1601, 8):
        for N in (300, 20000, 200000):
            p = P(H=H, W=W, N=N, D=D, in_dtype=b.TLIN_F32, out_dtype=b.TLIN_F32)
            if H * W * 2 * (64 * 4 + 8) <= b.STATIC_WS_BYTES:        # one partition and the window
                assert b.workspace_bytes(p) <= b.STATIC_WS_BYTES, (H, N)
                seen += 1
    assert seen > 100


def test_slide_planning_and_argument_checks():
    # 256 chunks of 512 rows, 32 heads: plenty of work items, so one partition per chunk history
    # plus the window partial = 2 fp32 partial slots per output row
    p = P(B=1, H=32, W=512, N=131072, D=128)
    rows = 32 * 256 * 2 * 512
    assert b.slide_workspace_bytes(p) == rows * 128 * 4 + 2 * rows * 4
    # a short sequence is split further; the ragged last chunk still gets whole slots
    small = P(B=1, H=1, W=128, N=1000, D=64)
    need = b.slide_workspace_bytes(small)
    per_slot = 128 * 64 * 4 + 2 * 128 * 4
    assert need % (8 * per_slot) == 0 and need // (8 * per_slot) >= 2
    forced = P(B=1, H=1, W=128, N=1000, D=64, num_splits=3)
    assert b.slide_workspace_bytes(forced) == 8 * 4 * per_slot
    assert b.slide_workspace_bytes(P(N=0)) == 0 and b.slide_workspace_bytes(P(D=130)) == 0
    big = 1 << 40
    assert b.slide_layer_attn_raw(P(N=0), A, A, A, A, A, A, A, big, None) == b.TLIN_ERR_INVALID_ARG
    assert b.slide_layer_attn_raw(P(combine=2), A, A, A, A, A, A, A, big, None) == b.TLIN_ERR_INVALID_ARG
    assert b.slide_layer_attn_raw(p, A, A, None, A, A, A, A, big, None) == b.TLIN_ERR_INVALID_ARG
    assert b.slide_layer_attn_raw(p, A, A, A, A, A + 4, A, A, big, None) == b.TLIN_ERR_INVALID_ARG
    assert b.slide_layer_attn_raw(p, A, A, A, A, A, A, None, 0, None) == b.TLIN_ERR_WORKSPACE
    assert b.slide_layer_attn_raw(p, A, A, A, A, A, A, A, 1 << 20, None) == b.TLIN_ERR_WORKSPACE


@pytest.mark.skipif(shutil.which("nm") is None, reason="nm not found")
def test_no_kernel_is_compiled_that_the_dispatch_cannot_reach():
    """Non-temporal tile loads are for histories only, the log-sum-exp variants for causal kernels only."""
    names = subprocess.run(["nm", "-C", b.LIB_PATH], capture_output=True, text=True, check=True).stdout
    kernels = {tuple(k.split(", ")) for k in re.findall(r"attn_bf16_kernel<([^>]*)>", names)}
    assert len(kernels) >= 20
    assert set(re.findall(r"\b(attn_\w+_kernel)\b", names)) == {"attn_bf16_kernel", "attn_bf16_pair_kernel", "attn_bf16_resident_pipe_kernel",
                                                              "attn_f32_kernel", "attn_f32_pair_kernel"}
    for d, nw, qb, causal, nstage, resident, columns, nt, lse in kernels:
        assert not (causal == "true" and nt == "true"), (d, nw, columns)
        assert lse == "false" or (causal == "true" and d == "64"), (d, nw, columns)


LLVM = "/opt/rocm/llvm/bin"


@pytest.mark.skipif(not all(os.path.exists(f"{LLVM}/{t}") for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf")), reason="ROCm's LLVM tools not found")
def test_registers_spilled(tmp_path):
    """No bf16 kernel spills; the fp32 ones a few registers (at most 18 are)."""
    fat, code = str(tmp_path / "fat"), str(tmp_path / "code")
    subprocess.run([f"{LLVM}/llvm-objcopy", "-O", "binary", "--only-section=.hip_fatbin", b.LIB_PATH, fat], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                    f"--input={fat}", f"--output={code}"], check=True)
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", code], capture_output=True, text=True, check=True).stdout
    kernels = dict(re.findall(r"\.name:\s+(_ZN4tlin\S+).*?\.vgpr_spill_count:\s+(\d+)", notes, flags=re.S))
    assert len(kernels) > 100
    spilled = {k: int(n) for k, n in kernels.items() if int(n)}
    assert all("attn_f32" in k for k in spilled) and max(spilled.values(), default=0) <= 20, spilled


def test_inline_assembly_loads_no_registers():
    """The compiler takes the output of an assembly load as there at once: only the direct loads into LDS,
    whose arrival is waited for by hand, are written that way."""
    csrc = os.path.join(ROOT, "paper_2508_20407_amd", "csrc")
    found = 0
    for name in sorted(os.listdir(csrc)):
        source = open(os.path.join(csrc, name)).read().replace("\\n", " ").replace("\\t", " ")
        for text in re.findall(r"asm volatile\((.*?)\);", source, flags=re.S):
            for op in re.findall(r"\b(?:ds_read|ds_load|global_load|buffer_load|flat_load|scratch_load|s_load)\w*[^\"]*", text):
                assert op.startswith("buffer_load") and op.rstrip().endswith(" lds"), (name, op)
                found += 1
    assert found == 2


def test_binding_fails_loudly_when_library_is_missing(monkeypatch):
    monkeypatch.setattr(b, "_lib", None)
    monkeypatch.setattr(b, "LIB_PATH", "/nonexistent/libtlinattn.so")
    with pytest.raises(ImportError, match="no fallback"):
        b.lib()
