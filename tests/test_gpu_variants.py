"""GPU parity at the edges of the kernels' size classes: every kernel variant that the host's dispatch
chooses by size, at the smallest and largest size of its class, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import tlin_inputs as ti
import paper_2508_20407_amd as tl
from helpers import assert_close, f32_rel_bound, to_host64
from test_gpu_parity import padded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [28, 32, 36, 48, 52, 68, 96, 100])
@pytest.mark.parametrize("W,N", [(40, 1300), (161, 700), (257, 2100)])
def test_columns_computed_and_waves_without_rows(D, W, N):
    """bf16 at both sides of the column counts that have a kernel of their own (32, 48, 64, 96, 128), with
    windows that leave the last waves of a workgroup without rows: history, window and both layers."""
    w = ti.Workload(f"columns_{D}_{W}_{N}", 1, 2, D, N, W, ti.BF16, 1.0, 2468 + D + 7 * W + N)
    host = ti.make(w)
    dev = {k: padded(v, w.dtype) for k, v in host.items()}
    o, lse = tl.tlin_history_attn(dev["Q"], dev["Kh"], dev["Vh"], scale=w.scale, return_lse=True)
    ro, rl = oracle.history(host["Q"], host["Kh"], host["Vh"], w.dtype, w.scale)
    assert_close(o, ro, w.dtype, f"{w.name} history")
    # these shapes sum the fp32 weights: exact to fp32 rounding of scores of this size (a key that is lost or
    # counted twice among 2100 is 5e-4)
    np.testing.assert_allclose(lse.cpu().numpy(), rl, rtol=1e-5, atol=1e-5)
    o = tl.tlin_window_causal_attn(dev["Q"], dev["Kw"], dev["Vw"], scale=w.scale)
    ro, _ = oracle.window_causal(host["Q"], host["Kw"], host["Vw"], w.dtype, w.scale)
    assert_close(o, ro, w.dtype, f"{w.name} window")
    for mode, omode in ((tl.TLIN_COMBINE_SUM, oracle.SUM), (tl.TLIN_COMBINE_JOINT, oracle.JOINT)):
        o = tl.tlin_layer_attn(dev["Q"], dev["Kh"], dev["Vh"], dev["Kw"], dev["Vw"], combine=mode, scale=w.scale)
        ro = oracle.layer(host["Q"], host["Kh"], host["Vh"], host["Kw"], host["Vw"], w.dtype, w.scale, omode)
        assert_close(o, ro, w.dtype, f"{w.name} layer mode {mode}")


def mirrored_heads(heads, W):
    """Heads (of batch * heads) whose blocks run from the short end, in four-wave workgroups of 128 rows: more
    than one and up to two to a compute unit, whole heads to an XCD, those behind the XCD's first 32 blocks."""
    blocks = -(-W // 128)
    if not 256 < heads * blocks <= 512 or heads % 8:
        return set()
    return {h for h in range(heads) if (h % (heads // 8) * blocks) >> 5 & 1}


@pytest.mark.parametrize("B,H,D,W,mirrored", [
    (1, 16, 64, 2050, False), (1, 16, 128, 2110, False), (2, 12, 36, 1409, False), (1, 8, 128, 4097, False), (1, 128, 128, 2049, False),
    (1, 16, 128, 4096, True), (1, 16, 64, 4001, True), (1, 32, 64, 2048, True), (1, 32, 36, 2000, True), (2, 12, 100, 2500, True),
    (4, 16, 48, 1000, True)])
def test_causal_workgroup_shapes_and_order(B, H, D, W, mirrored):
    """Causal windows at both sides of the lines between workgroup shapes and block orders (two four-wave
    workgroups per compute unit with the heads behind the first 32 of an XCD mirrored; more than two; eight
    waves): every row of a few heads, mirrored ones and others among them, against the fp64 oracle."""
    w = ti.Workload(f"causal_{B}_{H}_{D}_{W}", B, H, D, 1, W, ti.BF16, 1.0, 97531 + H + D + W)
    heads = sorted({0, 1, H // 2, H // 2 + 1, H - 1})
    run_short = {(B - 1) * H + h for h in heads} & mirrored_heads(B * H, W)
    assert (0 < len(run_short) < len(heads)) if mirrored else not mirrored_heads(B * H, W)
    host = ti.make(w)
    dev = {k: padded(host[k], w.dtype) for k in ("Q", "Kw", "Vw")}
    o = tl.tlin_window_causal_attn(dev["Q"], dev["Kw"], dev["Vw"], scale=w.scale)
    for h in heads:
        sub = [np.ascontiguousarray(host[k][B - 1:, h:h + 1]) for k in ("Q", "Kw", "Vw")]
        ro, _ = oracle.window_causal(*sub, w.dtype, w.scale)
        assert_close(o[B - 1:, h:h + 1], ro, w.dtype, f"{w.name} head {h}")


@pytest.mark.parametrize("D", [8, 20, 36, 64, 68, 100, 124])
@pytest.mark.parametrize("B,H,W,N,splits", [(2, 3, 1, 1024, 5), (2, 3, 1, 1087, 5), (2, 3, 1, 5003, 7), (4, 25, 1, 4099, 11), (4, 25, 2, 4099, 11)])
def test_cache_hit_rows_of_every_length(D, B, H, W, N, splits):
    """The streaming kernel over bf16 rows shorter than its own (one piece, whole and cut last pieces),
    with ragged partitions, against the fp64 oracle; its weights and row sums are fp32, so outputs and
    log-sum-exp hold to fp32 rounding.  Two rows of up to 32 columns stay on the matrix-core path, whose
    weights are bf16."""
    w = ti.Workload(f"cache_hit_{D}_{B}_{H}_{W}_{N}", B, H, D, N, W, ti.BF16, 1.0, 1357 + D + 7 * W + N)
    host = ti.make(w)
    dev = {k: padded(host[k], w.dtype) for k in ("Q", "Kh", "Vh")}
    sub = [0, H // 2, H - 1]
    ro, rl = oracle.history(*(np.ascontiguousarray(host[k][B - 1:, sub]) for k in ("Q", "Kh", "Vh")), w.dtype, w.scale)
    for s in (0, splits):
        o, lse = tl.tlin_history_attn(dev["Q"], dev["Kh"], dev["Vh"], scale=w.scale, return_lse=True, num_splits=s)
        assert_close(o[B - 1:, sub], ro, w.dtype, f"{w.name} splits {s}")
        np.testing.assert_allclose(lse[B - 1:, sub].cpu().numpy(), rl, rtol=1e-5, atol=1e-5)
        o = tl.tlin_history_attn(dev["Q"], dev["Kh"], dev["Vh"], scale=w.scale, out_dtype=torch.float32, num_splits=s)
        assert_close(o[B - 1:, sub], ro, ti.F32 if W == 1 or D > 32 else w.dtype, f"{w.name} splits {s} f32 out")


@pytest.mark.parametrize("D,H,W", [(64, 3, 5), (128, 3, 5), (36, 16, 40), (128, 16, 32), (64, 27, 19), (100, 19, 27)])
@pytest.mark.parametrize("parts", [2, 5, 6, 7, 15, 16, 17, 31, 32, 33, 40, 75, 150])
def test_merge_partition_counts(D, H, W, parts):
    """The merge at both sides of the lines between its thread counts (6, 16 and 32 partials, the joint layer's
    window being one more; 512 and 513 rows), whole and cut batches of four: history with log-sum-exp and
    the joint layer."""
    w = ti.Workload(f"merge_{D}_{H}_{W}_{parts}", 1, H, D, 64 * parts, W, ti.F32, 1.0, 8642 + D + H + W + parts)
    assert tl.binding.num_splits(tl.binding.make_params(1, H, W, w.N, D, 0, 0, w.scale, parts)) == parts
    host = ti.make(w)
    dev = {k: padded(v, w.dtype) for k, v in host.items()}
    ro, rl = oracle.history(host["Q"], host["Kh"], host["Vh"], w.dtype, w.scale)
    rj = oracle.layer(host["Q"], host["Kh"], host["Vh"], host["Kw"], host["Vw"], w.dtype, w.scale, oracle.JOINT)
    o, lse = tl.tlin_history_attn(dev["Q"], dev["Kh"], dev["Vh"], scale=w.scale, return_lse=True, num_splits=parts)
    assert_close(o, ro, w.dtype, f"{w.name} history")
    np.testing.assert_allclose(lse.cpu().numpy(), rl, rtol=1e-5, atol=1e-5)
    o = tl.tlin_layer_attn(dev["Q"], dev["Kh"], dev["Vh"], dev["Kw"], dev["Vw"], combine=tl.TLIN_COMBINE_JOINT,
                           scale=w.scale, num_splits=parts)
    assert_close(o, rj, w.dtype, f"{w.name} joint")


def rides_on_partition_0(dtype, D, heads, W, tiles, parts):
    """The rule by which partition 0 of a layer call's history also takes the window block: the partitions are
    longer than the block (where the chip does not hold the window blocks beside the history blocks; four
    times as long otherwise), and number at most the square root of the tiles."""
    rows = 128 if dtype == ti.BF16 and D <= 64 else 256                 # windows of more than 128 rows
    places = 768 if rows == 128 else 256
    blocks = -(-W // rows)
    wt = -(-W // (64 if dtype == ti.BF16 else 32))
    cost = (wt * 5 // 4 if dtype == ti.BF16 else wt) + 2
    full = heads * blocks * (parts + 1) > places
    return parts >= 2 and tiles >= parts * parts and tiles // parts >= (cost + 2 if full else 4 * cost)


@pytest.mark.parametrize("dtype,D", [(ti.F32, 128), (ti.F32, 64), (ti.BF16, 128), (ti.BF16, 100), (ti.BF16, 64), (ti.BF16, 36)])
@pytest.mark.parametrize("W,heads,parts", [(161, 96, 4), (257, 64, 5), (257, 4, 2)])
def test_window_block_in_short_partitions(dtype, D, W, heads, parts):
    """Layer calls around the shortest partition whose workgroup also takes the window block: the shortest
    history for which it does and one key tile less, in ragged tiles, with waves (the last workgroup's) that own
    no rows, for full and for mostly empty chips."""
    tile = 64 if dtype == ti.BF16 else 32
    tiles = next(t for t in range(parts, 10 ** 4) if rides_on_partition_0(dtype, D, heads, W, t, parts))
    for t in (tiles, tiles - 1):
        assert rides_on_partition_0(dtype, D, heads, W, t, parts) == (t == tiles)
        w = ti.Workload(f"short_partitions_{dtype}_{D}_{t}_{W}", 1, heads, D, tile * t - 5, W, dtype, 1.0, 7531 + D + t + W)
        p = tl.binding.make_params(1, heads, W, w.N, D, dtype, dtype, w.scale, parts)
        assert tl.binding.num_splits(p) == parts
        host = ti.make(w)
        dev = {k: padded(v, w.dtype) for k, v in host.items()}
        sub = [0, heads // 2, heads - 1]
        cut = [np.ascontiguousarray(host[k][:, sub]) for k in ("Q", "Kh", "Vh", "Kw", "Vw")]
        for mode, omode in ((tl.TLIN_COMBINE_SUM, oracle.SUM), (tl.TLIN_COMBINE_JOINT, oracle.JOINT)):
            o = tl.tlin_layer_attn(dev["Q"], dev["Kh"], dev["Vh"], dev["Kw"], dev["Vw"], combine=mode, scale=w.scale, num_splits=parts)
            assert_close(o[:, sub], oracle.layer(*cut, w.dtype, w.scale, omode), w.dtype, f"{w.name} mode {mode}")
        o = tl.tlin_window_causal_attn(dev["Q"], dev["Kw"], dev["Vw"], scale=w.scale)
        ro, _ = oracle.window_causal(cut[0], cut[3], cut[4], w.dtype, w.scale)
        assert_close(o[:, sub], ro, w.dtype, f"{w.name} window")


@pytest.mark.parametrize("H,W,D,N,splits,parts", [(8, 1, 36, 4100, 1, 0), (8, 2, 96, 1500, 1, 0), (800, 1, 64, 1025, 0, 0), (600, 2, 80, 1025, 0, 0),
                                                 (12, 1, 36, 20000, 0, 35), (12, 1, 36, 20000, 7, 7)])
def test_few_rows_with_the_workspace_of_the_matrix_core_path(H, W, D, N, splits, parts):
    """History calls of one or two bf16 rows that bring no workspace (a single partition) or one that holds the
    matrix-core path's partials only, with the log-sum-exp, against the oracle; nothing behind it is written."""
    w = ti.Workload(f"few_rows_{H}_{W}_{D}_{N}", 1, H, D, N, W, ti.BF16, 1.0, 2244 + H + D + N)
    host = ti.make(w)
    dev = {k: padded(host[k], w.dtype) for k in ("Q", "Kh", "Vh")}
    o = torch.empty((1, H, W, -(-D // 8) * 8), dtype=torch.bfloat16, device="cuda")[..., :D]
    lse = torch.empty((1, H, W), dtype=torch.float32, device="cuda")
    p = tl.params_for(dev["Q"], N, None, w.scale, splits, kh=dev["Kh"], vh=dev["Vh"], o=o)
    need = H * parts * W * ((64 if D <= 64 else 128) * 4 + 8)
    ws = torch.full((need + 512,), 0xA5, dtype=torch.uint8, device="cuda")
    assert ws.data_ptr() % 256 == 0
    st = tl.binding.history_attn_raw(p, dev["Q"].data_ptr(), dev["Kh"].data_ptr(), dev["Vh"].data_ptr(), o.data_ptr(),
                                     lse.data_ptr(), ws.data_ptr() if need else None, need, torch.cuda.current_stream().cuda_stream)
    assert st == tl.binding.TLIN_OK
    sub = [0, H // 2, H - 1]
    ro, rl = oracle.history(*(np.ascontiguousarray(host[k][:, sub]) for k in ("Q", "Kh", "Vh")), w.dtype, w.scale)
    assert_close(o[:, sub], ro, w.dtype, w.name)
    # fp32 weights and row sums: the log-sum-exp holds to fp32 rounding of scores of this size
    np.testing.assert_allclose(lse[:, sub].cpu().numpy(), rl, rtol=1e-5, atol=1e-5)
    assert bool((ws[need:] == 0xA5).all())


@pytest.mark.parametrize("D", [16, 32, 36, 48, 52, 64])
@pytest.mark.parametrize("W", [50, 128, 300, 2049])
def test_causal_rows_are_convex_combinations(D, W):
    """Stand-alone causal attention in bf16 at head dimensions up to 64 divides by the sum of the weights it
    multiplies the values with: over values of one all outputs are one, up to the rounding of two fp32 sums of
    the same W terms (chains of at most 16 terms a tile and one addition per tile on either side: 2 (16 + 33)
    2^-24 < 1e-5), whether the log-sum-exp is asked for or not; the log-sum-exp is that of the fp32 weights.
    The same through the layer call without a history and the sliding schedule of a single chunk."""
    w = ti.Workload(f"convex_{D}_{W}", 1, 8, D, 1, W, ti.BF16, 1.0, 9753 + D + W)
    host = ti.make(w)
    dev = {k: padded(host[k], w.dtype) for k in ("Q", "Kw", "Vw")}
    ones = padded(np.full_like(host["Vw"], 0x3F80), w.dtype)
    kw = dict(scale=w.scale, out_dtype=torch.float32)
    o = tl.tlin_window_causal_attn(dev["Q"], dev["Kw"], ones, **kw)
    assert (o - 1).abs().max().item() <= 1e-5
    o2, lse = tl.tlin_window_causal_attn(dev["Q"], dev["Kw"], ones, return_lse=True, **kw)
    assert torch.equal(o, o2)
    ro, rl = oracle.window_causal(host["Q"], host["Kw"], host["Vw"], w.dtype, w.scale)
    np.testing.assert_allclose(lse.cpu().numpy(), rl, rtol=1e-5, atol=1e-5)
    assert_close(tl.tlin_window_causal_attn(dev["Q"], dev["Kw"], dev["Vw"], scale=w.scale), ro, w.dtype, w.name)
    o = tl.tlin_layer_attn(dev["Q"], None, None, dev["Kw"], ones, **kw)
    assert (o - 1).abs().max().item() <= 1e-5
    for mode in (tl.TLIN_COMBINE_SUM, tl.TLIN_COMBINE_JOINT):
        o = tl.tlin_slide_layer_attn(dev["Q"], dev["Kw"], ones, dev["Kw"], ones, W, combine=mode, **kw)
        assert (o - 1).abs().max().item() <= 1e-5


@pytest.mark.parametrize("D", [36, 64, 100])
@pytest.mark.parametrize("W", [9, 32, 33, 64])
@pytest.mark.parametrize("N", [20, 1500, 9001])
def test_two_wave_workgroups_in_fp32(D, W, N):
    """fp32 windows of up to 64 rows, in workgroups whose second wave owns no row, one, or all of its rows:
    history, window, both layers (over 9001 rows the window block rides on partition 0) and the sliding
    schedule, whose last chunk is shorter."""
    w = ti.Workload(f"two_waves_{D}_{W}_{N}", 1, 3, D, N, W, ti.F32, 1.0, 5454 + D + W + N)
    host = ti.make(w)
    dev = {k: padded(v, w.dtype) for k, v in host.items()}
    o = tl.tlin_history_attn(dev["Q"], dev["Kh"], dev["Vh"], scale=w.scale)
    assert_close(o, oracle.history(host["Q"], host["Kh"], host["Vh"], w.dtype, w.scale)[0], w.dtype, f"{w.name} history")
    o = tl.tlin_window_causal_attn(dev["Q"], dev["Kw"], dev["Vw"], scale=w.scale)
    assert_close(o, oracle.window_causal(host["Q"], host["Kw"], host["Vw"], w.dtype, w.scale)[0], w.dtype, f"{w.name} window")
    for mode, omode in ((tl.TLIN_COMBINE_SUM, oracle.SUM), (tl.TLIN_COMBINE_JOINT, oracle.JOINT)):
        for splits in (0, 2):
            o = tl.tlin_layer_attn(dev["Q"], dev["Kh"], dev["Vh"], dev["Kw"], dev["Vw"], combine=mode, scale=w.scale, num_splits=splits)
            ro = oracle.layer(host["Q"], host["Kh"], host["Vh"], host["Kw"], host["Vw"], w.dtype, w.scale, omode)
            assert_close(o, ro, w.dtype, f"{w.name} layer mode {mode} splits {splits}")
    if N == 1500:
        kh, vh = dev["Kh"], dev["Vh"]
        o = tl.tlin_slide_layer_attn(kh, kh, vh, kh, vh, W, combine=tl.TLIN_COMBINE_JOINT, scale=w.scale)
        nats = w.scale * float((host["Kh"].astype(np.float64) ** 2).sum(-1).max())      # a key row meets itself
        assert_close(o, oracle.window_causal(host["Kh"], host["Kh"], host["Vh"], w.dtype, w.scale)[0], w.dtype, f"{w.name} slide",
                     f32_rel=f32_rel_bound(nats))


@pytest.mark.parametrize("D", [16, 36, 48, 64, 80, 96, 100, 128])
@pytest.mark.parametrize("W", [32, 65, 129, 257])
def test_fp32_operands_in_parts(D, W):
    """fp32 operands are multiplied as three bf16 parts.  A part or a product of parts that got lost leaves 2^-17 of
    single terms or more (2-norm above 2e-6); with all of them the 2-norm error is that of fp32 sums, a few 2^-24
    (measured up to 2.2e-7, bound 2^-21).  And the split commutes with powers of two: inputs scaled by them, far up and
    down the exponent range, give the same bits."""
    w = ti.Workload(f"parts_{D}_{W}", 1, 2, D, 1111, W, ti.F32, 1.0, 6363 + D + W)
    host = ti.make(w)
    dev = {k: padded(v, w.dtype) for k, v in host.items()}
    q, kh, vh, kw, vw = (dev[k] for k in ("Q", "Kh", "Vh", "Kw", "Vw"))
    for call, ref in ((lambda q, k, v: tl.tlin_history_attn(q, k, v, scale=w.scale), oracle.history),
                      (lambda q, k, v: tl.tlin_window_causal_attn(q, k, v, scale=w.scale), oracle.window_causal)):
        k, v, hk, hv = (kh, vh, "Kh", "Vh") if ref is oracle.history else (kw, vw, "Kw", "Vw")
        o = call(q, k, v)
        r = ref(host["Q"], host[hk], host[hv], w.dtype, w.scale)[0]
        d = o.cpu().numpy().astype(np.float64) - r
        assert np.sqrt((d * d).sum() / (r * r).sum()) <= 2.0 ** -21
        for eq, ev in ((60, 90), (-60, -90), (20, 0)):
            sq, sk, sv = padded(host["Q"] * np.float32(2.0 ** eq), w.dtype), padded(host[hk] * np.float32(2.0 ** -eq), w.dtype), padded(host[hv] * np.float32(2.0 ** ev), w.dtype)
            assert torch.equal(call(sq, sk, sv), o * 2.0 ** ev), (eq, ev)


@pytest.mark.parametrize("D", [36, 48, 64, 96, 128])
@pytest.mark.parametrize("W", [40, 129, 300])
@pytest.mark.parametrize("jump,vexp", [(6.0, 0), (12.0, 0), (60.0, 0), (12.0, 85)])
def test_logits_far_above_the_first_tiles(D, W, jump, vexp):
    """bf16 rows whose largest logits come late: keys from the fifth tile on are `jump` times as large, so that the
    reference point of the first tile is left behind by some 20, 45 and 200 nats, and values near the end of the
    range.  Unscaled outputs within the bf16 tolerance; scores of hundreds of nats are fp32 sums and carry their error
    (2^-22 of them) into the weights."""
    N = 700
    w = ti.Workload(f"late_{D}_{W}_{jump}", 1, 2, D, N, W, ti.BF16, 1.0, 1357 + D + W + int(jump))
    host = ti.make(w)

    def late(a):
        x = (a.astype(np.uint32) << 16).view(np.float32).copy()
        x[:, :, 256:] *= np.float32(jump)
        return (x.view(np.uint32) >> 16).astype(np.uint16)      # (jump has few bits; what is cut off is part of the input)

    host["Kh"], host["Kw"] = late(host["Kh"]), late(host["Kw"])
    dev = {k: padded(v, w.dtype) for k, v in host.items()}
    big = {k: padded((((v.astype(np.uint32) << 16).view(np.float32) * np.float32(2.0 ** vexp)).view(np.uint32) >> 16).astype(np.uint16), w.dtype)
           for k, v in host.items() if k in ("Vh", "Vw")}
    for splits in (1, 2):
        ro, rl = oracle.history(host["Q"], host["Kh"], host["Vh"], w.dtype, w.scale)
        o, lse = tl.tlin_history_attn(dev["Q"], dev["Kh"], big["Vh"], scale=w.scale, num_splits=splits, out_dtype=torch.float32, return_lse=True)
        assert_close(o * 2.0 ** -vexp, ro, w.dtype, f"{w.name} history splits {splits}, both outputs")
        np.testing.assert_allclose(lse.cpu().numpy(), rl, rtol=1e-5, atol=1e-5)
        o = tl.tlin_history_attn(dev["Q"], dev["Kh"], big["Vh"], scale=w.scale, num_splits=splits, out_dtype=torch.float32)
        assert_close(o * 2.0 ** -vexp, ro, w.dtype, f"{w.name} history splits {splits}")
        for mode, omode in ((tl.TLIN_COMBINE_SUM, oracle.SUM), (tl.TLIN_COMBINE_JOINT, oracle.JOINT)):
            o = tl.tlin_layer_attn(dev["Q"], dev["Kh"], big["Vh"], dev["Kw"], big["Vw"], combine=mode, scale=w.scale, num_splits=splits, out_dtype=torch.float32)
            ro2 = oracle.layer(host["Q"], host["Kh"], host["Vh"], host["Kw"], host["Vw"], w.dtype, w.scale, omode)
            assert_close(o * 2.0 ** -vexp, ro2, w.dtype, f"{w.name} layer mode {mode} splits {splits}")
    for lse in (False, True):
        o = tl.tlin_window_causal_attn(dev["Q"], dev["Kw"], big["Vw"], scale=w.scale, out_dtype=torch.float32, return_lse=lse)
        o = o[0] if lse else o
        assert_close(o * 2.0 ** -vexp, oracle.window_causal(host["Q"], host["Kw"], host["Vw"], w.dtype, w.scale)[0], w.dtype, f"{w.name} window lse {lse}")


@pytest.mark.parametrize("dtype,D", [(ti.BF16, 128), (ti.BF16, 84), (ti.F32, 128), (ti.F32, 72)])
@pytest.mark.parametrize("H,W,N", [(3, 256, 2600), (3, 257, 2600), (3, 384, 2600), (3, 385, 2600), (24, 384, 1200), (2, 300, 40)])
def test_workgroup_shapes_of_ragged_windows(dtype, D, H, W, N):
    """Windows at both sides of the lines between eight-wave and four-wave workgroups (257 and 384 rows; 24 heads x 384
    over a short history stay with eight waves, one partition over 40 rows): history, both layers, and the array of the
    library, whose capacity no plan may exceed where 32 heads' partials fit."""
    w = ti.Workload(f"ragged_{D}_{H}_{W}_{N}", 1, H, D, N, W, dtype, 1.0, 2121 + D + H + W + N)
    host = ti.make(w)
    dev = {k: padded(v, w.dtype) for k, v in host.items()}
    heads = sorted({0, H - 1})
    sub = {k: np.ascontiguousarray(v[:, heads]) for k, v in host.items()}
    o, lse = tl.tlin_history_attn(dev["Q"], dev["Kh"], dev["Vh"], scale=w.scale, return_lse=True)
    ro, rl = oracle.history(sub["Q"], sub["Kh"], sub["Vh"], w.dtype, w.scale)
    assert_close(o[:, heads], ro, w.dtype, f"{w.name} history")
    np.testing.assert_allclose(lse[:, heads].cpu().numpy(), rl, rtol=1e-5, atol=1e-5)
    for mode, omode in ((tl.TLIN_COMBINE_SUM, oracle.SUM), (tl.TLIN_COMBINE_JOINT, oracle.JOINT)):
        ro = oracle.layer(sub["Q"], sub["Kh"], sub["Vh"], sub["Kw"], sub["Vw"], w.dtype, w.scale, omode)
        o = tl.tlin_layer_attn(dev["Q"], dev["Kh"], dev["Vh"], dev["Kw"], dev["Vw"], combine=mode, scale=w.scale)
        assert_close(o[:, heads], ro, w.dtype, f"{w.name} layer mode {mode}")
        o = tl.tlin_layer_attn_static_ws(dev["Q"], dev["Kh"], dev["Vh"], dev["Kw"], dev["Vw"], combine=mode)
        assert_close(o[:, heads], ro, w.dtype, f"{w.name} layer mode {mode}, the library's array")


@pytest.mark.parametrize("D,N", [(128, 1), (128, 40), (128, 64), (128, 65), (128, 128), (128, 129), (128, 180), (128, 192), (128, 193), (128, 256),
                                 (96, 60), (96, 180), (64, 128), (64, 200), (64, 256), (64, 300), (36, 128), (36, 129)])
def test_long_query_sides_over_few_keys(D, N):
    """Queries of twelve heads, which do not divide the compute units, over keys that stay in LDS: odd and even tile
    counts, ragged last tiles, and both sides of the lines where the ring kernel takes over; with log-sum-exp."""
    W = 22050
    w = ti.Workload(f"few_keys_{D}_{N}", 1, 12, D, N, W, ti.BF16, 1.0, 808 + D + N)
    host = ti.make(w)
    dev = {k: padded(host[k], w.dtype) for k in ("Q", "Kh", "Vh")}
    rows = np.unique(np.concatenate([np.arange(0, 300), np.arange(W - 300, W), np.arange(300, W - 300, 97)]))
    o, lse = tl.tlin_history_attn(dev["Q"], dev["Kh"], dev["Vh"], scale=w.scale, return_lse=True)
    for h in (0, 11):
        sub = [np.ascontiguousarray(host["Q"][:, h:h + 1, rows]), np.ascontiguousarray(host["Kh"][:, h:h + 1]), np.ascontiguousarray(host["Vh"][:, h:h + 1])]
        ro, rl = oracle.history(*sub, w.dtype, w.scale)
        assert_close(o[:, h:h + 1, torch.from_numpy(rows).cuda()], ro, w.dtype, f"{w.name} head {h}")
        # (the unpipelined resident body, for up to 64 columns and for odd tile counts, sums rounded weights: 2^-8)
        rounded = N <= (256 if D > 48 else 128) if D <= 64 else -(-N // 64) == 3 or D < 128 and -(-N // 64) == 1
        np.testing.assert_allclose(lse[:, h:h + 1, torch.from_numpy(rows).cuda()].cpu().numpy(), rl, rtol=0 if rounded else 1e-5, atol=4.5e-3 if rounded else 1e-5)


def bf16_bits(x):
    """The upper halves of fp32 values (what is cut off must be zero or not matter)."""
    return (np.asarray(x, dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16)


def masked_inputs(name, D, W, N, dtype, hist, win, mask, seed):
    """Inputs whose history keys `hist` and window keys `win` (slices) are masked through column 0: the keys that
    stay have 0 there, the masked ones `mask`, and the queries 2 or (every third row) 4, so that a masked key's logit is
    -inf, also where `mask` is the type's lowest number (the product overflows)."""
    w = ti.Workload(name, 1, 2, D, N, W, dtype, 1.0, seed)
    host = ti.make(w)
    bits = bf16_bits if dtype == ti.BF16 else np.float32
    host["Q"][..., 0] = bits(np.where(np.arange(W) % 3 == 0, 4.0, 2.0).astype(np.float32))
    for k, s in (("Kh", hist), ("Kw", win)):
        host[k][..., 0] = 0
        host[k][:, :, s, 0] = bits(np.float32(mask))
    return w, host


LOWEST = {ti.BF16: -(2.0 - 2.0 ** -7) * 2.0 ** 127, ti.F32: -float(np.finfo(np.float32).max)}


def check_masked(w, host, hist, win, splits_list=(1, 2)):
    """History, causal and layer calls of masked inputs against the oracle over the visible keys alone.  Window rows
    that see masked window keys only have no value (0 / 0) and are left out."""
    H, W, N = w.H, w.W, w.N
    dev = {k: padded(v, w.dtype) for k, v in host.items()}
    vh, vw = np.ones(N, bool), np.ones(W, bool)
    vh[hist], vw[win] = False, False
    kh, vvh = (np.ascontiguousarray(host[k][:, :, vh]) for k in ("Kh", "Vh"))
    seen = np.cumsum(vw)                              # visible window keys of each row
    rows = np.flatnonzero(seen > 0)
    f32_rel = f32_rel_bound(25.0)

    def window(i):                                    # oracle of window row i over its visible keys
        pick = np.flatnonzero(vw[:i + 1])
        return [np.ascontiguousarray(host[k][:, :, r]) for k, r in (("Q", [i]), ("Kw", pick), ("Vw", pick))]

    some = sorted({int(rows[0]), int(rows[-1])} | {int(i) for i in rows[:: max(1, len(rows) // 12)]})
    if vh.any():
        ro, rl = oracle.history(host["Q"], kh, vvh, w.dtype, w.scale)
        for splits in splits_list:
            o, lse = tl.tlin_history_attn(dev["Q"], dev["Kh"], dev["Vh"], scale=w.scale, num_splits=splits, out_dtype=torch.float32, return_lse=True)
            assert_close(o, ro, w.dtype, f"{w.name} history splits {splits}, both outputs", f32_rel=f32_rel)
            np.testing.assert_allclose(lse.cpu().numpy(), rl, rtol=1e-5, atol=1e-5)
            o = tl.tlin_history_attn(dev["Q"], dev["Kh"], dev["Vh"], scale=w.scale, num_splits=splits, out_dtype=torch.float32)
            assert_close(o, ro, w.dtype, f"{w.name} history splits {splits}", f32_rel=f32_rel)
    for lse in (False, True):
        o = tl.tlin_window_causal_attn(dev["Q"], dev["Kw"], dev["Vw"], scale=w.scale, out_dtype=torch.float32, return_lse=lse)
        o = o[0] if lse else o
        for i in some:
            assert_close(o[:, :, i:i + 1], oracle.history(*window(i), w.dtype, w.scale)[0], w.dtype, f"{w.name} window row {i} lse {lse}", f32_rel=f32_rel)
    for splits in splits_list:
        o = tl.tlin_layer_attn(dev["Q"], dev["Kh"], dev["Vh"], dev["Kw"], dev["Vw"], combine=tl.TLIN_COMBINE_JOINT, scale=w.scale, num_splits=splits, out_dtype=torch.float32)
        for i in some:
            q, kw, vv = window(i)
            ro = oracle.history(q, np.ascontiguousarray(np.concatenate([kh, kw], 2)), np.ascontiguousarray(np.concatenate([vvh, vv], 2)), w.dtype, w.scale)[0]
            assert_close(o[:, :, i:i + 1], ro, w.dtype, f"{w.name} layer joint row {i} splits {splits}", f32_rel=f32_rel)


MASKS = [(slice(0, 64), slice(0, 0)), (slice(0, 300), slice(0, 70)), (slice(640, 700), slice(0, 130)), (slice(0, 637), slice(5, 64))]


@pytest.mark.parametrize("D", [36, 64, 96, 128])
@pytest.mark.parametrize("W", [40, 129, 300])
@pytest.mark.parametrize("hist,win", MASKS)
@pytest.mark.parametrize("kind", ["inf", "lowest"])
def test_masked_keys_bf16(D, W, hist, win, kind):
    """Keys masked by -inf or by the type's lowest number: whole first tiles, all but the last tile, last tiles, and
    partitions of three tiles and more."""
    mask = -np.inf if kind == "inf" else LOWEST[ti.BF16]
    win = slice(min(win.start, W - 20), min(win.stop, W - 20))
    w, host = masked_inputs(f"masked_{D}_{W}_{hist.start}_{hist.stop}_{kind}", D, W, 700, ti.BF16, hist, win, mask, 4242 + D + W)
    check_masked(w, host, hist, win)


@pytest.mark.parametrize("D", [36, 64, 96, 128])
@pytest.mark.parametrize("W", [12, 129, 300])
@pytest.mark.parametrize("hist,win", MASKS)
@pytest.mark.parametrize("kind", ["inf", "lowest"])
def test_masked_keys_fp32(D, W, hist, win, kind):
    """The same in fp32, whose operands are split into parts that an infinity does not have."""
    mask = -np.inf if kind == "inf" else LOWEST[ti.F32]
    win = slice(min(win.start, max(0, W - 20)), min(win.stop, max(0, W - 20)))
    w, host = masked_inputs(f"masked_f32_{D}_{W}_{hist.start}_{hist.stop}_{kind}", D, W, 700, ti.F32, hist, win, mask, 2424 + D + W)
    check_masked(w, host, hist, win)


@pytest.mark.parametrize("D", [36, 64, 96, 128])
@pytest.mark.parametrize("W", [12, 129, 300])
def test_infinite_values_fp32(D, W):
    """An infinite value makes its column infinite in the rows that see it, and no other column."""
    w = ti.Workload(f"inf_value_{D}_{W}", 1, 2, D, 700, W, ti.F32, 1.0, 31 + D + W)
    host = ti.make(w)
    dev = {k: padded(v, w.dtype) for k, v in host.items()}
    f32_rel = f32_rel_bound(10.0)
    for k, call, ref in (("h", tl.tlin_history_attn, oracle.history), ("w", tl.tlin_window_causal_attn, oracle.window_causal)):
        v = dev["V" + k].clone() if dev["V" + k].is_contiguous() else padded(host["V" + k], w.dtype)
        v[:, :, 7, 3], v[:, :, 9, 5] = float("inf"), float("-inf")
        o = call(dev["Q"], dev["K" + k], v, scale=w.scale)
        ro = ref(host["Q"], host["K" + k], host["V" + k], w.dtype, w.scale)[0]
        assert (o[:, :, 9:, 3] == float("inf")).all() and (o[:, :, 9:, 5] == float("-inf")).all()
        cols = [c for c in range(D) if c not in (3, 5)]
        assert_close(o[..., cols], ro[..., cols], w.dtype, f"{w.name} {k}", f32_rel=f32_rel)


@pytest.mark.parametrize("D", [36, 64, 96, 128])
@pytest.mark.parametrize("W", [12, 129, 300])
@pytest.mark.parametrize("eq,ek,ev,columns", [(115, -115, 0, 1), (-115, 115, 0, 1), (110, -110, 0, 2), (0, 0, -115, 1), (0, 0, -122, 2), (0, 0, 110, 1)])
def test_far_ends_of_the_range_fp32(D, W, eq, ek, ev, columns):
    """Queries, keys and values (every one, or every second column) near the ends of fp32's range: their parts leave
    bf16's, the results keep fp32's accuracy."""
    w = ti.Workload(f"far_{D}_{W}_{eq}_{ev}_{columns}", 1, 2, D, 700, W, ti.F32, 1.0, 63 + D + W)
    host = ti.make(w)
    for k, e in (("Q", eq), ("Kh", ek), ("Kw", ek), ("Vh", ev), ("Vw", ev)):
        host[k][..., ::columns] *= np.float32(2.0 ** e)
    dev = {k: padded(v, w.dtype) for k, v in host.items()}
    for splits in (1, 2):
        o, lse = tl.tlin_history_attn(dev["Q"], dev["Kh"], dev["Vh"], scale=w.scale, num_splits=splits, return_lse=True)
        ro, rl = oracle.history(host["Q"], host["Kh"], host["Vh"], w.dtype, w.scale)
        for c in range(columns):
            assert_close(to_host64(o)[..., c::columns], ro[..., c::columns], w.dtype, f"{w.name} history splits {splits}")
        np.testing.assert_allclose(lse.cpu().numpy(), rl, rtol=1e-5, atol=1e-5)
    o = tl.tlin_window_causal_attn(dev["Q"], dev["Kw"], dev["Vw"], scale=w.scale)
    ro = oracle.window_causal(host["Q"], host["Kw"], host["Vw"], w.dtype, w.scale)[0]
    for c in range(columns):
        assert_close(to_host64(o)[..., c::columns], ro[..., c::columns], w.dtype, f"{w.name} window")
    o = tl.tlin_layer_attn(dev["Q"], dev["Kh"], dev["Vh"], dev["Kw"], dev["Vw"], combine=tl.TLIN_COMBINE_JOINT, scale=w.scale)
    ro = oracle.layer(host["Q"], host["Kh"], host["Vh"], host["Kw"], host["Vw"], w.dtype, w.scale, oracle.JOINT)
    for c in range(columns):
        assert_close(to_host64(o)[..., c::columns], ro[..., c::columns], w.dtype, f"{w.name} layer")


@pytest.mark.parametrize("D", [36, 64, 128])
@pytest.mark.parametrize("W", [33, 100, 300])
def test_no_offset_over_long_histories_fp32(D, W):
    """The bf16 matrix instruction rounds towards minus infinity: 1e-9 of the values per key if nothing is done about it,
    which over 10^6 keys is four times the error of fp32 sums.  Mean error of outputs of values around zero, whose 2-norm
    is 1 / sqrt(N): independent roundings of 4e-7 leave a standard error of 4e-7 / sqrt(N W D) (3e-11 at most here,
    bound 1e-10)."""
    w = ti.Workload(f"offset_{D}_{W}", 1, 1, D, 200000, W, ti.F32, 1.0, 11 + D + W)
    gen = torch.Generator(device="cuda").manual_seed(w.seed)
    q, k, v = (torch.randn(1, 1, r, D, generator=gen, device="cuda") for r in (W, w.N, w.N))
    for splits in (0, 16):
        o = tl.tlin_history_attn(0.5 * q, 0.5 * k, v, scale=w.scale, num_splits=splits)
        r = torch.softmax((0.5 * q).double() @ (0.5 * k).double().transpose(-1, -2).contiguous() * w.scale, -1) @ v.double()
        d = o.double() - r
        assert abs(d.mean().item()) <= 1e-10, d.mean().item()


@pytest.mark.parametrize("D,N,hist", [(128, 180, slice(0, 64)), (128, 256, slice(0, 200)), (128, 50, slice(9, 50)), (96, 250, slice(0, 130)),
                                      (64, 200, slice(0, 70)), (36, 300, slice(0, 256))])
def test_masked_keys_of_long_query_sides(D, N, hist):
    """The same where keys stay in LDS and a workgroup walks over many query blocks."""
    W = 22050
    w = ti.Workload(f"masked_few_{D}_{N}", 1, 12, D, N, W, ti.BF16, 1.0, 515 + D + N)
    host = ti.make(w)
    host["Q"][..., 0] = bf16_bits(np.where(np.arange(W) % 3 == 0, 4.0, 2.0))
    host["Kh"][..., 0] = 0
    host["Kh"][:, :, hist, 0] = bf16_bits(LOWEST[ti.BF16])
    seen = np.ones(N, bool)
    seen[hist] = False
    o = tl.tlin_history_attn(*(padded(host[k], w.dtype) for k in ("Q", "Kh", "Vh")), scale=w.scale)
    rows = np.arange(0, W, 41)
    for h in (0, 11):
        sub = [np.ascontiguousarray(host[k][:, h:h + 1, r]) for k, r in (("Q", rows), ("Kh", seen), ("Vh", seen))]
        assert_close(o[:, h:h + 1, torch.from_numpy(rows).cuda()], oracle.history(*sub, w.dtype, w.scale)[0], w.dtype, f"{w.name} head {h}")


@pytest.mark.parametrize("dtype", [ti.BF16, ti.F32])
@pytest.mark.parametrize("D", [36, 64, 96, 128])
@pytest.mark.parametrize("W,N", [(40, 700), (300, 700), (300, 90)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_a_bad_query_row_stays_alone(dtype, D, W, N, bad):
    """A query row that is not finite leaves every other row's bits as they are."""
    w = ti.Workload(f"bad_row_{D}_{W}_{N}", 1, 2, D, N, W, dtype, 1.0, 99 + D + W)
    host = ti.make(w)
    dev = {k: padded(v, w.dtype) for k, v in host.items()}
    rows = [3, 21, W - 1]
    q = dev["Q"].clone() if dev["Q"].is_contiguous() else padded(host["Q"], w.dtype)
    q[:, :, rows, 0] = bad
    keep = torch.ones(W, dtype=torch.bool, device="cuda")
    keep[rows] = False
    for call in (lambda x: tl.tlin_history_attn(x, dev["Kh"], dev["Vh"], scale=w.scale),
                 lambda x: tl.tlin_history_attn(x, dev["Kh"], dev["Vh"], scale=w.scale, return_lse=True)[0],
                 lambda x: tl.tlin_window_causal_attn(x, dev["Kw"], dev["Vw"], scale=w.scale),
                 lambda x: tl.tlin_window_causal_attn(x, dev["Kw"], dev["Vw"], scale=w.scale, return_lse=True)[0],
                 lambda x: tl.tlin_layer_attn(x, dev["Kh"], dev["Vh"], dev["Kw"], dev["Vw"], scale=w.scale)):
        good, got = call(dev["Q"]), call(q)
        assert torch.isnan(got[:, :, rows].float()).any(-1).all()
        if dtype == ti.BF16:
            assert torch.equal(got[:, :, keep], good[:, :, keep])
        else:
            assert_close(got[:, :, keep], to_host64(good[:, :, keep]), w.dtype, w.name)


@pytest.mark.parametrize("D", [36, 64, 96, 128])
@pytest.mark.parametrize("W", [40, 129, 300])
def test_outputs_do_not_depend_on_the_log_sum_exp(D, W):
    """bf16: asking for the log-sum-exp changes no bit of O."""
    w = ti.Workload(f"both_{D}_{W}", 1, 2, D, 1111, W, ti.BF16, 1.0, 77 + D + W)
    host = ti.make(w)
    dev = {k: padded(v, w.dtype) for k, v in host.items()}
    for call in (lambda lse: tl.tlin_history_attn(dev["Q"], dev["Kh"], dev["Vh"], scale=w.scale, return_lse=lse),
                 lambda lse: tl.tlin_history_attn(dev["Q"], dev["Kh"], dev["Vh"], scale=w.scale, num_splits=1, return_lse=lse),
                 lambda lse: tl.tlin_window_causal_attn(dev["Q"], dev["Kw"], dev["Vw"], scale=w.scale, return_lse=lse)):
        assert torch.equal(call(False), call(True)[0])
