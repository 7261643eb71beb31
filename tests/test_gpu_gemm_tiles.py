"""The GEMM kernels' tile shapes at sizes where they can go wrong: every output tile of the large kernels, matrices that end inside
a tile in rows, in columns and inside a 16-byte chunk of a row, gradients that are stored and gradients that are added to."""
import numpy as np
import pytest

from paper_2406_17145_amd import binding as B
from paper_2406_17145_amd import workloads as W
from tests.parity_util import compare, run_gpu, run_oracle
from tests.test_gemm_choice_cpu import least_workspace
from tests.test_gpu_schedule import _run

pytestmark = pytest.mark.gpu


def _chain(rows, widths, acts, branches, n_micro, dtype=W.BF16):
    """`branches` chains of Linear layers over the given widths, side by side, a squared loss on all of them."""
    g = W._Graph()
    outs = []
    for _ in range(branches):
        x = g.input(widths[0], dtype)
        for k, n, act in zip(widths, widths[1:], acts):
            x = g.linear(x, k, n, act, dtype)
        outs.append(x)
    y, total = outs[0], widths[-1] * branches
    if branches > 1:
        y = g.add("concat", outs, out_features=total, dtype=dtype)
    t = g.input(total, W.F32, role="target")
    g.add("loss_mse", (y, t), loss_scale=1.0 / (rows * n_micro * total))
    rng = np.random.Generator(np.random.PCG64(rows + total))
    params = W._draw_params(g.ops, rng)
    for p in params.values():
        p["b"] = 0.1 * rng.standard_normal(p["b"].shape).astype(np.float32)
    batches = W._draw_batches(g.ops, rows, n_micro, rng, {})
    return W.Workload("gemm_tiles", g.ops, rows, n_micro, params, batches, 2e-2 if dtype == W.BF16 else 1e-4)


def _plan(wl, slots=1, flags=0):
    d, keep = B.build_desc(wl.ops, wl.micro_batch, slots, flags)
    return B.gpp_stage_describe(d)


# What the second launch of a layer over slices of its contraction does to the sum of the slices: every activation, a residual
# addend, both storage types, a result of the stage, a result inside a merge buffer (on 16 bytes, on 8, on 2).  The sums lie over
# the slot's gradient buffers, so the backward pass that follows finds arbitrary bits in every row's padding.
@pytest.mark.parametrize("kind", ["none", "relu", "gelu", "f32", "residual", "output", "merge_0", "merge_12", "merge_13"])
@pytest.mark.parametrize("slots,flags", [(1, 0), (1, B.FLAG_GROUPED_DW), (2, B.FLAG_GROUPED_DW)])
def test_sums_over_slices(kind, slots, flags):
    rows, k, n, n_micro = 100, 16000, 1000, 3
    g = W._Graph()
    act = kind if kind in ("relu", "gelu") else "none"
    y = g.linear(g.input(k, W.BF16), k, n, act, W.BF16, out_dtype=W.F32 if kind == "f32" else None)
    if kind == "residual":
        y = g.add("add", (y, g.input(n, W.BF16)), out_features=n, dtype=W.BF16)
    if kind.startswith("merge"):
        col = int(kind[6:])
        parts = ([g.input(col, W.BF16)] if col else []) + [y]
        m = g.add("concat", parts, out_features=col + n, dtype=W.BF16)
        y, n = g.linear(m, col + n, 40, "gelu", W.BF16), 40
    if kind != "output":
        g.add("loss_mse", (y, g.input(n, W.F32, role="target")), loss_scale=1.0 / (rows * n_micro * n))
    rng = np.random.Generator(np.random.PCG64(len(kind)))
    params = W._draw_params(g.ops, rng)
    for p in params.values():
        p["b"] = 0.1 * rng.standard_normal(p["b"].shape).astype(np.float32)
    wl = W.Workload("gemm_tiles", g.ops, rows, n_micro, params, W._draw_batches(g.ops, rows, n_micro, rng, {}), 2e-2)
    gouts = [{y: W.round_to_bf16(rng.standard_normal((rows, n)).astype(np.float32))} for _ in range(n_micro)] if kind == "output" else None
    print(f"[case] slices {kind} slots={slots} flags={flags}", flush=True)
    assert [p["slices"] > 1 for p in _plan(wl, slots, flags) if p["kernel"] == "gemm_big_fwd"] == [True]
    _, res, grads = _run(wl, slots, 1, slots > 1, slots=slots, flags=flags, gouts=gouts)
    stage, ref = run_oracle(wl, gouts)
    compare(wl, res, grads, stage, ref, label=f"gemm_tiles slices {kind}")


def test_sums_over_slices_in_the_static_workspace():
    wl = _chain(256, (16384, 1024), ("gelu",), 1, 2)
    assert max(p["slices"] for p in _plan(wl)) > 1
    st = B.Stage(wl.ops, wl.micro_batch, wl.params, static_workspace=True)
    st.close()


def _label(p):
    """Kernel and tile of a launch, as the cases below name it (launches of the few-row family that run on ring-buffered tiles: ring)."""
    name = p["kernel"].replace("gemm_", "")
    if name.startswith("skinny") and p["ring"]:
        return name.replace("skinny", "ring") + f" {p['ring']}"
    return name + f" {p['tile']}" + (f" of {p['slices']}" if p["slices"] else "")


# The bar is that of bf16 storage with fp32 accumulation: the oracle rounds at the same places, so what is left is the order of
# fp32 sums and results that fall on the other side of a rounding boundary.
# `want`: kernel and tile that the plan must hold, or the case has lost what it is here for.
@pytest.mark.parametrize("rows,widths,acts,branches,want", [
    # 128 x 128: ragged in both directions, in rows only, contractions and slices of a merge that end inside a 16-byte chunk
    (2000, (128, 2056, 136), ("gelu", "none"), 2, ("big_fwd 64", "big_dx 64", "dw_ksplit 0")),
    (1900, (1904, 136, 2000), ("none", "gelu"), 2, ("big_dx 64", "bwd_merged_dx_dw 0")),
    (700, (1203, 333, 1207), ("gelu", "gelu"), 4, ("big_fwd 64", "big_dx 64", "big_dw 64")),
    # 256 x 256 with a last column inside a chunk: forward with the stash, backward-data with the derivative
    (1000, (2000, 4003), ("gelu",), 4, ("big_fwd 256",)),
    (1000, (64, 4003, 2000), ("gelu", "none"), 4, ("big_dx 256",)),
    # 128 x 256 forward, a last row tile of 122 rows, and ring-buffered tiles; the same with columns that end inside a chunk
    (250, (520, 2056, 520), ("gelu", "gelu"), 9, ("big_fwd 128", "ring_fwd 64", "ring_dx 128")),
    (250, (520, 2051, 520), ("gelu", "gelu"), 9, ("big_fwd 128", "ring_fwd 64", "ring_dx 128")),
    # 128 x 256 forward next to 128 x 128 backward-data: the same two
    (378, (1032, 2056, 200), ("gelu", "gelu"), 9, ("big_fwd 128", "big_dx 64")),
    (378, (2056, 2051, 200), ("gelu", "gelu"), 9, ("big_fwd 128", "big_dx 64")),
    # ring-buffered 64 x 64 tiles forward: one row more than two row blocks, columns that end inside a chunk, the smallest and an
    # ordinary launch with a choice; backward-data of these with the weight gradients, by the few-row body
    (129, (1000, 1500, 1000), ("gelu", "gelu"), 7, ("ring_fwd 64", "bwd_merged_dx_dw 0")),
    (300, (203, 333, 70), ("gelu", "none"), 3, ("ring_fwd 64", "ring_dx 64", "big_dw 64")),
    (65, (64, 128, 8), ("gelu", "none"), 1, ("ring_fwd 64", "bwd_merged_dx_dw 0")),
    (700, (600, 2000, 72), ("gelu", "none"), 1, ("ring_fwd 64", "skinny_fwd 0", "bwd_merged_dx_dw 0")),
    # few-row kernel: a contraction of 141 steps; backward-data of 11 and 25 column blocks (a group of 16 and one of 9) in several row blocks
    (100, (9000, 1000), ("none",), 1, ("skinny_fwd 0",)),
    (200, (352, 2000), ("gelu",), 1, ("ring_fwd 64", "bwd_merged_dx_dw 0")),
    (100, (800, 300, 470), ("gelu", "none"), 1, ("skinny_fwd 0", "ring_fwd 64", "bwd_merged_dx_dw 0")),
    # narrow results of many rows on the tiled kernel (64 x 64)
    (9000, (64, 60), ("gelu",), 16, ("mfma_fwd 64",)),
    # sums over 16 slices of the contraction, the last one shorter
    (130, (20008, 523, 64), ("gelu", "none"), 1, ("big_fwd 0 of 16",)),
    # few-row kernel, forward and backward-data each in a launch of its own: one row more than one and than two row blocks, a last
    # row block of 8 and of 44 rows, columns and contractions that end inside a chunk, a mask and a derivative in the epilogue
    (65, (2051, 131, 2051, 77), ("gelu", "relu", "none"), 1, ("skinny_fwd 0", "skinny_dx 0", "big_dw 64")),
    (129, (1000, 203, 4099, 70), ("gelu", "gelu", "none"), 2, ("skinny_fwd 0", "skinny_dx 0", "big_dw 128")),
    (200, (2051, 203, 3003, 70), ("gelu", "gelu", "none"), 2, ("skinny_fwd 0", "skinny_dx 0", "ring_dx 128")),
    (300, (2051, 333), ("gelu",), 3, ("skinny_fwd 0", "ring_dx 128")),
])
@pytest.mark.parametrize("grouped", [False, True])
def test_tiles_of_every_shape(rows, widths, acts, branches, want, grouped):
    wl = _chain(rows, widths, acts, branches, 2)          # (ungrouped: the second micro-batch adds to the gradients of the first)
    print(f"[case] rows={rows} widths={widths} branches={branches} grouped={grouped}", flush=True)
    held = {_label(p) for p in _plan(wl)}
    assert grouped or held.issuperset(want), held
    if grouped:
        _, res, grads = _run(wl, 2, 2, False, flags=B.FLAG_GROUPED_DW)
    else:
        res, grads = run_gpu(wl)
    stage, ref = run_oracle(wl)
    compare(wl, res, grads, stage, ref, label="gemm_tiles")


# A workspace that lacks only the gradient copies of a merge off 16 bytes: the stage runs on the gradients in place.
@pytest.mark.parametrize("act", ["relu", "gelu"])
@pytest.mark.parametrize("slots,flags", [(1, 0), (2, B.FLAG_GROUPED_DW)])
def test_merge_off_16_bytes_without_room_for_the_copies(act, slots, flags, monkeypatch):
    wl = _chain(300, (120, 77, 203), (act, act), 3, 2)
    least = least_workspace(wl.ops, wl.micro_batch, slots, flags)
    assert least < B.gpp_stage_workspace_bytes(B.build_desc(wl.ops, wl.micro_batch, slots, flags)[0])
    print(f"[case] merge off 16 bytes {act} slots={slots} flags={flags}", flush=True)
    stage, ref = run_oracle(wl)
    for room in (None, least):
        if room:
            monkeypatch.setattr(B, "gpp_stage_workspace_bytes", lambda d: room)
        _, res, grads = _run(wl, slots, 1, slots > 1, slots=slots, flags=flags)
        compare(wl, res, grads, stage, ref, label="gemm_tiles merge off 16 bytes")


# Launch tables on 16 bytes, where on cache lines they would not fit: 256 bytes less in every copy of them.
@pytest.mark.parametrize("slots,flags", [(1, 0), (2, B.FLAG_GROUPED_DW)])
def test_launch_tables_that_fit_on_16_bytes_only(slots, flags, monkeypatch):
    wl = _chain(33, (64,) * 14, ("relu",) * 13, 1, 2)
    room = least_workspace(wl.ops, wl.micro_batch, slots, flags) - 256 * slots
    print(f"[case] launch tables slots={slots} flags={flags}", flush=True)
    results = [_run(wl, slots, 1, slots > 1, slots=slots, flags=flags)[1:]]
    monkeypatch.setattr(B, "gpp_stage_workspace_bytes", lambda d: room)
    results.append(_run(wl, slots, 1, slots > 1, slots=slots, flags=flags)[1:])
    stage, ref = run_oracle(wl)
    for res, grads in results:
        compare(wl, res, grads, stage, ref, label="gemm_tiles launch tables")


# Weight gradients on one round of 256 x 128 tiles over a long contraction, ragged in all three directions.
@pytest.mark.parametrize("rows,n_micro,flags", [(2050, 2, 0), (4100, 1, B.FLAG_GROUPED_DW)])
def test_weight_gradient_on_large_tiles(rows, n_micro, flags):
    wl = _chain(rows, (4090, 4084), ("none",), 1, n_micro)
    print(f"[case] 256 x 128 weight gradient rows={rows} flags={flags}", flush=True)
    assert [p["tile"] for p in _plan(wl, 1, flags) if p["kernel"] == "gemm_big_dw"] == [256]
    _, res, grads = _run(wl, 1, 1, False, flags=flags)
    stage, ref = run_oracle(wl)
    compare(wl, res, grads, stage, ref, label="gemm_tiles")


# fp32: the small tiles (32 x 32, contraction in steps of 64, split over four waves) around their edges, and launches that are
# large enough for the 64 x 64 ones (forward; backward, whose first column of tiles also sums the bias gradient).  The bar is that of the fp32 path; a sum of 1100 products in another order is far below it.
@pytest.mark.parametrize("rows,widths,branches", [
    (1, (1, 1), 1), (8, (64, 128, 64), 2), (33, (65, 31, 97), 3), (64, (300, 32, 129), 2), (31, (400, 63, 1), 4), (1100, (1024, 1000), 1),
    (2100, (65, 1000), 1), (1100, (1000, 2050), 1)])
def test_fp32_tiles(rows, widths, branches):
    wl = _chain(rows, widths, ("relu", "none")[2 - len(widths) + 1:], branches, 2, dtype=W.F32)
    print(f"[case] fp32 rows={rows} widths={widths} branches={branches}", flush=True)
    res, grads = run_gpu(wl)
    stage, ref = run_oracle(wl)
    compare(wl, res, grads, stage, ref, label="gemm_tiles fp32")
