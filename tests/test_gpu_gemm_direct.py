"""GEMM kernels that copy their operands straight into LDS, where the last tile, the last k-step or the last 16-byte chunk of a row
is only partly inside the matrix; copies of rows in 16-byte pieces; what the launches around them leave to each other."""
import numpy as np
import pytest

from paper_2406_17145_amd import binding as B
from paper_2406_17145_amd import workloads as W
from tests.parity_util import compare, run_gpu, run_oracle, t2n
from tests.test_gemm_choice_cpu import nested_merge, skipped
from tests.test_gpu_gemm_tiles import _chain, _plan
from tests.test_gpu_schedule import _run

pytestmark = pytest.mark.gpu


def _held(wl, flags=0):
    return {p["kernel"].replace("gemm_", "") + f" {p['tile']}" for p in _plan(wl, 1, flags)}


# Backward-data on 128 x 256 tiles: a last row tile of 122 rows, a last column tile that ends inside a chunk and one of a single
# column block; with a stashed derivative, with a mask and with neither.  (The bar is that of bf16 storage with fp32 sums.)
@pytest.mark.parametrize("rows,widths,acts,branches", [
    (250, (64, 2051, 1024), ("gelu", "none"), 9), (250, (64, 2056, 776), ("relu", "none"), 9), (635, (1288, 2000), ("none",), 7)])
def test_backward_data_on_128_x_256_tiles(rows, widths, acts, branches):
    wl = _chain(rows, widths, acts, branches, 2)
    print(f"[case] backward-data 128 x 256 rows={rows} widths={widths}", flush=True)
    assert "big_dx 128" in _held(wl)
    res, grads = run_gpu(wl)
    stage, ref = run_oracle(wl)
    compare(wl, res, grads, stage, ref, label="gemm_direct")


# Ring-buffered tiles: a contraction of one k-step and of less than the buffers hold, one that ends inside a k-step and inside a
# chunk, a last row tile of one row, columns that end inside a tile and inside a chunk, one row block; every activation, and a
# result that is stored as fp32.  `want`: tile rows of the ring launches, forward and backward-data.
@pytest.mark.parametrize("rows,widths,acts,branches,want", [
    (513, (1000, 1000, 1000), ("gelu", "gelu"), 4, {("fwd", 128), ("dx", 128)}),
    (300, (203, 333, 70), ("gelu", "none"), 3, {("fwd", 64), ("dx", 64)}),
    (129, (1000, 1500, 1003), ("relu", "gelu"), 7, {("fwd", 64), ("dx", 64)}),
    (700, (130, 603, 132), ("gelu", "relu"), 3, {("fwd", 64), ("dx", 64)}),
    (2047, (64, 65, 128), ("gelu", "none"), 1, {("fwd", 64), ("dx", 64)}),
    (300, (1, 200, 9), ("relu", "none"), 2, {("fwd", 64), ("dx", 64)}),
])
def test_ring_buffered_tiles(rows, widths, acts, branches, want):
    wl = _chain(rows, widths, acts, branches, 2)
    print(f"[case] ring rows={rows} widths={widths} branches={branches}", flush=True)
    held = {(p["kernel"].split("_")[2], p["ring"]) for p in _plan(wl, 2, B.FLAG_GROUPED_DW) if p["ring"]}
    assert held >= want, held
    stage, ref = run_oracle(wl)
    _, res, grads = _run(wl, 2, 2, False, flags=B.FLAG_GROUPED_DW)
    compare(wl, res, grads, stage, ref, label="gemm_direct ring")
    res, grads = run_gpu(wl)
    compare(wl, res, grads, stage, ref, label="gemm_direct ring")


# Weight gradients on 256 x 128 tiles: rows that end inside a k-step, slots one behind the other and around the end of the stash,
# a second group that adds, matrices that end inside a tile in both directions and inside a chunk.
@pytest.mark.parametrize("rows,n_micro,slots", [(515, 4, 2), (543, 3, 3), (577, 3, 2)])
def test_grouped_weight_gradients_on_256_x_128_tiles(rows, n_micro, slots):
    wl = _chain(rows, (2034, 2051), ("gelu",), 4, n_micro)
    print(f"[case] 256 x 128 weight gradients rows={rows} micro-batches={n_micro} slots={slots}", flush=True)
    assert [p["tile"] for p in _plan(wl, slots, B.FLAG_GROUPED_DW) if p["pass"] == "weights"] == [256]
    _, res, grads = _run(wl, slots, slots, False, flags=B.FLAG_GROUPED_DW)
    stage, ref = run_oracle(wl)
    compare(wl, res, grads, stage, ref, label="gemm_direct dw")


# Weight gradients of three and more levels in one launch behind their own backward pass, stored by the first micro-batch and added
# to by the others; on 64 x 64, 128 x 64 and 128 x 128 tiles, with matrices that end inside a tile and inside a chunk and rows that
# end inside a k-step, of which there may be one.
@pytest.mark.parametrize("rows,widths,branches,want", [
    (1, (64, 64, 64, 64), 1, (64, 64)), (40, (72, 65, 129, 200), 2, (64, 64)), (300, (203, 333, 70, 129), 3, (64, 64)),
    (700, (1000, 1000, 263, 520), 2, (128, 128)), (300, (520, 1000, 1003, 520), 4, (64, 0))])
@pytest.mark.parametrize("slots,two_streams", [(1, False), (2, True)])
def test_weight_gradients_behind_their_backward_pass(rows, widths, branches, want, slots, two_streams):
    wl = _chain(rows, widths, ("gelu", "relu", "none"), branches, 3)
    print(f"[case] weight gradients at the end rows={rows} widths={widths} slots={slots}", flush=True)
    (step,) = [p for p in _plan(wl, slots, 0) if p["kernel"] in ("gemm_big_dw", "gemm_dw_ksplit", "gemm_bwd_merged_dx_dw")]
    assert step["pass"] == "backward" and step["records"] == 3 * branches and (step["tile"], step["ring"]) == want
    _, res, grads = _run(wl, slots, 1, two_streams, slots=slots)
    stage, ref = run_oracle(wl)
    compare(wl, res, grads, stage, ref, label="gemm_direct weights at the end")


# Copies in pieces of 16 bytes: rows of every length around a piece, which therefore start at every element address, into padded rows
# and out of them; whole values, so nothing may differ.
@pytest.mark.parametrize("dtype", [W.BF16, W.F32])
@pytest.mark.parametrize("rows", [1, 3, 700])
def test_copies_of_rows_at_every_alignment(dtype, rows):
    widths = (1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 63, 65, 1003)
    g = W._Graph()
    ends = [g.add("add", (g.input(w, dtype), g.input(w, dtype)), out_features=w, dtype=dtype) for w in widths]
    g.linear(g.input(8, dtype), 8, 8, "none", dtype)
    rng = np.random.Generator(np.random.PCG64(rows))
    params = W._draw_params(g.ops, rng)
    ins = {i: W.round_to_bf16(rng.standard_normal((rows, o["out_features"])).astype(np.float32)) for i, o in enumerate(g.ops) if o["kind"] == "input"}
    st = B.Stage(g.ops, rows, params)
    outs, gins = st.alloc_outputs(), st.alloc_grad_inputs()
    gouts = [W.round_to_bf16(rng.standard_normal((rows, g.ops[i]["out_features"])).astype(np.float32)) for i in st.output_ids]
    print(f"[case] copies dtype={dtype} rows={rows}", flush=True)
    st.grad_reset()
    st.forward(0, st.stage_inputs(ins), outs)
    st.backward(0, [st.to_device(i, x) for i, x in zip(st.output_ids, gouts)], gins)
    st.sync_status()
    got_out = {i: t2n(t) for i, t in zip(st.output_ids, outs)}
    got_gin = {i: t2n(t) for i, t in zip(st.input_ids, gins) if t is not None}
    st.close()
    gout = dict(zip(st.output_ids, gouts))
    for e in ends:
        a, b = g.ops[e]["inputs"]
        want = ins[a] + ins[b]
        assert np.array_equal(got_out[e], W.round_to_bf16(want) if dtype == W.BF16 else want), e
        assert np.array_equal(got_gin[a], gout[e]) and np.array_equal(got_gin[b], gout[e]), e


# Activations in front of a merge: all of them GELU on 16 bytes (their derivatives are one matrix), one off 16 bytes, of mixed kinds,
# and a merge that two operators read.
@pytest.mark.parametrize("kind", ["gelu", "off", "mixed", "two_readers", "output"])
@pytest.mark.parametrize("slots,flags", [(1, 0), (2, B.FLAG_GROUPED_DW)])
def test_merged_activations(kind, slots, flags):
    rows, widths = 90, (40, 77, 64) if kind == "off" else (40, 72, 64)
    g = W._Graph()
    outs = [g.linear(g.input(50, W.BF16), 50, w, "relu" if kind == "mixed" and w == 72 else "gelu", W.BF16) for w in widths]
    total = sum(widths)
    y = g.add("concat", outs, out_features=total, dtype=W.BF16)
    z = g.linear(y, total, 48, "gelu", W.BF16)
    if kind == "two_readers":
        z = g.add("concat", (z, g.linear(y, total, 24, "gelu", W.BF16)), out_features=72, dtype=W.BF16)
    n = 72 if kind == "two_readers" else 48
    if kind != "output":
        g.add("loss_mse", (z, g.input(n, W.F32, role="target")), loss_scale=1.0 / (rows * 2 * n))
    rng = np.random.Generator(np.random.PCG64(len(kind)))
    params = W._draw_params(g.ops, rng)
    wl = W.Workload("merged_activations", g.ops, rows, 2, params, W._draw_batches(g.ops, rows, 2, rng, {}), 2e-2)
    gouts = [{z: W.round_to_bf16(rng.standard_normal((rows, n)).astype(np.float32))} for _ in range(2)] if kind == "output" else None
    print(f"[case] merged activations {kind} slots={slots} flags={flags}", flush=True)
    _, res, grads = _run(wl, slots, slots if flags else 1, False, slots=slots, flags=flags, gouts=gouts)
    stage, ref = run_oracle(wl, gouts)
    compare(wl, res, grads, stage, ref, label=f"merged activations {kind}")


# The dot interaction on the matrix cores: the fewest vectors, ragged and full 32 (and 33, which stay on the vector path), a batch that
# ends inside a workgroup, every width.  (Two vectors of one sample are no case: their gradients are one product's bf16 gradient times the
# other vector, and where that sum of 40 terms cancels, its one rounding is the whole error: 4.7e-2 on either path, 3e-3 over 40 samples.)
@pytest.mark.parametrize("F,d,b", [(2, 64, 41), (3, 128, 5), (17, 64, 67), (27, 128, 130), (32, 256, 6), (33, 64, 9), (9, 32, 10)])
def test_dot_interaction(F, d, b):
    g = W._Graph()
    vecs = [g.linear(g.input(24, W.BF16), 24, d, "none", W.BF16) for _ in range(F)]
    x = g.add("concat", vecs, out_features=F * d, dtype=W.BF16)
    w = d + F * (F - 1) // 2
    z = g.linear(g.add("dot_interact", (x,), in_features=d, out_features=w, dtype=W.BF16), w, 40, "none", W.BF16)
    g.add("loss_mse", (z, g.input(40, W.F32, role="target")), loss_scale=1.0 / (b * 2 * 40))
    rng = np.random.Generator(np.random.PCG64(F))
    params = W._draw_params(g.ops, rng)
    wl = W.Workload("dot_interaction", g.ops, b, 2, params, W._draw_batches(g.ops, b, 2, rng, {}), 2e-2)
    print(f"[case] interaction F={F} d={d} b={b}", flush=True)
    res, grads = run_gpu(wl)
    stage, ref = run_oracle(wl)
    compare(wl, res, grads, stage, ref, label="dot interaction")


# A merge of layers that is also an addend: layers with an activation multiply their slice of its gradient in place, so the other
# addend must not read the same buffer (it did, and got their masks); without one the two share it.
@pytest.mark.parametrize("act", ["relu", "gelu", "none"])
@pytest.mark.parametrize("layers", [1, 2])
def test_merge_added_to_a_layer(layers, act):
    g, outs = W._Graph(), []
    for _ in range(2):
        x = g.input(64, W.BF16)
        for _ in range(2):
            x = g.linear(x, 64, 64, act, W.BF16)
        outs.append(x)
    y, z = g.add("concat", outs, out_features=128, dtype=W.BF16), g.input(128, W.BF16)
    for _ in range(layers):
        z = g.linear(z, 128, 128, "none", W.BF16)
    y = g.linear(g.add("add", (y, z), out_features=128, dtype=W.BF16), 128, 64, "none", W.BF16)
    g.add("loss_mse", (y, g.input(64, W.F32, role="target")), loss_scale=1.0 / 6400)
    rng = np.random.Generator(np.random.PCG64(3))
    params = W._draw_params(g.ops, rng)
    wl = W.Workload("merge_added", g.ops, 100, 2, params, W._draw_batches(g.ops, 100, 2, rng, {}), 2e-2)
    print(f"[case] merge added layers={layers} act={act}", flush=True)
    res, grads = run_gpu(wl)
    stage, ref = run_oracle(wl)
    compare(wl, res, grads, stage, ref, label="merge added to a layer")


# The same with the activated layers in a merge inside the merge (and one further in), weight gradients per level, at the end of the
# pass and in one launch over the slots; the other addend reads its gradient at its own level or behind the masks of the layers.
@pytest.mark.parametrize("act", ["relu", "gelu", "none"])
@pytest.mark.parametrize("layers,depth,slots,flags", [
    (1, 1, 1, 0), (2, 1, 1, 0), (3, 2, 2, 0), (1, 1, 2, B.FLAG_GROUPED_DW), (2, 2, 2, B.FLAG_GROUPED_DW)])
def test_nested_merge_added_to_a_layer(layers, depth, slots, flags, act):
    wl = W.Workload("merge_nested", nested_merge(act, layers, depth), 100, 2, {}, [], 2e-2)
    rng = np.random.Generator(np.random.PCG64(depth))
    wl.params = W._draw_params(wl.ops, rng)
    wl.batches = W._draw_batches(wl.ops, 100, 2, rng, {})
    print(f"[case] nested merge added layers={layers} depth={depth} slots={slots} flags={flags} act={act}", flush=True)
    _, res, grads = _run(wl, slots, slots if flags else 1, False, slots=slots, flags=flags)
    stage, ref = run_oracle(wl)
    compare(wl, res, grads, stage, ref, label="nested merge added to a layer")


# An operator whose gradient arrives through two and three additions and then from as many operators of one level.
@pytest.mark.parametrize("hidden", [False, True])
@pytest.mark.parametrize("kinds", [("none", "none"), ("gelu", "none", "gelu"), ("none", "norm"), ("norm", "gelu", "norm")])
@pytest.mark.parametrize("slots,flags", [(1, 0), (2, B.FLAG_GROUPED_DW)])
def test_several_consumers_behind_additions(kinds, hidden, slots, flags):
    ops = skipped(kinds, hidden)
    rng = np.random.Generator(np.random.PCG64(len(kinds)))
    wl = W.Workload("several_consumers", ops, 100, 2, W._draw_params(ops, rng), W._draw_batches(ops, 100, 2, rng, {}), 2e-2)
    print(f"[case] several consumers {kinds} hidden={hidden} slots={slots} flags={flags}", flush=True)
    _, res, grads = _run(wl, slots, slots if flags else 1, False, slots=slots, flags=flags)
    stage, ref = run_oracle(wl)
    compare(wl, res, grads, stage, ref, label="several consumers behind additions")


# Operands around 2^32 bytes: the last matrix whose offsets fit 32 bits (whose last k-step of a weight gradient passes them) and a
# larger one.  Bars: bf16 storage of the results, and sums of a million products in fp32.
@pytest.mark.parametrize("rows", [1048575, 1048640])
def test_operands_of_four_gib(rows):
    import torch
    g = W._Graph()
    g.linear(g.input(2048, W.BF16), 2048, 64, "none", W.BF16)
    params = W._draw_params(g.ops, np.random.Generator(np.random.PCG64(1)))
    print(f"[case] operands of 4 GiB rows={rows}", flush=True)
    st = B.Stage(g.ops, rows, params)
    gen = torch.Generator(device=st.dev).manual_seed(rows)
    x = torch.randn(rows, 2048, device=st.dev, dtype=torch.bfloat16, generator=gen)
    dy = torch.randn(rows, 64, device=st.dev, dtype=torch.bfloat16, generator=gen)
    outs, gins, w = st.alloc_outputs(), st.alloc_grad_inputs(), torch.from_numpy(params[1]["W"]).to(st.dev)
    st.grad_reset()
    st.forward(0, [x], outs)
    st.backward(0, [dy], gins)
    st.sync_status()
    dw, db = torch.zeros(64, 2048, device=st.dev, dtype=torch.float64), dy.double().sum(0)
    for a in range(0, rows, 1 << 16):
        xs, ds = x[a:a + (1 << 16)].float(), dy[a:a + (1 << 16)].float()
        for got, want in ((outs[0][a:a + (1 << 16)], xs @ w.T), (gins[0][a:a + (1 << 16)], ds @ w)):
            assert ((got.float() - want).norm() / want.norm()).item() < 4e-3, a
        dw += (ds.T @ xs).double()
    grads = {k: torch.from_numpy(v).to(st.dev).double() for k, v in st.grads_numpy()[1].items()}
    st.close()
    assert ((grads["W"] - dw).norm() / dw.norm()).item() < 1e-4 and ((grads["b"] - db).norm() / db.norm()).item() < 1e-4
