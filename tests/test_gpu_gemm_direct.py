"""GEMM kernels that copy their operands straight into LDS, where the last tile, the last k-step or the last 16-byte chunk of a row
is only partly inside the matrix."""
import pytest

from paper_2406_17145_amd import binding as B
from tests.parity_util import compare, run_gpu, run_oracle
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
