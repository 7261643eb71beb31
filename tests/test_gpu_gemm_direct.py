"""GEMM kernels that copy their operands straight into LDS, where the last tile, the last k-step or the last 16-byte chunk of a row
is only partly inside the matrix."""
import pytest

from tests.parity_util import compare, run_gpu, run_oracle
from tests.test_gpu_gemm_tiles import _chain, _plan

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
