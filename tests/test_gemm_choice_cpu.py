"""Which GEMM kernels a stage's plan holds and what workspace it needs, from the library's own planner (no GPU): the sizes at
which a rule of the dispatch changes its answer."""
import re

import pytest

from paper_2406_17145_amd import binding as B
from paper_2406_17145_amd import workloads as W


def desc(ops, rows, slots=1, flags=0):
    return B.build_desc(ops, rows, slots, flags)


def plan(ops, rows, slots=1, flags=0):
    d, keep = desc(ops, rows, slots, flags)
    return B.gpp_stage_describe(d)


def layers(rows, k, n, branches=1, act="none", dtype=W.BF16, loss=False, out_dtype=None, grad=True):
    """`branches` Linear layers side by side over inputs of their own; a loss over the first one's output, or stage outputs."""
    g = W._Graph()
    for _ in range(branches):
        y = g.linear(g.input(k, dtype) if grad else g.input(k, dtype, role="fixed"), k, n, act, dtype, out_dtype=out_dtype)
    if loss:
        g.add("loss_mse", (y, g.input(n, W.F32, role="target")), loss_scale=1.0 / (rows * n))
    return g.ops


def least_workspace(ops, rows, slots=1, flags=0):
    """Bytes that creation insists on, from its refusal of a workspace of none (pointers are not followed before that)."""
    ptr = {i: [4096, 4096] for i, o in enumerate(ops) if o["kind"] == "linear"}
    d, keep = B.build_desc(ops, rows, slots, flags, ptr, ptr)
    with pytest.raises(B.GppError) as e:
        B.gpp_stage_create(d, 4096, 0)
    assert e.value.status == B.GPP_ERR_WORKSPACE
    return int(re.search(r"need (\d+) bytes", str(e.value)).group(1))


def merged(rows, widths, act="gelu"):
    """Layers of these output widths over inputs of 64 columns, merged, one layer behind, outputs handed on."""
    g = W._Graph()
    outs = [g.linear(g.input(64, W.BF16), 64, w, act, W.BF16) for w in widths]
    y = g.add("concat", outs, out_features=sum(widths), dtype=W.BF16)
    g.linear(y, sum(widths), 72, "none", W.BF16)
    return g.ops


def nested_merge(act, layers, depth):
    """ADD of a merge, whose layers with an activation sit `depth` merges further in, and `layers` plain layers; a layer and a loss."""
    g = W._Graph()
    y = g.add("concat", [g.linear(g.input(64, W.BF16), 64, 64, act, W.BF16) for _ in range(2)], out_features=128, dtype=W.BF16)
    for d in range(depth):
        y = g.add("concat", (y, g.linear(g.input(64, W.BF16), 64, 64, "none", W.BF16)), out_features=192 + 64 * d, dtype=W.BF16)
    n = 128 + 64 * depth
    z = g.input(n, W.BF16)
    for _ in range(layers):
        z = g.linear(z, n, n, "none", W.BF16)
    y = g.linear(g.add("add", (y, z), out_features=n, dtype=W.BF16), n, 64, "none", W.BF16)
    g.add("loss_mse", (y, g.input(64, W.F32, role="target")), loss_scale=1.0 / 6400)
    return g.ops


def skipped(kinds, hidden):
    """An operator with one consumer per entry of `kinds`, all of a level, each of them added to it again: its gradient arrives through
    the additions first, then from that level."""
    g = W._Graph()
    x = g.input(64, W.BF16)
    if hidden:
        x = g.linear(x, 64, 64, "gelu", W.BF16)
    ends = []
    for k in kinds:
        y = (g.linear(x, 64, 64, k, W.BF16) if k != "norm" else
             g.add("layernorm", (x,), in_features=64, out_features=64, dtype=W.BF16, eps=1e-5))
        ends.append(g.add("add", (y, x), out_features=64, dtype=W.BF16))
    n = 64 * len(ends)
    g.add("loss_mse", (g.add("concat", ends, out_features=n, dtype=W.BF16), g.input(n, W.F32, role="target")), loss_scale=1.0 / (100 * n))
    return g.ops


def line(n):
    return -(-n // 256) * 256


@pytest.mark.parametrize("rows,k,n", [(128, 20480, 4096), (256, 16384, 1024), (100, 16000, 1000)])
@pytest.mark.parametrize("slots,flags", [(1, 0), (1, B.FLAG_GROUPED_DW), (4, 0), (4, B.FLAG_GROUPED_DW)])
@pytest.mark.parametrize("grad", [True, False])
def test_sums_over_slices_need_no_workspace(rows, k, n, slots, flags, grad):
    """A stage of one layer holds, per slot, the input, the output and the target, and per slot or once both gradients: the sums
    of a contraction over slices add nothing (what is left are launch tables of a few kilobytes)."""
    ops = layers(rows, k, n, loss=True, grad=grad)
    d, keep = desc(ops, rows, slots, flags)
    ld = B.gpp_ld
    values = line(rows * ld(k) * 2) + line(rows * ld(n) * 2) + line(rows * ld(n) * 4)
    grads = line(rows * ld(n) * 2) + (line(rows * ld(k) * 2) if grad else 0)
    need = slots * (values + (grads if flags else 0)) + (0 if flags else grads)
    assert need < B.gpp_stage_workspace_bytes(d) < need + (32 << 10) * slots


def test_sums_over_slices_fit_the_gradients_they_lie_over():
    def slices(ops, rows, slots, flags):
        return [p["slices"] for p in plan(ops, rows, slots, flags) if p["kernel"] == "gemm_big_fwd"]
    wide = layers(256, 20480, 1024, loss=True)
    for slots, flags in ((1, 0), (1, B.FLAG_GROUPED_DW), (3, B.FLAG_GROUPED_DW)):
        (s,) = slices(wide, 256, slots, flags)
        assert 2 <= s and s * 256 * 1024 * 4 <= 256 * 20480 * 2     # (the input's gradient buffer)
    # gradients that the slots share may be in use by another micro-batch; without an input gradient there is nothing to lie over
    assert not any(slices(wide, 256, 2, 0))
    assert not any(slices(layers(256, 20480, 1024, loss=True, grad=False), 256, 1, B.FLAG_GROUPED_DW))


@pytest.mark.parametrize("slots,flags", [(1, 0), (3, 0), (3, B.FLAG_GROUPED_DW)])
def test_gradient_copies_of_a_merge_are_not_insisted_on(slots, flags):
    """Columns 100 and 305 of a merge are off 16 bytes: two gradients are copied, and may be read in place instead."""
    ops, rows = merged(500, (100, 100, 105, 40)), 500
    d, keep = desc(ops, rows, slots, flags)
    copies = line(rows * 128 * 2) + line(rows * 64 * 2)
    want, least = B.gpp_stage_workspace_bytes(d), least_workspace(ops, rows, slots, flags)
    assert abs(want - least - copies * (slots if flags else 1)) < 4096 * slots       # (launch tables differ by some records)
    aligned = merged(500, (104, 96, 104, 40))
    d, keep = desc(aligned, rows, slots, flags)
    assert B.gpp_stage_workspace_bytes(d) == least_workspace(aligned, rows, slots, flags)


@pytest.mark.parametrize("flags", [B.FLAG_FORCE_GENERIC_GEMM, B.FLAG_FORCE_GENERIC_GEMM | B.FLAG_GROUPED_DW])
def test_no_gradient_copies_without_matrix_cores(flags):
    ops, rows = merged(500, (100, 100, 105, 40)), 500
    d, keep = desc(ops, rows, 2, flags)
    assert B.gpp_stage_workspace_bytes(d) == least_workspace(ops, rows, 2, flags)
    # one element-wise launch of the backward pass ingests the output gradients, one applies the derivatives, one returns the
    # input gradients
    assert len([p for p in B.gpp_stage_describe(d) if p["pass"] == "backward" and p["kernel"] == "elt_bwd"]) == 3


def test_activation_of_a_copied_gradient_costs_no_launch():
    """Launches of the backward pass between the merged layer's GEMMs and the branches': one that copies and multiplies (GELU),
    none but the copies where the merged layer has applied the derivative of every branch (ReLU)."""
    for act in ("gelu", "relu"):
        steps = [p for p in plan(merged(500, (100, 100, 105, 40), act), 500) if p["pass"] == "backward"]
        elt = [p["records"] for p in steps if p["kernel"] == "elt_bwd"]
        # output gradients in; two copies, and in place the other two; input gradients that no GEMM stored itself
        assert elt[:2] == [1, 4 if act == "gelu" else 2]
        assert len(elt) <= 3


@pytest.mark.parametrize("branches,k,n,streams", [(1, 64, 64, 0), (1, 4096, 4096, 0), (1, 4096, 8191, 0), (1, 4096, 8192, 1),
                                                  (2, 4000, 4096, 0), (2, 4096, 4096, 1), (7, 4096, 4096, 1)])
def test_gradients_that_exceed_half_the_last_level_cache_are_stored_past_it(branches, k, n, streams):
    (step,) = [p for p in plan(layers(64, k, n, branches), 64, 1, B.FLAG_GROUPED_DW) if p["pass"] == "weights"]
    assert step["streams"] == streams


@pytest.mark.parametrize("rows,k,n,branches,flags,tile", [
    (1023, 4096, 4096, 1, 0, 64), (1024, 4096, 4096, 1, 0, 256), (4096, 300, 4096, 8, 0, 64), (4096, 64, 64, 256, B.FLAG_GROUPED_DW, 64), (2048, 4096, 4096, 1, 0, 256), (2048, 4090, 4084, 1, 0, 256), (2048, 3840, 4096, 1, 0, 64),
    (511, 2048, 2048, 4, B.FLAG_GROUPED_DW, 64), (4096, 2048, 2048, 4, B.FLAG_GROUPED_DW, 256), (4096, 2048, 1792, 4, B.FLAG_GROUPED_DW, 64)])
def test_weight_gradients_take_the_large_tile_for_long_contractions(rows, k, n, branches, flags, tile):
    (step,) = [p for p in plan(layers(rows, k, n, branches), rows, 1, flags) if p["kernel"] == "gemm_big_dw"]
    assert step["tile"] == tile


def tiles(rows, k, n, branches, kernel):
    return [p["tile"] for p in plan(layers(rows, k, n, branches), rows) if p["kernel"] == kernel]


def test_large_tiles_behind_a_short_contraction_take_whole_rounds():
    for k, want in ((16, 64), (1000, 64), (1024, 64), (1032, 256), (2000, 256)):          # 608 tiles of 256 x 256
        assert tiles(9679, k, 1000, 4, "gemm_big_fwd") == [want], k
    for k, want in ((16, 256), (512, 256), (1024, 256)):                                  # 512
        assert tiles(2048, k, 4096, 4, "gemm_big_fwd") == [want], k
    for k, want in ((512, 64), (768, 256)):                                               # 2432
        assert tiles(9679, k, 4096, 4, "gemm_big_fwd") == [want], k
    for n, want in ((64, 64), (256, 64), (264, 256), (1000, 256)):                        # 2432, backward-data
        assert tiles(9679, 4096, n, 4, "gemm_big_dx") == [want], n


def test_narrow_results_of_many_rows():
    for k, n, kernel in ((64, 64, "gemm_mfma_fwd"), (128, 64, "gemm_mfma_fwd"), (136, 64, "gemm_skinny_fwd"), (128, 72, "gemm_big_fwd")):
        fwd = [p["kernel"] for p in plan(layers(40000, k, n, 4), 40000) if p["pass"] == "forward"]
        assert kernel in fwd, (k, n, fwd)


def test_narrow_weight_gradients_are_split_over_the_rows():
    for rows, k, n, branches, kernel in ((800, 4096, 16, 4, "gemm_dw_ksplit"), (921, 1899, 9, 7, "gemm_dw_ksplit"), (800, 4096, 65, 4, "gemm_big_dw"),
                                         (2000, 1000, 1000, 2, "gemm_dw_ksplit"), (1200, 1000, 1000, 4, "gemm_big_dw")):
        ops = layers(rows, k, n, branches, grad=False)
        assert [p["kernel"] for p in plan(ops, rows) if p["kernel"] in ("gemm_dw_ksplit", "gemm_big_dw")] == [kernel], (rows, k, n)


def test_fp32_launches_below_512_tiles_take_the_small_ones():
    def of(rows, k, n, which):
        return [p["tile"] for p in plan(layers(rows, k, n, dtype=W.F32), rows) if p["pass"] == which and p["kernel"].startswith("gemm")]
    assert of(64 * 511, 64, 64, "forward") == [32] and of(64 * 511 + 1, 64, 64, "forward") == [64]
    assert of(8, 64, 64, "backward") == [32] and of(1100, 1000, 2050, "backward") == [64]


def test_weight_gradients_of_three_levels_wait_for_the_end_of_the_pass():
    def weights(depth, flags=0, dtype=W.BF16, added=False):
        g = W._Graph()
        outs = []
        for _ in range(2):
            x = g.input(64, dtype)
            for _ in range(depth):
                x = g.linear(x, 64, 64, "relu", dtype)
            outs.append(x)
        y = g.add("concat", outs, out_features=128, dtype=dtype)
        if added:      # (the merge's gradient is a buffer of its own: its layers mask it in place)
            y = g.add("add", (y, g.linear(g.input(128, dtype), 128, 128, "none", dtype)), out_features=128, dtype=dtype)
        g.linear(y, 128, 64, "none", dtype)
        steps = [p for p in plan(g.ops, 100, 1, flags) if p["pass"] == "backward"]
        return [p["records"] for p in steps if p["kernel"] == "gemm_big_dw"], steps[-1]["kernel"]
    assert weights(1) == ([], "gemm_bwd_merged_dx_dw")            # two levels: each rides along with backward-data
    assert weights(2) == ([5], "gemm_big_dw") and weights(4)[0] == [9]
    assert weights(2, B.FLAG_FORCE_GENERIC_GEMM)[0] == [] and weights(3, dtype=W.F32)[0] == []
    assert weights(3, added=True)[0] == [8]


@pytest.mark.parametrize("layers", [1, 2, 3])
@pytest.mark.parametrize("depth", [0, 1, 2, 3])
@pytest.mark.parametrize("flags", [0, B.FLAG_GROUPED_DW])
def test_a_merge_with_masked_layers_anywhere_inside_shares_no_gradient(layers, depth, flags):
    """Layers with an activation multiply their columns of a merge's gradient in place: the merge has it to itself, and takes a copy
    of what the addition passes on; without an activation merge and addend read one buffer."""
    def of(act):
        ops = nested_merge(act, layers, depth)
        d, keep = desc(ops, 100, 1, flags)
        copies = [p["records"] for p in plan(ops, 100, 1, flags) if p["pass"] == "backward" and p["kernel"] == "elt_bwd"]
        return B.gpp_stage_workspace_bytes(d), copies
    (masked, m), (plain, p) = of("relu"), of("none")
    n = 128 + 64 * depth
    extra = line(100 * n * 2)
    assert extra <= masked - plain <= extra + 4096, (masked, plain)          # (launch tables)
    assert m[:1] == [1] and 2 in m and sum(m) == sum(p) + 3


@pytest.mark.parametrize("hidden", [False, True])
@pytest.mark.parametrize("kinds", [("none", "none"), ("gelu", "none", "gelu"), ("none", "norm"), ("norm", "gelu", "norm")])
def test_one_record_of_a_launch_adds_to_a_gradient_in_place(kinds, hidden):
    """What is already written is read and written by one record of a launch; the next one of the level, whose workgroups would run
    beside it, is in a launch behind it.  Nothing else than that is launched more."""
    steps = [p for p in plan(skipped(kinds, hidden), 100) if p["pass"] == "backward"]
    gemms = [p["records"] for p in steps if p["kernel"] in ("gemm_skinny_dx", "gemm_bwd_merged_dx_dw")]
    norms = [p["records"] for p in steps if p["kernel"] == "layernorm_bwd_dx"]
    n = sum(k != "norm" for k in kinds)
    assert gemms == [n + 1] + [1] * (n - 1) + [2] * hidden and norms == [1] * (len(kinds) - n)      # (weight gradients with the first)
    # a copy of the first addition's gradient, the others added to it, the level's derivatives (in copies of their own); then the
    # derivative of the layer in front, or the input's gradient on its way to the caller
    assert sum(p["kernel"] == "elt_bwd" for p in steps) == len(kinds) + ("gelu" in kinds) + 1, steps


@pytest.mark.parametrize("rows,kernel", [(1048512, "gemm_big_dw"), (1048513, "gemm_mfma_dw"), (1048575, "gemm_mfma_dw")])
@pytest.mark.parametrize("flags", [0, B.FLAG_GROUPED_DW])
def test_weight_gradients_whose_last_k_step_would_wrap_its_offsets(rows, kernel, flags):
    """Rows of 4 KiB: 1048576 of them are 2^32 bytes.  The large tiles fetch whole k-steps of 64 rows by 32-bit offsets and rely on rows
    beyond the matrix lying beyond its bytes; where the last k-step passes 2^32 they would read the first rows instead of zeros."""
    steps = [p for p in plan(layers(rows, 2048, 2048), rows, 1, flags) if p["kernel"].endswith("dw")]
    assert [p["kernel"] for p in steps] == [kernel]


def test_operands_of_four_gib_run_on_the_kernel_with_64_bit_addresses():
    """The matrix-core kernels form 32-bit offsets into an operand: its rows behind 2^32 bytes would be read from its start."""
    def kernels(rows, flags=0):
        steps = [p for p in plan(layers(rows, 2048, 64), rows, 1, flags) if p["kernel"].startswith("gemm")]
        return {(p["pass"], p["kernel"]) for p in steps}
    assert all("generic" not in k for _, k in kernels(1048575))
    for flags in (0, B.FLAG_GROUPED_DW):
        assert {("forward", "gemm_generic_fwd"), ("backward", "gemm_generic_bwd")} <= kernels(1048576, flags)
    weights = [p["kernel"] for p in plan(layers(300, 131072, 16384), 300) if p["kernel"].startswith("gemm")]       # (a 4 GiB weight matrix)
    assert weights[0] == "gemm_generic_fwd" and "gemm_generic_bwd" in weights


@pytest.mark.parametrize("rows,k,n,branches,kernel,tile", [
    (250, 520, 2056, 7, "gemm_skinny_fwd", 128), (250, 520, 2056, 8, "gemm_skinny_fwd", 128), (250, 520, 2056, 9, "gemm_big_fwd", 128),
    (250, 520, 2051, 9, "gemm_big_fwd", 128), (512, 512, 1000, 8, "gemm_skinny_fwd", 128), (512, 512, 1000, 9, "gemm_big_fwd", 128),
    (130, 1000, 1500, 10, "gemm_skinny_fwd", 64), (130, 1000, 1500, 12, "gemm_big_fwd", 128)])
def test_ring_tiles_that_begin_a_second_round(rows, k, n, branches, kernel, tile):
    """512 workgroups of 128 x 64 or 768 of 64 x 64 run at once; launches of up to half as many again go to the larger tiles."""
    (step,) = [p for p in plan(layers(rows, k, n, branches, act="relu", grad=False), rows) if p["kernel"].endswith("fwd") and "gemm" in p["kernel"]]
    assert (step["kernel"], step["ring"] or step["tile"]) == (kernel, tile)
