"""Column reductions at the edges of their row tiles (4, 8, 16 and 64 rows of
a workgroup, chosen by the number of rows, the row length and whether every
operand is column-major), against the oracle."""
import pytest

from gpu_util import assert_close, forced_table, random_inputs, run_device, say
from oracle import execute, layouts
from test_gpu_ops import norm_graph, softmax_graph, sum_norm_graph

pytestmark = pytest.mark.gpu

# rows, row length: 4-row tiles with a remainder, one value past
# a wavefront's share, the longest row they hold and the first they do not;
# 8-row tiles (long rows; short rows of a run of 64 / 8 values); 16-row tiles
# (rows of at most 64; every operand column-major and over 2048 rows); 64-row
# tiles
CASES = [(2, 257), (5, 513), (1023, 260), (3, 4100), (2, 8192), (2, 8193), (1025, 300), (37, 65), (41, 63),
         (2050, 257), (2055, 130), (32770, 33), (515, 300), (2049, 100)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("op", ["softmax", "layernorm"])
@pytest.mark.parametrize("case", CASES, ids=str)
def test_column_reduction_row_tiles(dtype, op, case, tmp_path):
    S, R = case
    if op == "softmax":
        og, a, p = softmax_graph(1, 1, S, R, dtype, 0, 0.7)
        row, col = (0, 1, 2, 3), (0, 1, 3, 2)
    else:
        og, a, p = norm_graph(1, S, R, dtype, op)
        row, col = (0, 1, 2), (0, 2, 1)
    xs, cs = random_inputs(og, S + R, scale=2.0)
    (ref,) = execute.run_canonical(og, xs, cs)
    for la, lp in ((col, row), (row, col), (col, col)):
        say(f"column {op} {dtype} {case} {la} {lp}")
        out, _, _ = run_device(og, forced_table(og, {a: la, p: lp}, {1: 1}), xs, cs, tmp_path)
        assert_close(out[0], ref, dtype, f"{op} {case} {la} {lp}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("op", ["layernorm", "rmsnorm"])
@pytest.mark.parametrize("case", [(1, 37, 260), (3, 171, 300), (4, 300, 96), (2, 1030, 72)], ids=str)
def test_column_residual_norm(dtype, op, case, tmp_path):
    """The norm of a residual sum in one launch: both summands and the output
    column-major, beside row-major ones, and with other orders of the rows."""
    og, a, b, sm, n = sum_norm_graph(*case, dtype, op)
    xs, cs = random_inputs(og, sum(case), 2.0)
    (ref,) = execute.run_canonical(og, xs, cs, on_chip={sm})
    row, col, batch = (0, 1, 2), (0, 2, 1), (2, 1, 0)
    L = set(map(tuple, layouts.layout_list(case)))
    for la, lb, ln in ((col, row, row), (row, col, row), (row, row, col), (col, col, col), (batch, col, col),
                       (row, batch, col), (row, row, batch)):
        if not {la, lb, ln} <= L:
            continue          # one batch: equivalent layouts are listed once
        say(f"column residual {op} {dtype} {case} {la} {lb} {ln}")
        obj = forced_table(og, {a: la, b: lb, n: ln}, {3: 1})
        obj["fused_sigs"] = [{"op": "add", "in_shapes": [list(case)] * 2, "out_shape": list(case),
                              "entries": [[[list(la), list(lb)], list(ln), [-1, 1, -1]]]}]
        obj["fused"] = [[2, 1, 0]]
        out, lp, _ = run_device(og, obj, xs, cs, tmp_path)
        assert lp.kernel(2) == f"add_{op}_col_{dtype}"
        assert_close(out[0], ref, dtype, f"{op} {case} {la} {lb} {ln}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(1, 3, 37, 37), (2, 5, 60, 300), (1, 16, 130, 130)], ids=str)
def test_column_causal_softmax(dtype, shape, tmp_path):
    """Causal rows through the column variant's small tiles: the query dim
    among the row dims in every order."""
    og, a, p = softmax_graph(*shape, dtype, 1, 0.3)
    xs, cs = random_inputs(og, sum(shape), scale=2.0)
    (ref,) = execute.run_canonical(og, xs, cs)
    L = list(map(tuple, layouts.layout_list(shape)))
    row = (0, 1, 2, 3)
    others = [l for l in ((0, 1, 3, 2), (0, 3, 1, 2), (0, 3, 2, 1), (0, 2, 3, 1), (0, 2, 1, 3)) if l in L]
    for la, lp in [(row, o) for o in others] + [(o, row) for o in others] + [(others[0], others[-1])]:
        say(f"column causal softmax {dtype} {shape} {la} {lp}")
        out, _, _ = run_device(og, forced_table(og, {a: la, p: lp}, {1: 1}), xs, cs, tmp_path)
        assert_close(out[0], ref, dtype, f"{shape} {la} {lp}")
