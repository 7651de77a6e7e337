"""Column reductions at the edges of their row tiles (4, 8, 16 and 64 rows of
a workgroup, chosen by the number of rows, the row length and whether every
operand is column-major), against the oracle."""
import pytest

from gpu_util import assert_close, forced_table, random_inputs, run_device, say
from oracle import execute
from test_gpu_ops import norm_graph, softmax_graph

pytestmark = pytest.mark.gpu

# rows, row length: 4-row tiles with a remainder, one value past
# a wavefront's share, the longest row they hold and the first they do not;
# 8-row tiles (long rows; short rows of a run of 64 / 8 values); 16-row tiles
# (rows of at most 64; every operand column-major and over 2048 rows); 64-row
# tiles
CASES = [(2, 257), (5, 513), (1023, 260), (3, 4100), (2, 8192), (2, 8193), (1025, 300), (37, 65), (41, 63),
         (2050, 257), (2055, 130), (32770, 33)]


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
