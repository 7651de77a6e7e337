"""GPU tests of the fp32 products of one to four rows on a packed weight
(MatMul variant 16): K of one 16-byte piece, below, at and past the runs that
the unrolled loop and its remainder take, columns one to three past a group of
four, two-level rows, and every epilogue step."""
from __future__ import annotations

import pytest

from gpu_util import assert_close, forced_table, random_inputs, run_device, say
from oracle import execute
from test_gpu_ops import EPILOGUES, _check_gemm, epilogue_graph, proj_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [4, 1020, 1028, 4096, 5124, 9000])
@pytest.mark.parametrize("rows", [(1, 1), (1, 2), (3, 1), (2, 2), (1, 4)], ids=str)
@pytest.mark.parametrize("N", [2, 5, 36])
def test_few_rows(K, rows, N, tmp_path):
    B, S = rows
    og, a, c = proj_graph(B, S, K, N, "f32")
    say(f"few rows {rows} K {K} N {N}")
    lp = _check_gemm(og, {}, {1: 16}, tmp_path, K + N, "f32")
    assert lp.kernel(1).startswith("gemm_f32_dl16x32w8_ak_bk_")


@pytest.mark.parametrize("rows", [(1, 1), (1, 3)], ids=str)
@pytest.mark.parametrize("chain", sorted(EPILOGUES))
def test_few_rows_epilogue(rows, chain, tmp_path):
    B, S = rows
    og, a, r, edges = epilogue_graph(B, S, 68, 43, "f32", False, chain)
    mm = og.producer(edges[0])
    xs, cs = random_inputs(og, 5)
    (ref,) = execute.run_canonical(og, xs, cs)
    say(f"few rows {rows} {chain}")
    out, lp, _ = run_device(og, forced_table(og, {}, {mm: 16}), xs, cs, tmp_path, no_reuse=True)
    assert_close(out[0], ref, "f32", f"{rows} {chain}")
