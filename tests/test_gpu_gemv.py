"""GPU tests of the fp32 products of one to four rows on a packed weight
(MatMul variant 16): K of one 16-byte piece, below, at and past the runs that
the unrolled loop and its remainder take, columns one to three past a group of
four, two-level rows, and every epilogue step."""
from __future__ import annotations

import pytest

from gpu_util import assert_close, forced_table, random_inputs, run_device, say
from oracle import execute
from test_gpu_ops import EPILOGUES, _check_gemm, epilogue_graph, proj_graph, reference_rounding_except, siblings_graph

pytestmark = pytest.mark.gpu


def row_kernel(M, K, N):
    """The rule by which variant 16 takes the row kernel."""
    return K >= 512 * (M if M <= 2 else 4) or (M == 1 and K >= 128 and N <= 4096)


@pytest.mark.parametrize("K", [4, 124, 128, 508, 512, 1020, 1028, 2044, 2048, 4096, 5124, 9000])
@pytest.mark.parametrize("rows", [(1, 1), (1, 2), (3, 1), (2, 2), (1, 4)], ids=str)
@pytest.mark.parametrize("N", [2, 5, 36])
def test_few_rows(K, rows, N, tmp_path):
    B, S = rows
    og, a, c = proj_graph(B, S, K, N, "f32")
    say(f"few rows {rows} K {K} N {N}")
    lp = _check_gemm(og, {}, {1: 16}, tmp_path, K + N, "f32")
    tile = "row4" if row_kernel(B * S, K, N) else "dl16x32w8"
    assert lp.kernel(1).startswith(f"gemm_f32_{tile}_ak_bk_")


@pytest.mark.parametrize("rows", [(1, 1), (1, 3)], ids=str)
@pytest.mark.parametrize("chain", sorted(EPILOGUES))
def test_few_rows_epilogue(rows, chain, tmp_path):
    B, S = rows
    og, a, r, edges = epilogue_graph(B, S, 2052, 43, "f32", False, chain)
    mm = og.producer(edges[0])
    xs, cs = random_inputs(og, 5)
    (ref,) = execute.run_canonical(og, xs, cs)
    say(f"few rows {rows} {chain}")
    out, lp, _ = run_device(og, forced_table(og, {}, {mm: 16}), xs, cs, tmp_path, no_reuse=True)
    assert lp.kernel(mm).startswith("gemm_f32_row4_ak_bk_")
    assert_close(out[0], ref, "f32", f"{rows} {chain}")


@pytest.mark.parametrize("rows", [(1, 1), (1, 2), (3, 1), (2, 2)], ids=str)
@pytest.mark.parametrize("K", [68, 4100])
def test_few_rows_grouped(rows, K, tmp_path):
    """Q, K and V products of at most four rows, each with its bias, in one
    launch (of the row kernel where K is long): the oracle's result, and bit for bit what the
    same products give when they are launched one by one."""
    import json

    import torch
    from paper_2411_09242_amd import fluid as F
    og, prods, outs = siblings_graph(*rows, K, 43, "f32")
    mms = [i for i, nd in enumerate(og.nodes) if nd.op == "matmul"]
    xs, cs = random_inputs(og, K)
    path = tmp_path / "table.json"
    path.write_text(json.dumps(forced_table(og, {}, {m: 16 for m in mms})))
    g = F.Graph.from_desc(og.export())
    lp = F.LayoutPlan(g, F.CostTable.load(str(path), g))
    ap = F.ArenaPlan(g, lp, no_reuse=True, epilogue=True)
    ex = F.Executor(g, lp, ap, cs, xs)
    launch, _, names = ex.schedule()
    assert len({launch[m] for m in mms}) == 1
    tile = "row4" if row_kernel(rows[0] * rows[1], K, 43) else "dl16x32w8"
    assert names[launch[mms[0]]].startswith(f"gemm_f32_{tile}_") and names[launch[mms[0]]].endswith("_eb_x3")
    say(f"few rows grouped {rows} K {K}")
    ex.arena.fill_(0xFF)
    whole = ex.run()[0].clone()
    ref = reference_rounding_except(og, xs, cs, set(prods))
    torch.cuda.synchronize()
    assert_close(whole.cpu().numpy(), ref[0], "f32", f"{rows} {K}")
    ex.arena.fill_(0xFF)
    ex.outputs[0].fill_(float("nan"))
    for n in range(g.n_nodes):       # one call per node (a product with its bias Add)
        if n in mms:
            ex.run_nodes([n, n + 1])
        elif n - 1 not in mms:
            ex.run_nodes([n])
    torch.cuda.synchronize()
    assert torch.equal(ex.outputs[0], whole)
