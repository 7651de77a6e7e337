"""GPU tests of the small bf16 GEMM tiles on K-contiguous operands (MatMul
variants 12 to 14, the weight packed): K slices of none, part of one, one, as
many as the DMA stages and more 64-k groups per wavefront, a partial last
group, and rows and columns one past a tile."""
from __future__ import annotations

import pytest

from gpu_util import say
from oracle import layouts
from test_gpu_ops import _check_gemm, proj_graph

pytestmark = pytest.mark.gpu


# K: per wavefront (4 or 8 of them) 0-1, 1, 1-2, 2, 3 and 5-9 groups of 64
@pytest.mark.parametrize("K", [8, 64, 256, 512, 520, 1032, 2056])
@pytest.mark.parametrize("rows", [(1, 31), (3, 11), (1, 65)], ids=str)
@pytest.mark.parametrize("variant", [12, 13, 14])
def test_group_counts(K, rows, variant, tmp_path):
    B, S = rows
    og, a, c = proj_graph(B, S, K, 36, "bf16")
    for pc in layouts.layout_list((B, S, 36)):
        say(f"small bf16 gemm K {K} {rows} v{variant} C{pc}")
        lp = _check_gemm(og, {c: pc}, {1: variant}, tmp_path, K, "bf16")
        tile = {12: "dma32w4", 13: "dma32w8", 14: "dma64x32w4"}[variant]
        assert lp.kernel(1).startswith(f"gemm_bf16_{tile}_ak_bk_")
