"""GPU tests of the small-M fp32 GEMM tiles (MatMul variants 6, 7, 16, 17):
K slices of none, one, as many as the DMA stages and one more 16-k groups per
wavefront, a partial last group, and rows and columns one past a tile, in
every operand orientation."""
from __future__ import annotations

import itertools

import pytest

from gpu_util import say
from oracle import layouts
from test_gpu_ops import _check_gemm, proj_graph

pytestmark = pytest.mark.gpu


# K: per wavefront (8 or 4 of them) 0-1, 1, 3, 3-4 and 4-7 groups of 16
@pytest.mark.parametrize("K", [4, 64, 128, 384, 388, 452])
@pytest.mark.parametrize("variant", [6, 7, 16, 17])
def test_group_counts(K, variant, tmp_path):
    B, S, N = 1, 36, 36
    og, a, c = proj_graph(B, S, K, N, "f32")
    for pa, pc in itertools.product(layouts.layout_list((B, S, K)), layouts.layout_list((B, S, N))):
        say(f"small gemm K {K} v{variant} A{pa} C{pc}")
        _check_gemm(og, {a: pa, c: pc}, {1: variant}, tmp_path, K, "f32")
