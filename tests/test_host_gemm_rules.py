"""Which kernel a MatMul variant prepares, on both sides of every rule of the
dispatch (host library): the row kernel of fp32 tile 6, the split tiles 8 and
9 of fp32, the DMA kernel of the small bf16 tiles."""
import json

import pytest

from paper_2411_09242_amd import fluid as F


def kernel(tmp_path, dtype, variant, a, N):
    """The kernel of a[.., K] times a K x N weight under one variant."""
    F.load(host_only=True)
    K, out = a[-1], [*a[:-1], N]
    eye = list(range(len(a)))
    g = F.Graph.from_desc(dict(dtype=dtype, inputs=[list(a)], consts=[dict(role="weight", shape=[K, N], dtype=dtype)],
                               nodes=[dict(op="matmul", ins=[0, ~0], out_shape=out)], outputs=[1]))
    path = tmp_path / "t.json"
    path.write_text(json.dumps({
        "format": "fluid-cost-table/1", "edges": [[eye], [eye]], "node_sig": [0],
        "sigs": [{"op": "matmul", "in_shapes": [list(a)], "out_shape": out,
                  "entries": [[[eye], eye, [1 if v == variant else -1 for v in range(20)]]]}]}))
    return F.LayoutPlan(g, F.CostTable.load(str(path), g)).kernel(0)


@pytest.mark.parametrize("rows,K,N,row", [
    ((1, 1), 124, 4096, False), ((1, 1), 128, 4096, True), ((1, 1), 128, 4100, False), ((1, 1), 512, 8192, True),
    ((1, 2), 1020, 64, False), ((1, 2), 1024, 64, True), ((3, 1), 2044, 64, False), ((3, 1), 2048, 64, True),
    ((2, 2), 2044, 64, False), ((2, 2), 2048, 64, True), ((1, 5), 4096, 64, False), ((1, 2, 1), 4096, 64, False)])
def test_row_kernel(rows, K, N, row, tmp_path):
    """At most four rows in one batch (the first two dims of a four-dimensional
    A are batches), K long enough; only with the weight packed K-contiguous."""
    a = (*rows, K)
    name = kernel(tmp_path, "f32", 16, a, N)
    assert name.startswith("gemm_f32_row4_ak_bk_" if row else "gemm_f32_dl16x32w8_ak_bk_"), name
    assert kernel(tmp_path, "f32", 6, a, N).startswith("gemm_f32_dl16x32w8_ak_bmn_")


@pytest.mark.parametrize("M,K,N,large,small", [
    (2048, 64, 4096, "s256x128", "t64"), (2048, 64, 2048, "t64", "t64"), (2048, 68, 2048, "s128", "s128"),
    (2048, 256, 2052, "s256x128", "s128"),      # one round of 136 tiles against two of 272
    (3000, 256, 3000, "s128", "s128"),          # two rounds against three
    (4096, 256, 4096, "s256x128", "s128"),      # two against four
    (4224, 256, 4224, "s128", "s128"),          # three against five
    (6000, 256, 4096, "s256x128", "s128")])     # three against six
@pytest.mark.parametrize("packed", [0, 10])
def test_split_tiles(M, K, N, large, small, packed, tmp_path):
    assert kernel(tmp_path, "f32", 8 + packed, (M, K), N).startswith(f"gemm_f32_{large}_ak_")
    assert kernel(tmp_path, "f32", 9 + packed, (M, K), N).startswith(f"gemm_f32_{small}_ak_")


@pytest.mark.parametrize("variant,tile", [(2, "32w4"), (3, "32w8"), (4, "64x32w4")])
def test_dma_tiles(variant, tile, tmp_path):
    """Both operands K-contiguous: the weight packed, K a multiple of 8."""
    assert kernel(tmp_path, "bf16", 10 + variant, (37, 96), 72).startswith(f"gemm_bf16_dma{tile}_ak_bk_")
    assert kernel(tmp_path, "bf16", variant, (37, 96), 72).startswith(f"gemm_bf16_sk{tile}_ak_bmn_")
    assert kernel(tmp_path, "bf16", 10 + variant, (37, 92), 72).startswith(f"gemm_bf16_sk{tile}_ag_bg_")
    assert kernel(tmp_path, "f32", 10 + variant, (37, 96), 72).startswith(f"gemm_f32_sk{tile}_ak_bk_")
