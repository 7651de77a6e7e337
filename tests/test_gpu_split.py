"""GPU tests of the fp32 GEMM tiles that multiply three-way bf16 splits
(MatMul variants 8, 9 and, on packed weights, 18, 19): tile edges and K-tile
remainders in every operand orientation, the error against 64-bit arithmetic
beside the fp32 MFMA tile's, and infinities, NaN and the largest floats."""
from __future__ import annotations

import itertools

import numpy as np
import pytest

from gpu_util import say
from oracle import layouts
from test_gpu_ops import _check_gemm, proj_graph

pytestmark = pytest.mark.gpu

VARIANTS = [8, 9, 18, 19]
LARGE = (2057, 2052)        # rows, columns for which tile 8 takes its 256 x 128 kernel


def split_kernel(variant, M, K, N, a_k=True):
    """Start of the launch's name: the 256 x 128 tile where it needs clearly
    fewer rounds of 256 workgroups, the 64 x 64 fp32 tile for a short K."""
    def rounds(tm):
        return -(-(-(-M // tm) * -(-N // 128)) // 256)
    if variant % 10 == 8 and a_k and 17 * rounds(256) < 10 * rounds(128):
        return "gemm_f32_s256x128_"
    return "gemm_f32_t64_" if K <= 64 else "gemm_f32_s128_"


def rows_cols(variant, M, N):
    """(M, N), or the large output for the variants of tile 8."""
    return LARGE if variant % 10 == 8 else (M, N)


def product(variant, x, w):
    """x @ w by one MatMul variant (row-major operands and result)."""
    import json
    import tempfile

    import torch
    from paper_2411_09242_amd import fluid as F
    (M, K), N = x.shape, w.shape[1]
    g = F.Graph.from_desc(dict(dtype="f32", inputs=[[M, K]], consts=[dict(role="weight", shape=[K, N], dtype="f32")],
                               nodes=[dict(op="matmul", ins=[0, ~0], out_shape=[M, N])], outputs=[1]))
    cost = [1 if v == variant else -1 for v in range(20)]
    table = {"format": "fluid-cost-table/1", "edges": [[[0, 1]], [[0, 1]]], "node_sig": [0],
             "sigs": [{"op": "matmul", "in_shapes": [[M, K]], "out_shape": [M, N],
                       "entries": [[[[0, 1]], [0, 1], cost]]}]}
    with tempfile.NamedTemporaryFile("w", suffix=".json") as f:
        json.dump(table, f)
        f.flush()
        t = F.CostTable.load(f.name, g)
    lp = F.LayoutPlan(g, t)
    if variant in VARIANTS:
        assert lp.kernel(0).startswith(split_kernel(variant, M, K, N))
    ex = F.Executor(g, lp, F.ArenaPlan(g, lp), [w], [x])
    y = ex.run()[0]
    torch.cuda.synchronize()
    return y.cpu().numpy()


EDGES = [(1, 4, 68, 4), (1, 257, 68, 132), (3, 43, 100, 260), (1, 128, 96, 128), (1, 257, 64, 132)]
LARGE_EDGES = [(1, 2057, 68, 2052), (3, 700, 100, 2052), (1, 2304, 64, 2048)]      # tile 8 only


@pytest.mark.parametrize("variant,shape", [(v, s) for v in VARIANTS for s in EDGES + (LARGE_EDGES if v % 10 == 8 else [])],
                         ids=str)
def test_split_tile_edges(shape, variant, tmp_path):
    """One element past a tile, K not a multiple of a K-tile, exact tiles, the
    longest K that the 128 x 128 tile leaves to the 64 x 64 one and outputs
    large enough for the 256 x 128 tile; A and C in every layout."""
    B, S, K, N = shape
    og, a, c = proj_graph(B, S, K, N, "f32")
    for pa, pc in itertools.product(layouts.layout_list((B, S, K)), layouts.layout_list((B, S, N))):
        say(f"split {shape} v{variant} A{pa} C{pc}")
        lp = _check_gemm(og, {a: pa, c: pc}, {1: variant}, tmp_path, S + K, "f32")
        assert lp is None or lp.kernel(1).startswith(split_kernel(variant, B * S, K, N, lp.kernel(1).count("_ak_")))


@pytest.mark.parametrize("dist", ["normal", "positive", "wide"])
@pytest.mark.parametrize("variant", VARIANTS)
def test_split_error(dist, variant):
    """Every element within the bound of any fp32 summation, (K + 1) 2^-24
    sum |a b|; the root mean square of the errors in units of sum |a b| no
    larger than the 64 x 64 fp32 MFMA tile's, for values spread over ten
    decades ("wide") too."""
    rng = np.random.default_rng(7)
    (M, N), K = rows_cols(variant, 200, 136), 1024
    x, w = rng.standard_normal((M, K)), 0.02 * rng.standard_normal((K, N))
    if dist == "positive":
        x, w = np.abs(x), np.abs(w)
    elif dist == "wide":
        x, w = x * np.exp(4 * rng.standard_normal((M, K))), w * np.exp(4 * rng.standard_normal((K, N)))
    x, w = x.astype(np.float32), w.astype(np.float32)
    exact = x.astype(np.float64) @ w.astype(np.float64)
    size = np.abs(x).astype(np.float64) @ np.abs(w)
    err = {v: (product(v, x, w) - exact) / size for v in (variant, 1)}
    assert (np.abs(err[variant]) <= (K + 1) * 2.0 ** -24).all()
    rms = {v: float(np.sqrt((e * e).mean())) for v, e in err.items()}
    say(dist, variant, rms)
    assert rms[variant] <= rms[1]


@pytest.mark.parametrize("variant", VARIANTS)
def test_split_exceptions(variant):
    """Infinities, NaN, values that round to a bf16 infinity and overflowing
    sums give what fp32 arithmetic gives, and leave other tiles alone."""
    rng = np.random.default_rng(8)
    (M, N), K = rows_cols(variant, 300, 264), 68
    x, w = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((K, N)).astype(np.float32)
    big = np.float32(3.4e38)
    x[3, 5], w[5, 2] = np.inf, 0.0            # inf * 0: NaN in column 2
    w[5, 4] = 1.0                             # inf * 1 (exact in bf16): inf
    x[7, 9], w[9] = big, 0.5 * np.sign(w[9])  # rounds to a bf16 infinity, the product is finite
    x[60, 1] = np.nan
    w[8, 20] = -np.inf
    x[9, 8] = 0.0
    w[10:12] = 0.25
    x[20, 10], x[20, 11], w[10:12, 3] = big, big, 1.0   # overflows in column 3 alone
    got = product(variant, x, w)
    with np.errstate(all="ignore"):
        ref = x.astype(np.float64) @ w.astype(np.float64)
        ref = np.where(np.abs(ref) > np.finfo(np.float32).max, np.sign(ref) * np.inf, ref)
    assert (np.isnan(got) == np.isnan(ref)).all()
    inf = np.isinf(ref)
    assert (got[inf] == ref[inf]).all() and np.isfinite(got[np.isfinite(ref)]).all()
    ok = np.isfinite(ref)
    bound = (K + 1) * 2.0 ** -24 * (np.abs(np.nan_to_num(x, posinf=0)).astype(np.float64) @
                                    np.abs(np.nan_to_num(w, neginf=0)))
    assert (np.abs(got - ref)[ok] <= bound[ok]).all()


# (x, Co, kernel): one pixel and one channel past a tile, K not a multiple of
# four (4-byte weight loads), a K-tile more than the pipeline holds, two images
CONVS = [((1, 3, 10, 9), 65, 3), ((2, 5, 9, 11), 33, 2), ((1, 40, 12, 12), 64, 3), ((1, 130, 5, 5), 31, 1)]


def convolution(variant, x, w, b):
    import json
    import tempfile

    import torch
    from paper_2411_09242_amd import fluid as F
    out = [x.shape[0], w.shape[0], x.shape[2] - w.shape[2] + 1, x.shape[3] - w.shape[3] + 1]
    eye = [0, 1, 2, 3]
    g = F.Graph.from_desc(dict(dtype="f32", inputs=[list(x.shape)],
                               consts=[dict(role="weight", shape=list(w.shape), dtype="f32"),
                                       dict(role="bias", shape=list(b.shape), dtype="f32")],
                               nodes=[dict(op="conv", ins=[0, ~0, ~1], out_shape=out)], outputs=[1]))
    table = {"format": "fluid-cost-table/1", "edges": [[eye], [eye]], "node_sig": [0],
             "sigs": [{"op": "conv", "in_shapes": [list(x.shape)], "out_shape": out,
                       "entries": [[[eye], eye, [1 if v == variant else -1 for v in range(6)]]]}]}
    with tempfile.NamedTemporaryFile("w", suffix=".json") as f:
        json.dump(table, f)
        f.flush()
        t = F.CostTable.load(f.name, g)
    lp = F.LayoutPlan(g, t)
    ex = F.Executor(g, lp, F.ArenaPlan(g, lp), [w, b], [x])
    y = ex.run()[0]
    torch.cuda.synchronize()
    return y.cpu().numpy()


@pytest.mark.parametrize("case", CONVS, ids=str)
@pytest.mark.parametrize("variant", [0, 2, 4])
def test_split_convolution(case, variant):
    """Every output within (K + 2) 2^-24 of its sum |x w| + |b|, the bound of
    any fp32 summation; an infinite and a huge input give what fp32 gives."""
    from numpy.lib.stride_tricks import sliding_window_view
    shape, Co, k = case
    rng = np.random.default_rng(Co)
    x = rng.standard_normal(shape).astype(np.float32)
    w = rng.standard_normal((Co, shape[1], k, k)).astype(np.float32)
    b = rng.standard_normal(Co).astype(np.float32)

    def exact(x, w):
        win = sliding_window_view(x.astype(np.float64), (k, k), axis=(2, 3))
        with np.errstate(all="ignore"):
            return np.einsum("nchwuv,ocuv->nohw", win, w.astype(np.float64))

    ref = exact(x, w) + b[:, None, None]
    bound = (shape[1] * k * k + 2) * 2.0 ** -24 * (exact(np.abs(x), np.abs(w)) + np.abs(b)[:, None, None])
    say("conv", case, variant)
    assert (np.abs(convolution(variant, x, w, b) - ref) <= bound).all()
    x[0, 1, 2, 2], x[0, 2, -1, -1] = np.inf, 3.4e38
    w *= np.float32(2.0 ** -4) * (np.abs(w) < 3)
    ref = exact(x, w) + b[:, None, None]
    got = convolution(variant, x, w, b)
    assert (np.isnan(got) == np.isnan(ref)).all() and (got[np.isinf(ref)] == ref[np.isinf(ref)]).all()
    assert np.isfinite(got[np.isfinite(ref)]).all()


# operand sizes whose bf16 parts, unscaled, would be subnormal or vanish, each
# beside a size that makes the products ordinary floats; the last pair's sums
# leave the range of the scaled accumulator
SIZES = [(1e-31, 1e31), (1e-36, 1e36), (1e-38, 1e37), (1e-40, 1e37), (1e-44, 1e37), (1e36, 1e-36), (1e15, 1e15)]


@pytest.mark.parametrize("sizes", SIZES, ids=str)
@pytest.mark.parametrize("variant", VARIANTS)
def test_split_operand_sizes(sizes, variant):
    """Small, subnormal and large operands: the bound of any fp32 summation
    (plus half the smallest float per product)."""
    rng = np.random.default_rng(9)
    (M, N), K = rows_cols(variant, 132, 136), 68
    x = (sizes[0] * rng.standard_normal((M, K))).astype(np.float32)
    w = (sizes[1] * rng.standard_normal((K, N))).astype(np.float32)
    x[rng.random((M, K)) < 0.1] = 0.0
    exact = x.astype(np.float64) @ w.astype(np.float64)
    bound = (K + 1) * (2.0 ** -24 * (np.abs(x).astype(np.float64) @ np.abs(w)) + 2.0 ** -150)
    say("sizes", sizes, variant)
    assert (np.abs(product(variant, x, w) - exact) <= bound).all()


@pytest.mark.parametrize("sizes", SIZES, ids=str)
@pytest.mark.parametrize("variant", [0, 2, 4])
def test_split_convolution_operand_sizes(sizes, variant):
    from numpy.lib.stride_tricks import sliding_window_view
    rng = np.random.default_rng(10)
    x = (sizes[0] * rng.standard_normal((1, 6, 9, 11))).astype(np.float32)
    w = (sizes[1] * rng.standard_normal((33, 6, 3, 3))).astype(np.float32)

    def exact(x, w):
        win = sliding_window_view(x.astype(np.float64), (3, 3), axis=(2, 3))
        return np.einsum("nchwuv,ocuv->nohw", win, w.astype(np.float64))

    bound = (6 * 9 + 1) * (2.0 ** -24 * exact(np.abs(x), np.abs(w)) + 2.0 ** -150)
    say("conv sizes", sizes, variant)
    got = convolution(variant, x, w, np.zeros(33, np.float32))
    assert (np.abs(got - exact(x, w)) <= bound).all()


@pytest.mark.parametrize("dist", ["normal", "positive", "wide"])
def test_split_convolution_error(dist):
    """The root mean square of the errors against 64-bit arithmetic, in units
    of sum |x w|, no larger than the fp32 MFMA kernel's."""
    from numpy.lib.stride_tricks import sliding_window_view
    rng = np.random.default_rng(11)
    x, w = rng.standard_normal((1, 96, 18, 18)), 0.05 * rng.standard_normal((72, 96, 3, 3))
    if dist == "positive":
        x = np.maximum(x, 0.0)
    elif dist == "wide":
        x, w = x * np.exp(4 * rng.standard_normal(x.shape)), w * np.exp(4 * rng.standard_normal(w.shape))
    x, w = x.astype(np.float32), w.astype(np.float32)

    def exact(x, w):
        win = sliding_window_view(x.astype(np.float64), (3, 3), axis=(2, 3))
        return np.tensordot(win, w.astype(np.float64), ([1, 4, 5], [1, 2, 3])).transpose(0, 3, 1, 2)

    ref, size = exact(x, w), exact(np.abs(x), np.abs(w))
    rms = {}
    for v in (0, 1, 2, 4):
        e = (convolution(v, x, w, np.zeros(72, np.float32)) - ref) / size
        rms[v] = float(np.sqrt((e * e).mean()))
    say("conv error", dist, rms)
    assert all(rms[v] <= rms[1] for v in (0, 2, 4))


@pytest.mark.parametrize("variant", [0, 2, 4])
@pytest.mark.parametrize("case", [((2, 5, 12, 8), (9, 5, 2, 4)), ((1, 6, 7, 40), (35, 6, 3, 1)), ((3, 4, 70, 3), (33, 4, 3, 3))],
                         ids=str)
def test_split_convolution_layouts(case, variant, tmp_path):
    """Rows of pixels along W and, for inputs contiguous along H, along H: tall
    and wide images, several of them, kernels that are not square."""
    from test_gpu_conv import _check, conv_graph
    og, a, c = conv_graph(*case, True)
    L = set(map(tuple, layouts.layout_list(case[0]))), set(map(tuple, layouts.layout_list(og.edge_shape(c))))
    for pa in ((0, 1, 2, 3), (0, 1, 3, 2), (0, 3, 1, 2), (1, 3, 0, 2), (3, 0, 1, 2), (0, 2, 3, 1)):
        for pc in ((0, 1, 2, 3), (0, 1, 3, 2), (0, 2, 3, 1)):
            if pa in L[0] and pc in L[1]:
                say(f"split conv {case} v{variant} x{pa} y{pc}")
                _check(og, {a: pa, c: pc}, {og.producer(c): variant}, tmp_path, sum(case[0]))
