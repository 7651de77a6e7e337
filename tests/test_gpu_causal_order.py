"""Causal attention with more tiles than two rounds of the 256 compute units,
whose P V tiles are enumerated from the longest row to the shortest with every
second round reversed: every output tile is produced once, whatever the tile
shape, with whole and partial rounds, against the oracle."""
import pytest

from gpu_util import say
from test_gpu_ops import _check_gemm, causal_attn_graph


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,variants", [("f32", (1, 2, 4, 6, 7)), ("bf16", (0, 1, 2, 3, 6, 7, 8))])
@pytest.mark.parametrize("shape", [(1, 40, 520, 32), (3, 11, 257, 72)], ids=str)
def test_causal_tile_order(dtype, variants, shape, tmp_path):
    og, q, k, s, p, o = causal_attn_graph(*shape, dtype)
    for v in variants:
        say(f"causal order {dtype} {shape} v{v}")
        _check_gemm(og, {}, {4: v}, tmp_path, 3, dtype)


def test_causal_order_is_a_bijection():
    """The workgroup -> tile map, on the CPU."""
    for tm, tn, G in ((8, 1, 32), (17, 1, 40), (9, 3, 33), (5, 2, 1), (1, 1, 700), (33, 4, 24)):
        total, per_m, seen = tm * tn * G, tn * G, set()
        for bid in range(total):
            i = bid ^ 248 if bid & 256 and (bid | 255) < total else bid
            m, q = divmod(i, per_m)
            t, g = divmod(q, G)
            seen.add((g * tm + tm - 1 - m) * tn + t)
        assert seen == set(range(total))
