"""Causal attention with more tiles than two rounds of the 256 compute units,
whose P V tiles are enumerated from the longest row to the shortest with every
second round reversed: every output tile is produced once, whatever the tile
shape, with whole and partial rounds, against the oracle."""
import os
import subprocess

import pytest

from gpu_util import say
from test_gpu_ops import _check_gemm, causal_attn_graph

S, D = 264, 32
ROWS = {"f32": {0: 128, 1: 64, 2: 32, 4: 64, 6: 16, 7: 32}, "bf16": {0: 128, 1: 64, 2: 32, 3: 32, 4: 64, 6: 256, 7: 128, 8: 256}}


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,variant", [(d, v) for d in ROWS for v in ROWS[d]])
def test_causal_tile_order(dtype, variant, tmp_path):
    per_head = -(-S // ROWS[dtype][variant])
    heads = 512 // per_head + 3
    tiles = heads * per_head
    assert tiles >= 512 and tiles % 256 != 0
    og, q, k, s, p, o = causal_attn_graph(1, heads, S, D, dtype)
    # P row-major, its rows contiguous, and (tiles that take it) its heads
    for lay in [(0, 1, 2, 3), (0, 1, 3, 2), (0, 2, 3, 1)]:
        say(f"causal order {dtype} v{variant} {heads} heads {lay}")
        lp = _check_gemm(og, {p: lay}, {4: variant}, tmp_path, 3, dtype)
        assert lp is not None or lay != (0, 1, 2, 3)


PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "kparams.h"
int main(int, char** a) {
  const uint32_t m = atoi(a[1]), n = atoi(a[2]), G = atoi(a[3]);
  for (uint32_t b = 0; b < m * n * G; ++b) printf("%u\n", fluid::longest_first(b, m, n, G));
}
"""


def test_causal_order_is_a_bijection(tmp_path):
    """The workgroup -> tile map, compiled for the host: every tile once, in
    rounds of 256 from the longest tile row to the shortest."""
    host = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2411_09242_amd", "csrc", "host")
    src = tmp_path / "order.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "order")
    subprocess.run(["g++", "-std=c++17", "-I", host, str(src), "-o", exe], check=True)
    for tm, tn, G in ((8, 1, 32), (17, 1, 40), (9, 3, 33), (5, 2, 1), (1, 1, 700), (33, 4, 24), (2, 1, 300)):
        out = subprocess.run([exe, str(tm), str(tn), str(G)], check=True, capture_output=True, text=True).stdout
        order = [int(t) for t in out.split()]
        assert sorted(order) == list(range(tm * tn * G))
        rows = [t // tn % tm for t in order]
        for r in range(0, len(rows) - 256, 256):
            assert min(rows[r:r + 256]) >= max(rows[r + 256:r + 512])
