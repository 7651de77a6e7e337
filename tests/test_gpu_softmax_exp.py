"""The exponential of the bf16 softmax is as accurate as an fp32 one, in every
kernel variant: the share of stored values that differ from the exact result
rounded to bf16, far below the maximum and down to bf16's subnormals."""
import json

import numpy as np
import pytest

from gpu_util import say
from oracle import numerics

pytestmark = pytest.mark.gpu


def softmax(variant, x, tmp_path):
    import torch
    from paper_2411_09242_amd import fluid as F
    shape = list(x.shape)
    eye = list(range(len(shape)))
    g = F.Graph.from_desc(dict(dtype="bf16", inputs=[shape], consts=[], outputs=[1],
                               nodes=[dict(op="softmax", ins=[0], out_shape=shape, fattr=1.0, iattr=0)]))
    table = {"format": "fluid-cost-table/1", "edges": [[eye], [eye]], "node_sig": [0],
             "sigs": [{"op": "softmax", "in_shapes": [shape], "out_shape": shape,
                       "entries": [[[eye], eye, [1 if v == variant else -1 for v in range(3)]]]}]}
    path = tmp_path / "t.json"
    path.write_text(json.dumps(table))
    lp = F.LayoutPlan(g, F.CostTable.load(str(path), g))
    ex = F.Executor(g, lp, F.ArenaPlan(g, lp), [], [torch.from_numpy(x)])
    y = ex.run()[0]
    torch.cuda.synchronize()
    return y.double().cpu().numpy()


# the row variants hold 4096 values, the workgroup-per-row one 16-byte pieces
@pytest.mark.parametrize("variant,row", [(0, 2048), (0, 1001), (1, 2048), (1, 1001), (1, 9000), (2, 2048)])
def test_softmax_exponential(row, variant, tmp_path):
    rng = np.random.default_rng(row)
    x = numerics.round_bf16(rng.uniform(-80.0, -60.0, (1, 400, row)))
    # a maximum of its own per row: some 20000 distinct differences
    x[..., 0] = numerics.round_bf16(rng.uniform(0.125, 1.0, (1, 400)))
    x[..., 1] = -90.0        # e^-90 is subnormal in fp32 and bf16
    x[..., 2] = -np.inf
    e = np.exp(x - x[..., :1])
    want = e / e.sum(-1, keepdims=True)
    got = softmax(variant, x.astype(np.float32), tmp_path)
    assert (got[..., 2] == 0).all()
    assert (np.abs(got[..., 1] - want[..., 1]) <= 2.0 ** -133).all()   # one place of a bf16 subnormal
    # an error of 2^-21.5 (the exponential, the sum, its reciprocal and the
    # product) crosses a rounding boundary, 2^-8 apart at least, for 2^-13.5
    # of the values
    off = got[..., 3:] != numerics.round_bf16(want[..., 3:])
    say("softmax exponential", row, variant, off.mean())
    assert off.mean() <= 2.0 ** -13.5
    x[0, 3, 5] = np.nan
    assert np.isnan(softmax(variant, x.astype(np.float32), tmp_path)[0, 3]).all()
