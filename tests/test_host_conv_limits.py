"""Which convolution kernel a variant prepares by the input's size (host
library): the split kernels address their operands by buffer loads, below
2 GiB; a larger input runs the fp32 kernel after them."""
import json

import pytest

from paper_2411_09242_amd import fluid as F

# 64 channels, 32-bit: 4 * 64 * H * W bytes
BELOW, ABOVE = (2896, 2896), (2897, 2896)
KERNELS = {0: ("conv_f32_s128x64_kcuv_ks4", "conv_f32_t64_kuvc"), 2: ("conv_f32_s64x64_kcuv_ks4", "conv_f32_t64_kuvc_ks4"),
           4: ("conv_f32_s64x32_kcuv_ks8", "conv_f32_t32_kuvc_ks8")}


@pytest.mark.parametrize("variant", sorted(KERNELS))
def test_split_convolution_limit(variant, tmp_path):
    F.load(host_only=True)
    for image, large in ((BELOW, 0), (ABOVE, 1)):
        assert (4 * 64 * image[0] * image[1] >= 0x7fffffff) == bool(large)
        x, w = [1, 64, *image], [8, 64, 3, 3]
        y = [1, 8, image[0] - 2, image[1] - 2]
        eye = [0, 1, 2, 3]
        g = F.Graph.from_desc(dict(dtype="f32", inputs=[x], consts=[dict(role="weight", shape=w, dtype="f32")],
                                   nodes=[dict(op="conv", ins=[0, ~0], out_shape=y)], outputs=[1]))
        path = tmp_path / "t.json"
        path.write_text(json.dumps({
            "format": "fluid-cost-table/1", "edges": [[eye], [eye]], "node_sig": [0],
            "sigs": [{"op": "conv", "in_shapes": [x], "out_shape": y,
                      "entries": [[[eye], eye, [1 if v == variant else -1 for v in range(6)]]]}]}))
        lp = F.LayoutPlan(g, F.CostTable.load(str(path), g))
        assert lp.kernel(0) == KERNELS[variant][large]
