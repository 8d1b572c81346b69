"""Convolutions on the fp32 matrix instruction (any channel count, fp32 and bf16 storage), layer by layer against the oracle."""
import pytest

from oracle import nets

from gpu_util import Case
from test_gpu_step import check_layers

pytestmark = pytest.mark.gpu

SHAPES = {
    # four channels per load, one and two column tiles of 16, 128-row tiles with a ragged last one (66 * 32 * 32 rows)
    "vec4_tall": (dict(kind=1, widths=[12, 20], blocks=[1, 1], stem_width=12), lambda: nets.resnet20(widths=(12, 20), blocks=(1, 1)),
                  66, 32),
    # one channel per load: odd channel counts, ragged tiles in every dimension
    "scalar": (dict(kind=1, widths=[5, 33], blocks=[1, 1], stem_width=5), lambda: nets.resnet20(widths=(5, 33), blocks=(1, 1)), 3, 13),
    # more than 64 columns and a contraction of many taps; fewer pixels than one step of the weight gradient
    "columns": (dict(kind=1, widths=[68, 132], blocks=[1, 1], stem_width=68), lambda: nets.resnet20(widths=(68, 132), blocks=(1, 1)),
                1, 7),
    # 7x7 stride-2 stem on odd images, 1x1 filters with and without stride
    "bottleneck": (dict(kind=2, widths=[6, 12], blocks=[1, 1], stem_width=20),
                   lambda: nets.resnet50(classes=10, widths=(6, 12), blocks=(1, 1), stem=20), 5, 37),
    # 4100 channels into the average pool: more vectors than one block takes
    "many_channels": (dict(kind=2, widths=[1025], blocks=[1], stem_width=4),
                      lambda: nets.resnet50(classes=10, widths=(1025,), blocks=(1,), stem=4), 2, 16),
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", list(SHAPES))
def test_generic_convolutions_layers(name, dtype):
    kw, mk, batch, res = SHAPES[name]
    c = Case(kw, mk(), dtype, batch, res, 10)
    check_layers(c, c.gpu())
