"""Host-side: the shapes that the GPU tests compare with the oracle or with 64
bits reach every fp32 convolution kernel that the plans can return, split and
unsplit, pooled and not."""
import random

import pytest

from paper_2112_15317_amd import sb
from tests.test_gpu_kernels import CONV_SHAPES, FUSED_F32_SHAPES
from tests.test_gpu_split_fp32 import POOL_SHAPES, SHAPES

PASSES = {"forward": sb.SB_PASS_FWD, "data gradient": sb.SB_PASS_BWD_DATA,
          "weight gradient": sb.SB_PASS_BWD_WEIGHT, "pooled forward": sb.SB_PASS_FWD_POOL}


def _form(shape, pass_):
    """Kernel of a pass and whether its reduction is split; None if it is refused."""
    n, c, h, w, k = shape
    if pass_ == sb.SB_PASS_FWD_POOL and (h % 2 or w % 2):
        return None
    d = sb.conv_desc(n, c, h, w, k, sb.SB_F32)
    if sb.sb_conv3x3_workspace_bytes(d, pass_) == sb.SIZE_MAX:
        return None
    name, grid = sb.sb_conv3x3_plan_string(d, pass_).split(" grid=")
    return name, pass_ != sb.SB_PASS_BWD_WEIGHT and not grid.endswith("x1")


def _sweep():
    rng = random.Random(1)
    for _ in range(30000):
        h = rng.choice((1, 2, 3, 4, 5, 7, 8, 9, 14, 16, 20, 32, 40, 64))
        w = h if rng.random() < 0.5 else rng.choice((1, 2, 3, 4, 6, 8, 12, 16, 20, 32, 36, 64))
        n, c, k = (int(2 ** rng.uniform(0, 9)) for _ in range(3))
        yield n, c, h, w, k


@pytest.mark.parametrize("name", PASSES)
def test_every_kernel_is_compared(name):
    p = PASSES[name]
    listed = (FUSED_F32_SHAPES + POOL_SHAPES if name == "pooled forward" else CONV_SHAPES + SHAPES)
    reached = {_form(s, p) for s in listed}
    planned = {}
    for s in _sweep():
        f = _form(s, p)
        if f and (f not in planned or s[0] * s[1] * s[4] < planned[f][0] * planned[f][1] * planned[f][4]):
            planned[f] = s
    missing = {f: s for f, s in planned.items() if f not in reached}
    assert not missing, missing
