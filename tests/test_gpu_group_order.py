"""Grouped convolutions whose workgroups run the groups innermost (small groups,
or images that outweigh the weights) or outermost, against the fp64 oracle: a
group of several column tiles, one pixel row tile, stride phases of different
sizes, more than one split of backward-weight, and both sides of the rule."""
import numpy as np
import pytest

import gpu_util as U
from paper_2102_06725_amd import inputs as I

pytestmark = pytest.mark.gpu

SHAPES = [
    # name, n, c, h, w, k, r, stride, pad, groups
    ("inner_8x3", 2, 24, 9, 11, 24, 3, 1, 1, 3),
    ("inner_24x4_k40", 8, 96, 28, 27, 160, 3, 1, 1, 4),
    ("inner_72x2_k104", 4, 144, 30, 31, 208, 1, 1, 0, 2),    # two column tiles per group
    ("inner_8x5_s2", 4, 40, 57, 55, 80, 3, 2, 1, 5),         # phases of different sizes
    ("inner_16x3_s3", 2, 48, 31, 32, 48, 5, 3, 2, 3),        # one launch per phase
    ("inner_64x2_s2", 8, 128, 56, 56, 128, 3, 2, 1, 2),
    ("inner_sg8", 4, 128, 56, 56, 128, 3, 1, 1, 16),
    ("outer_64x3", 1, 192, 14, 13, 192, 3, 1, 1, 3),
    ("outer_128x2_s2", 2, 256, 28, 28, 256, 3, 2, 1, 2),
    ("outer_136x2", 2, 272, 20, 21, 272, 1, 1, 0, 2),        # past 128 channels
]


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("s", SHAPES, ids=[s[0] for s in SHAPES])
def test_group_order_parity(nnlib, oracle_lib, s, dtype):
    name, n, c, h, w, k, r, stride, pad, groups = s
    case = U.Case(I.Layer(name, n, c, h, w, k, r, r, stride, pad, 1, groups), layout="nhwc",
                  dtype=dtype, x_kind="normal", cfg=95, layer_id=SHAPES.index(s), alpha=0.75)
    t = case.tensors()
    a, b = U.run_gpu(case, t), U.run_gpu(case, t)
    for key in ("y_bits", "dx_bits"):
        assert np.array_equal(a[key], b[key]), key
    U.full_parity(case)
