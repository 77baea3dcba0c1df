"""Weight gradients of the fp32 kernel (whole 16-byte slots of channels) and of the general kernel (any channels, columns run
over taps and channels) against the CPU checker's training step: tile and reduction remainders on both sides."""
import numpy as np
import pytest
import torch  # noqa: F401

from paper_2003_10688_amd import workloads as wl
from test_gpu_training import compare, gpu_train, oracle_train, sol  # noqa: F401  (sol: the module fixture)

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, N, C, H, W, K, k, s, p
    ("f32", 1, 4, 1, 1, 4, 1, 1, 0),          # one pixel, one slot of columns
    ("f32", 3, 64, 1, 11, 64, 1, 1, 0),       # one full tile, one pixel more than a round of 32
    ("f32", 2, 12, 9, 7, 68, 3, 1, 1),        # 108 columns, 68 filters: a remainder of both
    ("f32", 5, 36, 11, 13, 132, 5, 2, 2),     # stride 2, 900 columns, slots that change the tap inside a tile
    ("f32", 2, 8, 6, 5, 8, 3, 1, 2),          # padding wider than the filter needs
    ("f32", 9, 128, 8, 8, 64, 3, 2, 1),       # several splits
    ("f32", 3, 3, 23, 21, 64, 7, 2, 3),       # general kernel: 147 columns
    ("f32", 2, 5, 9, 9, 70, 3, 1, 1),
    ("bf16", 2, 5, 9, 9, 70, 3, 1, 1),
    ("bf16", 3, 30, 7, 12, 9, 5, 2, 2),       # 750 columns, fewer filters than a tile
]


@pytest.mark.parametrize("case", CASES)
def test_weight_gradient(sol, case):  # noqa: F811
    dt, N, C, H, W, K, k, s, p = case
    layers = [wl.conv(K, k, s=s, p=p, bn=False, act="none"), wl.gap(), wl.linear(10)]
    params = wl.make_params(layers, C, 17 + C, dt == "bf16", bias_std=0.2)
    x = wl.make_input((N, C, H, W), 5 + K, "normal", dt == "bf16")
    labels = wl.make_labels(N, 10, 3)
    _, got = gpu_train(sol, layers, params, x, labels, dt)
    ref = oracle_train(layers, params, x, labels, dt)
    compare(got[0], ref[0], layers, dt, elementwise=dt == "f32", tag=str(case))
