"""Convolutions of three input channels on the vector units (`conv_small_kernel`) against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2003_10688_amd import workloads as wl
from test_gpu_parity import TOL, rel_err, sol  # noqa: F401  (sol: the module fixture)

pytestmark = pytest.mark.gpu

CASES = [
    # N, H, W, filters, filter, stride, pool, act
    (1, 1, 1, 8, 3, 1, None, "relu"),          # one pixel: every tap but one in the padding
    (1, 2, 3, 16, 3, 1, "max", "relu"),        # one pooling window
    (3, 9, 7, 24, 3, 1, "max", "none"),        # odd extents: the last row and column belong to no window
    (2, 8, 13, 40, 3, 1, "avg", "relu"),
    (5, 11, 10, 68, 3, 1, None, "none"),       # several rows of channel groups, the last one partly empty
    (2, 9, 12, 32, 3, 2, None, "relu"),
    (1, 7, 7, 8, 7, 2, None, "relu"),
    (2, 31, 22, 64, 7, 2, None, "none"),       # strips of four pixels with a remainder
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES)
def test_three_channels(sol, case, dtype):  # noqa: F811
    N, H, W, K, k, s, pool, act = case
    bf16 = dtype == "bf16"
    pd = wl.pool_desc(pool, 2, 2, 0) if pool else None
    layers = [wl.conv(K, k, s=s, act=act, pool=pd)]
    rng = np.random.default_rng([N, H, W, K])
    x = rng.standard_normal((N, 3, H, W)).astype(np.float32)
    if bf16:
        x = wl.to_bf16_grid(x)
    prm = wl.make_params(layers, 3, 2 + K, bf16=bf16, bias_std=0.3)
    want = orc.network_forward(layers, prm, x, bf16=bf16)
    net = sol.Network(layers, x.shape, sol.BF16 if bf16 else sol.F32)
    net.set_params(prm)
    y = net.forward(sol.to_device_nhwc(x, net.dt))
    torch.cuda.synchronize()
    assert rel_err(sol.to_host_nchw(y).reshape(want.shape), want) <= TOL[dtype]


def test_infinity_and_nan(sol):  # noqa: F811
    """An infinity reaches the 3x3 outputs around it and no others; a NaN becomes 0 behind a ReLU, as in the other kernels."""
    layers = [wl.conv(8, 3, bn=False)]
    prm = wl.make_params(layers, 3, 1)
    prm[0]["w"][:] = 0.5
    x = np.ones((1, 3, 8, 9), dtype=np.float32)
    x[0, 1, 2, 3], x[0, 2, 6, 7] = np.inf, np.nan
    net = sol.Network(layers, x.shape, sol.F32)
    net.set_params(prm)
    y = sol.to_host_nchw(net.forward(sol.to_device_nhwc(x, sol.F32)))[0]
    inf, nan = np.zeros((8, 9), dtype=bool), np.zeros((8, 9), dtype=bool)
    inf[1:4, 2:5], nan[5:8, 6:9] = True, True
    assert np.isposinf(y[:, inf]).all() and (y[:, nan] == 0).all() and np.isfinite(y[:, ~inf]).all() and (y[:, ~inf & ~nan] > 0).all()
