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
    (1, 7, 7, 8, 7, 2, None, "relu"),          # 7x7 filters stay on the gather and stem kernels
    (2, 31, 22, 64, 7, 2, None, "none"),
]
PADDINGS = [
    # N, H, W, filters, stride, padding
    (2, 9, 12, 32, 1, 0), (1, 7, 8, 20, 1, 2), (1, 11, 7, 12, 2, 0), (3, 8, 5, 36, 2, 2), (2, 13, 9, 8, 2, 1)
]


def check(sol, layers, shape, bf16, seed, kernel):  # noqa: F811
    rng = np.random.default_rng(seed)
    x = rng.standard_normal(shape).astype(np.float32)
    if bf16:
        x = wl.to_bf16_grid(x)
    prm = wl.make_params(layers, 3, 2 + layers[0]["cout"], bf16=bf16, bias_std=0.3)
    want = orc.network_forward(layers, prm, x, bf16=bf16)
    net = sol.Network(layers, x.shape, sol.BF16 if bf16 else sol.F32)
    net.set_params(prm)
    y = net.forward(sol.to_device_nhwc(x, net.dt))
    torch.cuda.synchronize()
    assert sol.sol_debug_conv_kernel() == kernel
    assert rel_err(sol.to_host_nchw(y).reshape(want.shape), want) <= TOL["bf16" if bf16 else "f32"]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES)
def test_three_channels(sol, case, dtype):  # noqa: F811
    N, H, W, K, k, s, pool, act = case
    bf16 = dtype == "bf16"
    pd = wl.pool_desc(pool, 2, 2, 0) if pool else None
    layers = [wl.conv(K, k, s=s, act=act, pool=pd)]
    check(sol, layers, (N, 3, H, W), bf16, [N, H, W, K], "small" if k == 3 and not (bf16 and s == 2) else "")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", PADDINGS)
def test_paddings_and_strides(sol, case, dtype):  # noqa: F811
    """No padding, a ring of outputs that see the padding only, odd extents under stride 2 (fp32; in bf16 the other kernels')."""
    N, H, W, K, s, p = case
    check(sol, [wl.conv(K, 3, s=s, p=p)], (N, 3, H, W), dtype == "bf16", [N, H, W, K, p], "" if dtype == "bf16" and s == 2 else "small")


@pytest.mark.parametrize("dtype,n,hw,k,pool,kernel", [
    ("bf16", 8, 64, 64, None, "small"), ("bf16", 8, 65, 64, None, ""), ("bf16", 1, 224, 64, None, ""), ("bf16", 1, 224, 64, "max", "small"), ("bf16", 1, 224, 96, None, "small"),
    ("bf16", 1, 180, 96, None, ""), ("bf16", 1, 224, 68, None, "small"), ("bf16", 4, 100, 256, None, ""), ("bf16", 16, 112, 32, None, "small"),
    ("f32", 1, 224, 256, None, "small"), ("f32", 8, 224, 256, None, ""), ("f32", 8, 224, 224, None, "small"), ("f32", 8, 224, 256, "avg", "small")])
def test_which_kernel(sol, dtype, n, hw, k, pool, kernel):  # noqa: F811
    """Full channel tiles of many pixels stay on the gather kernel, which was up to 1.6 times faster there; it is then what runs, bit for bit."""
    layers = [wl.conv(k, 3, pool=wl.pool_desc(pool, 2, 2, 0) if pool else None)]
    net = sol.Network(layers, (n, 3, hw, hw), sol.BF16 if dtype == "bf16" else sol.F32)
    net.set_params(wl.make_params(layers, 3, 1, bf16=dtype == "bf16"))
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(k)
    x = torch.randn((n, hw, hw, 3), generator=gen, device="cuda:0").to(sol.torch_dtype(net.dt))
    y = net.forward(x).clone()
    assert sol.sol_debug_conv_kernel() == kernel
    net.set_tiles({0: 99})                       # the general kernels
    general = net.forward(x)
    assert sol.sol_debug_conv_kernel() == ""
    assert torch.equal(y, general) or kernel == "small"
    assert rel_err(y.float().cpu().numpy(), general.float().cpu().numpy()) <= TOL[dtype]


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
