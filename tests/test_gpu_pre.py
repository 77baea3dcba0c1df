"""1x1 convolutions with BN + ReLU on the input side over whole 64-channel chunks (`conv_pre_kernel`) against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2003_10688_amd import workloads as wl
from test_gpu_parity import TOL, rel_err, sol  # noqa: F401  (sol: the module fixture)

pytestmark = pytest.mark.gpu

CASES = [
    # N, H, W, input channels, filters, pool, act, residual
    (1, 1, 1, 64, 128, None, "none", False),      # one pixel, one chunk
    (2, 7, 9, 128, 256, None, "relu", True),      # two channel tiles, a last pixel tile that is not full; a residual
    (1, 16, 16, 192, 128, "avg", "none", False),  # windows fill the pixel tiles
    (3, 5, 7, 256, 128, "avg", "none", False),    # odd extents: the last row and column belong to no window; a turn of the ring more
    (1, 6, 4, 320, 384, "max", "relu", False),
    (1, 3, 3, 1024, 128, None, "relu", False),    # the most channels
]


@pytest.mark.parametrize("case", CASES)
def test_pre_activation_1x1(sol, case):  # noqa: F811
    N, H, W, C, K, pool, act, res = case
    pd = wl.pool_desc(pool, 2, 2, 0) if pool else None
    layers = [wl.conv(C, 1, p=0)] + ([wl.conv(K, 1, p=0, src=0)] if res else [])
    layers.append(wl.conv(K, 1, p=0, act=act, bn=True, pool=pd, pre_bn=True, src=0, res=1 if res else -1))
    layers.append(wl.conv(8, 1, p=0, bn=False, act="none"))
    rng = np.random.default_rng([N, H, W, C])
    x = wl.to_bf16_grid(rng.standard_normal((N, 32, H, W)))
    prm = wl.make_params(layers, 32, 4 + K, bf16=True, bias_std=0.3)
    outs, _ = orc.network_forward(layers, prm, x, bf16=True, return_all=True)
    net = sol.Network(layers, x.shape, sol.BF16)
    net.set_params(prm)
    net.workspace.fill_(0xff)                     # NaNs: nothing that was not written may be looked at
    net.forward(sol.to_device_nhwc(x, sol.BF16))
    torch.cuda.synchronize()
    i = len(layers) - 2
    net.run_layer(i, sol.to_device_nhwc(x, sol.BF16))
    torch.cuda.synchronize()
    assert sol.sol_debug_conv_kernel() == "pre"
    assert rel_err(sol.to_host_nchw(net.layer_output(i)).reshape(outs[i].shape), outs[i]) <= TOL["bf16"]


def test_prefix_of_a_wider_tensor(sol):  # noqa: F811
    """Input pitch above the channel count: what lies behind the prefix is not looked at."""
    rng = np.random.default_rng(5)
    C, K = 128, 128
    x = rng.standard_normal((2, 5, 6, C + 64)).astype(np.float32)
    x[..., C:] = np.nan
    w = rng.standard_normal((K, C, 1, 1)).astype(np.float32) * 0.1
    ps, ph = rng.uniform(0.5, 1.5, C).astype(np.float32), rng.uniform(-0.2, 0.2, C).astype(np.float32)
    xd = torch.from_numpy(x).cuda().to(torch.bfloat16)
    cd = sol.ConvDesc(K, C, 1, 1, 1, 1, 0, 0)
    wp = sol.sol_pack_conv_weights(cd, sol.BF16, sol.dev_f32(w))
    y = sol.sol_conv2d_preact_fused(xd, cd, wp, sol.dev_f32(ps), sol.dev_f32(ph), channels=C)
    assert sol.sol_debug_conv_kernel() == "pre"
    t = (xd[..., :C].float() * sol.dev_f32(ps) + sol.dev_f32(ph)).relu().to(torch.bfloat16).double()
    want = t.reshape(-1, C) @ torch.from_numpy(w).cuda().to(torch.bfloat16).double().reshape(K, C).T
    assert rel_err(y.float().cpu().numpy().reshape(-1, K), want.cpu().numpy()) <= TOL["bf16"]


@pytest.mark.parametrize("c,k,tile,kernel", [(128, 128, 0, "pre"), (128, 128, 2, ""), (96, 128, 0, ""), (128, 96, 0, ""), (1024, 128, 0, "pre"), (1088, 128, 0, "")])
def test_which_kernel(sol, c, k, tile, kernel):  # noqa: F811
    """Whole 64-channel chunks up to 1024, multiples of 128 filters, no tile asked for; what the register-staged kernel computes, bit for bit."""
    layers = [wl.conv(k, 1, p=0, act="none", bn=False, pre_bn=True)]
    net = sol.Network(layers, (2, c, 9, 7), sol.BF16)
    net.set_params(wl.make_params(layers, c, 3, bf16=True, bias_std=0.3))
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(c)
    x = torch.randn((2, 9, 7, c), generator=gen, device="cuda:0").bfloat16()
    net.set_tiles({0: tile})
    y = net.forward(x).clone()
    assert sol.sol_debug_conv_kernel() == kernel
    net.set_tiles({0: 99})
    assert torch.equal(y, net.forward(x)) and sol.sol_debug_conv_kernel() == ""
