"""The depth-first dense-layer kernel (BN + ReLU, 1x1 to 128 channels, BN + ReLU, 3x3 to 32 channels in one launch) in each of
its patch sizes, inside plans that write the features of a dense block into one buffer, against the CPU checker."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2003_10688_amd import workloads as wl
from test_gpu_parity import TOL, rel_err, sol  # noqa: F401  (sol: the module fixture)

pytestmark = pytest.mark.gpu

CASES = [
    # N, H, W, block input channels, dense layers
    (1, 1, 1, 64, 2),        # one pixel: every tap but one in the padding
    (5, 7, 7, 96, 3),        # a prefix that is no whole chunk of 64 channels: masked; many images to a tile
    (2, 14, 13, 160, 2),
    (1, 3, 61, 64, 2),       # wide rows: the larger patches only
    (1, 2, 130, 128, 1),     # halo as large as the patch allows
    (1, 3, 183, 64, 1),      # the widest image: 16 pixels to a patch of 384 rows
    (1, 5, 9, 992, 1),       # sixteen chunks, the last one half masked
]


@pytest.mark.parametrize("variant", [0, 91, 92, 93, 94, 95, 96])
@pytest.mark.parametrize("case", CASES)
def test_dense_layer(sol, case, variant):  # noqa: F811
    N, H, W, C, depth = case
    layers = [wl.conv(C, 1, p=0)]
    feat, dense = 0, []
    for _ in range(depth):
        layers.append(wl.conv(128, 1, p=0, src=feat, pre_bn=True))
        layers.append(wl.conv(32, 3, bn=False, act="none"))
        dense.append(len(layers) - 1)
        layers.append(wl.concat(feat, len(layers) - 1))
        feat = len(layers) - 1
    layers.append(wl.conv(40, 1, p=0, bn=False, act="none"))
    rng = np.random.default_rng([variant, N, H, W, C])
    x = wl.to_bf16_grid(rng.standard_normal((N, 64, H, W)))
    prm = wl.make_params(layers, 64, 3 + C, bf16=True, bias_std=0.3)
    outs, _ = orc.network_forward(layers, prm, x, bf16=True, return_all=True)
    net = sol.Network(layers, x.shape, sol.BF16)
    net.set_params(prm)
    net.workspace.fill_(0xff)                    # NaNs: nothing of what lies behind a prefix may be looked at
    xd = sol.to_device_nhwc(x, sol.BF16)
    net.forward(xd)
    assert [net.fused_into(i - 1) for i in dense] == dense
    if variant:
        net.workspace.fill_(0xff)
        for i in range(len(layers)):
            sol.sol_debug_set_conv_tile(variant if i in dense else 0)
            try:
                net.run_layer(i, xd)
            finally:
                sol.sol_debug_set_conv_tile(0)
    torch.cuda.synchronize()
    # the last convolution sums the features of every layer; two roundings (t1, the feature) lie between it and the input
    assert rel_err(sol.to_host_nchw(net.y).reshape(outs[-1].shape), outs[-1]) <= TOL["bf16"]


@pytest.mark.parametrize("variant", [91, 92, 93, 94, 95, 96])
def test_dense_layer_infinity(sol, variant):  # noqa: F811
    """One pixel of the 1x1's output overflows to +inf: the 3x3 window around it is +inf (its weights are positive), all else finite."""
    N, H, W, C = 2, 9, 11, 64
    layers = [wl.conv(C, 1, p=0, bn=False, act="none"), wl.conv(128, 1, p=0, src=0, pre_bn=True), wl.conv(32, 3, bn=False, act="none"), wl.concat(0, 2),
              wl.conv(8, 1, p=0, bn=False, act="none")]
    rng = np.random.default_rng(variant)
    prm = wl.make_params(layers, 64, 7, bf16=True)
    prm[0]["w"] = np.eye(64, dtype=np.float32).reshape(64, 64, 1, 1)
    prm[1]["w"][:] = np.abs(prm[1]["w"])
    prm[1]["w"][1:, 0] = 0.0                     # the huge input channel reaches one of the 128 channels only
    prm[1]["w"][0, 0] = 2.0 ** 120
    prm[2]["w"][:] = np.abs(prm[2]["w"])
    x = wl.to_bf16_grid(np.abs(rng.standard_normal((N, 64, H, W))))
    x[:, 0] = 0.0
    prm[1]["pre_beta"][0] = prm[1]["pre_mean"][0] = 0.0
    x[1, 0, 4, 6] = 2.0 ** 100
    net = sol.Network(layers, x.shape, sol.BF16)
    net.set_params(prm)
    xd = sol.to_device_nhwc(x, sol.BF16)
    net.forward(xd)
    assert net.fused_into(1) == 2
    sol.sol_debug_set_conv_tile(variant)
    try:
        net.run_layer(2, xd)
    finally:
        sol.sol_debug_set_conv_tile(0)
    torch.cuda.synchronize()
    y = sol.to_host_nchw(net.layer_output(3))[:, 64:]        # the new features, written in place behind the block's input
    inside = np.zeros(y.shape, bool)
    inside[1, :, 3:6, 5:8] = True
    assert np.isposinf(y[inside]).all() and np.isfinite(y[~inside]).all()


@pytest.mark.parametrize("case", [(5, 7, 7, 96), (1, 3, 183, 64), (16, 20, 160, 64)])
def test_dense_layer_two_launches(sol, case):  # noqa: F811
    """The same layer one by one, as one launch, in the plan's own choice and in the auto-tuner's."""
    N, H, W, C = case
    layers = [wl.conv(C, 1, p=0), wl.conv(128, 1, p=0, src=0, pre_bn=True), wl.conv(32, 3, bn=False, act="none"), wl.concat(0, 2),
              wl.conv(8, 1, p=0, bn=False, act="none")]
    x = wl.to_bf16_grid(np.random.default_rng(case).standard_normal((N, 64, H, W)))
    prm = wl.make_params(layers, 64, 3 + C, bf16=True, bias_std=0.3)
    outs, _ = orc.network_forward(layers, prm, x, bf16=True, return_all=True)
    net = sol.Network(layers, x.shape, sol.BF16)
    net.set_params(prm)
    assert net.dense_state(2) == (W != 160)                 # 51200 pixels of images 160 wide are more than one round of tiles
    xd = sol.to_device_nhwc(x, sol.BF16)
    for choice in (0, 1, "tuned", "restored"):
        if choice == "tuned":
            tiles = net.autotune(xd, reps=2)
            assert tiles["2d"] == net.dense_state(2)
        elif choice == "restored":
            net.set_tiles(tiles)
            assert tiles["2d"] == net.dense_state(2)
        else:
            net.set_dense(2, choice)
        net.workspace.fill_(0xff)
        net.forward(xd)
        torch.cuda.synchronize()
        assert rel_err(sol.to_host_nchw(net.y).reshape(outs[-1].shape), outs[-1]) <= TOL["bf16"], choice
        if choice == 0:
            assert rel_err(sol.to_host_nchw(net.layer_output(1)), outs[1]) <= TOL["bf16"]


def test_dense_layer_tiles_are_used(sol):  # noqa: F811
    """Tiles set for, or forced on, the two convolutions of a dense layer are used (and one that cannot apply is refused)."""
    layers = [wl.conv(64, 1, p=0), wl.conv(128, 1, p=0, src=0, pre_bn=True), wl.conv(32, 3, bn=False, act="none"), wl.concat(0, 2),
              wl.conv(8, 1, p=0, bn=False, act="none")]
    x = wl.to_bf16_grid(np.random.default_rng(4).standard_normal((3, 64, 9, 10)))
    prm = wl.make_params(layers, 64, 5, bf16=True, bias_std=0.3)
    outs, _ = orc.network_forward(layers, prm, x, bf16=True, return_all=True)
    net = sol.Network(layers, x.shape, sol.BF16)
    net.set_params(prm)
    xd = sol.to_device_nhwc(x, sol.BF16)

    def check():
        net.workspace.fill_(0xff)
        net.forward(xd)
        torch.cuda.synchronize()
        assert rel_err(sol.to_host_nchw(net.y).reshape(outs[-1].shape), outs[-1]) <= TOL["bf16"]
        assert rel_err(sol.to_host_nchw(net.layer_output(1)), outs[1]) <= TOL["bf16"]       # stored: two launches

    net.set_tiles({1: 3, 2: 6})
    check()
    sol.sol_debug_set_conv_tile(5)
    try:
        net.set_tiles({})
        check()
    finally:
        sol.sol_debug_set_conv_tile(0)
    net.set_tiles({1: 11})                                   # a DMA ring tile cannot apply BN + ReLU to its input
    with pytest.raises(sol.SolError) as e:
        net.forward(xd)
    assert e.value.status == 6


def test_dense_layer_static_workspace(sol):  # noqa: F811
    """A pass that stores no 1x1 output needs no buffer for it: 31 MiB of the static workspace's 32 do, 55 would not."""
    layers = [wl.conv(64, 1, p=0), wl.conv(128, 1, p=0, src=0, pre_bn=True), wl.conv(32, 3, bn=False, act="none"), wl.concat(0, 2),
              wl.conv(8, 1, p=0, bn=False, act="none")]
    net = sol.Network(layers, (32, 64, 56, 56), sol.BF16)
    net.set_params(wl.make_params(layers, 64, 9, bf16=True))
    x = torch.randn((32, 56, 56, 64), device="cuda:0").bfloat16()
    y = net.forward(x).clone()
    net.y.zero_()
    assert torch.equal(net.forward_static(x), y)
    net.set_dense(2, 0)
    with pytest.raises(sol.SolError) as e:
        net.forward_static(x)
    assert e.value.status == 5
    net.workspace = net.workspace[:net.workspace.numel() - 32 * 56 * 56 * 128 * 2]      # one launch: accepted, and left alone by the auto-tuner
    net.set_dense(2, 1)
    assert torch.equal(net.forward(x), y) and net.autotune(x, reps=1)["2d"] == 1


@pytest.mark.parametrize("variant", [91, 92, 93, 94, 95, 96])
@pytest.mark.parametrize("C", [64, 128, 192, 224, 256, 320, 384, 448, 576])
def test_dense_layer_chunk_counts(sol, C, variant):  # noqa: F811
    """Every number of chunks that the pipeline of x chunks and weight stages starts and drains differently for: fewer than are in flight,
    and each remainder of the register sets behind whole turns of them.  Two rows of images, so that patches reach over their borders."""
    layers = [wl.conv(C, 1, p=0), wl.conv(128, 1, p=0, src=0, pre_bn=True), wl.conv(32, 3, bn=False, act="none"), wl.concat(0, 2),
              wl.conv(8, 1, p=0, bn=False, act="none")]
    rng = np.random.default_rng([variant, C])
    x = wl.to_bf16_grid(rng.standard_normal((3, 64, 9, 10)))
    prm = wl.make_params(layers, 64, 5 + C, bf16=True, bias_std=0.3)
    outs, _ = orc.network_forward(layers, prm, x, bf16=True, return_all=True)
    net = sol.Network(layers, x.shape, sol.BF16)
    net.set_params(prm)
    net.workspace.fill_(0xff)
    xd = sol.to_device_nhwc(x, sol.BF16)
    net.forward(xd)
    assert net.fused_into(1) == 2
    sol.sol_debug_set_conv_tile(variant)
    try:
        net.run_layer(2, xd)
    finally:
        sol.sol_debug_set_conv_tile(0)
    torch.cuda.synchronize()
    assert rel_err(sol.to_host_nchw(net.layer_output(3)), outs[3]) <= TOL["bf16"]
