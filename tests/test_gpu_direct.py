"""The small-tile kernel for layers with few output pixels (reduction split over the waves of a workgroup) in each of its
tile shapes against the CPU checker, at the edges of its tiles and of its reduction split."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2003_10688_amd import workloads as wl
from test_gpu_parity import TOL, make_block, rel_err, run_block, sol  # noqa: F401  (sol: the module fixture)

pytestmark = pytest.mark.gpu

TILES = [81, 82, 83, 84, 85]
CASES = [
    # N, C, H, W, K, k, s, p, res, pool
    (1, 64, 1, 1, 10, 1, 1, 0, False, None),        # one pixel, one reduction stage (bf16): three of the four waves have none
    (1, 64, 7, 7, 520, 3, 1, 1, True, None),        # nine taps, ragged channels
    (2, 128, 14, 14, 80, 1, 1, 0, True, None),      # two stages (bf16): half of the waves idle
    (3, 192, 9, 11, 136, 3, 2, 1, False, None),     # stride, 27 stages over four waves
    (5, 64, 5, 3, 33, 5, 1, 2, False, None),        # 25 taps, channels not a multiple of 4, images narrower than the filter
    (130, 64, 2, 2, 64, 3, 1, 1, True, None),       # many tiny images in one pixel tile
    (2, 64, 9, 10, 72, 3, 1, 1, False, "max"),      # fused 2x2 pools over an odd extent
    (2, 64, 9, 10, 70, 1, 1, 0, False, "avg"),
    (2, 64, 3, 3, 16, 1, 1, 1, True, None),         # padded 1x1: pixels whose every tap is padding
]


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES)
def test_direct_tiles(sol, dt, case, tile):  # noqa: F811
    N, C, H, W, K, k, s, p, res, pool = case
    rng = np.random.default_rng([tile, N, C, H, K, k, s])
    l, x, prm, r = make_block(sol, rng, dt, N, C, H, W, K, k, s, p, res=res, pool=wl.pool_desc(pool, 2, 2, 0) if pool else None)
    want = orc.fused_conv(x, prm, l, r, bf16=(dt == "bf16"))[0]
    sol.sol_debug_set_conv_tile(tile)
    try:
        got, _, _ = run_block(sol, dt, l, x, prm, r)
    finally:
        sol.sol_debug_set_conv_tile(0)
    assert rel_err(got, want) <= TOL[dt]


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("cp,cm,stride,cout,hw", [(64, 64, 1, 72, (9, 7)), (192, 64, 2, 136, (13, 9)), (64, 320, 2, 64, (4, 4))])
def test_direct_projection_pair(sol, tile, cp, cm, stride, cout, hw):  # noqa: F811
    """The last 1x1 convolution of a bottleneck and the projection shortcut it adds in one launch of this kernel: reductions of
    unequal length meet inside a wave's run of stages; the shortcut is not rounded on the way (within one more rounding)."""
    c = wl.conv
    layers = [c(cp, 3), c(cm, 1, p=0, s=stride, src=0), c(cout, 1, s=stride, p=0, act="none", src=0), c(cout, 1, p=0, src=1, res=2), c(16, 1, p=0)]
    rng = np.random.default_rng([tile, cp, cm])
    x = wl.to_bf16_grid(rng.standard_normal((3, 3) + hw))
    prm = wl.make_params(layers, 3, 5 + cout, bf16=True, bias_std=0.3)
    outs, _ = orc.network_forward(layers, prm, x, bf16=True, return_all=True)
    net = sol.Network(layers, x.shape, sol.BF16)
    net.set_params(prm)
    xd = sol.to_device_nhwc(x, sol.BF16)
    net.forward(xd)
    net.layer_output(3).zero_()
    sol.sol_debug_set_conv_tile(tile)
    try:
        net.run_layer(3, xd)
    finally:
        sol.sol_debug_set_conv_tile(0)
    torch.cuda.synchronize()
    assert net.fused_into(2) == 3
    assert rel_err(sol.to_host_nchw(net.layer_output(3)).reshape(outs[3].shape), outs[3]) <= 2 * TOL["bf16"]


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(1, 128, 4, 4, 512, 3, 1, 1, True, None), (2, 64, 9, 7, 1024, 1, 1, 0, True, None), (1, 192, 6, 5, 256, 3, 2, 1, False, None),
                                  (1, 64, 2, 3, 264, 3, 1, 3, True, None)])
def test_direct_channel_slices(sol, dt, case, tile):  # noqa: F811
    """Weights larger than the input: an XCD takes a set of channel tiles (tile counts that 8 divides, and one that it does not);
    and windows that lie wholly in a padding as wide as the filter."""
    N, C, H, W, K, k, s, p, res, pool = case
    rng = np.random.default_rng([tile, N, C, H, K, k, s, 7])
    l, x, prm, r = make_block(sol, rng, dt, N, C, H, W, K, k, s, p, res=res, pool=None)
    want = orc.fused_conv(x, prm, l, r, bf16=(dt == "bf16"))[0]
    sol.sol_debug_set_conv_tile(tile)
    try:
        got, _, _ = run_block(sol, dt, l, x, prm, r)
    finally:
        sol.sol_debug_set_conv_tile(0)
    assert rel_err(got, want) <= TOL[dt]
