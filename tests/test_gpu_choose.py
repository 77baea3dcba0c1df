"""The automatic choice of kernel and tile by estimated time: whatever it takes computes what the general path (the implicit-GEMM kernels
alone, tile 99) and the oracle compute, over the forms that it accepts and at the limits of the kernels it picks between."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2003_10688_amd import workloads as wl
from test_gpu_parity import TOL, make_block, rel_err, run_block, sol  # noqa: F401  (sol: the module fixture)

pytestmark = pytest.mark.gpu

CASES = [
    # N, C, H, W, K, k, s, p, res, pool, and the tiles they run on, fp32 and bf16 (tests/test_choose_host.py sees to it that they do)
    (2, 64, 31, 31, 128, 3, 1, 1, True, None, 83, 83), (2, 64, 31, 32, 128, 3, 1, 1, True, None, 83, 83),       # small tiles, odd and even rows
    (1, 64, 17, 62, 64, 3, 1, 1, False, None, 82, 82), (1, 64, 17, 63, 64, 3, 1, 1, False, None, 82, 82),
    (3, 128, 20, 62, 64, 3, 1, 1, True, None, 83, 83), (33, 64, 8, 8, 1000, 3, 2, 1, False, None, 83, 85),
    # halo tiles: the widest image of each, and one column more
    (53, 64, 20, 31, 96, 3, 1, 1, False, None, 83, 41), (53, 64, 20, 32, 96, 3, 1, 1, False, None, 83, 45),
    (61, 128, 13, 31, 16, 3, 1, 1, False, None, 81, 48), (61, 128, 13, 32, 16, 3, 1, 1, False, None, 81, 81),
    (14, 64, 31, 31, 40, 3, 1, 1, False, None, 85, 49), (14, 64, 31, 32, 40, 3, 1, 1, False, None, 85, 26),
    (50, 64, 7, 62, 16, 3, 1, 1, False, None, 81, 45), (50, 64, 7, 63, 16, 3, 1, 1, False, None, 81, 83),       # one chunk of channels
    (29, 128, 16, 62, 16, 3, 1, 1, False, None, 81, 50), (29, 128, 16, 63, 16, 3, 1, 1, False, None, 81, 83),   # two
    (29, 128, 16, 62, 16, 3, 1, 1, True, None, 81, 50), (40, 256, 14, 14, 256, 3, 1, 1, False, None, 85, 48),
    (9, 32, 24, 23, 32, 3, 1, 1, False, None, 83, 15), (9, 32, 24, 24, 32, 3, 1, 1, False, "max", 83, 15),      # rows of 64 bytes, few filters
    (5, 96, 19, 19, 40, 3, 2, 1, False, None, 81, 15),                                                          # half a chunk over, ragged filters
    (50, 64, 33, 33, 16, 1, 1, 0, True, None, 6, 6), (20, 32, 63, 63, 16, 1, 1, 0, False, None, 6, 14),         # many pixels, few filters
    (13, 192, 47, 47, 16, 1, 1, 0, True, None, 6, 24), (13, 128, 35, 35, 33, 1, 2, 0, False, None, 81, 26),
    (20, 128, 28, 28, 512, 1, 1, 0, True, None, 18, 21), (33, 256, 15, 15, 1000, 1, 1, 0, False, None, 18, 21),  # channels that no tile divides
    (8, 128, 41, 41, 1000, 1, 2, 0, False, None, 18, 23), (33, 32, 64, 64, 96, 1, 2, 0, False, None, 6, 18),
    (16, 512, 14, 14, 512, 3, 2, 1, False, None, 83, 84), (30, 128, 30, 30, 128, 3, 1, 1, False, "avg", 18, 61),
    (20, 384, 25, 25, 1000, 1, 2, 0, False, None, 18, 61), (64, 192, 17, 17, 33, 3, 1, 1, False, None, 81, 65),
    (33, 32, 39, 39, 1000, 1, 2, 0, False, None, 18, 66), (64, 96, 28, 28, 96, 1, 1, 0, False, None, 6, 67),
    (12, 64, 26, 26, 33, 1, 2, 0, False, None, 82, 15),                                                         # not a multiple of 4
    (3, 32, 61, 61, 33, 1, 2, 0, False, None, 33, 15), (5, 96, 56, 56, 32, 1, 1, 0, False, None, 24, 15),
    (20, 32, 25, 25, 33, 1, 2, 0, False, None, 15, 15), (64, 64, 19, 19, 33, 1, 2, 0, True, None, 26, 15),
]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES)
def test_choice_against_general_path(sol, dt, case):  # noqa: F811
    N, C, H, W, K, k, s, p, res, pool = case[:10]
    rng = np.random.default_rng([N, C, H, K, k, s])
    l, x, prm, r = make_block(sol, rng, dt, N, C, H, W, K, k, s, p, res=res, pool=wl.pool_desc(pool, 2, 2, 0) if pool else None)
    got = run_block(sol, dt, l, x, prm, r)[0]
    sol.sol_debug_set_conv_tile(99)
    try:
        general = run_block(sol, dt, l, x, prm, r)[0]
    finally:
        sol.sol_debug_set_conv_tile(0)
    # two sums of the same terms in different orders, both within the tolerance of the exact one
    assert rel_err(got, general) <= 2 * TOL[dt]
    few = np.sort(rng.choice(N, min(N, 2), replace=False))             # the oracle's loops take two images
    want = orc.fused_conv(x[few], prm, l, None if r is None else r[few], bf16=(dt == "bf16"))[0]
    assert rel_err(got[few], want) <= TOL[dt]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("n,c,h,w,k", [(2, 64, 9, 7, 40), (33, 128, 20, 21, 64), (40, 32, 24, 24, 32)])
def test_choice_with_winners(sol, dt, n, c, h, w, k):  # noqa: F811
    """A fused max pool that also stores its winners and the tensor in front of it: the three fit one another exactly."""
    rng = np.random.default_rng([n, c, k])
    l, x, prm, r = make_block(sol, rng, dt, n, c, h, w, k, 3, 1, 1, pool=wl.pool_desc("max", 2, 2, 0))
    y, arg, pre = run_block(sol, dt, l, x, prm, r, want_argmax=True, want_prepool=True)
    p, q = h // 2, w // 2
    assert np.array_equal(y, pre[..., :2 * p, :2 * q].reshape(n, k, p, 2, q, 2).max((3, 5)))
    assert np.array_equal(y, np.take_along_axis(pre.reshape(n, k, -1), arg.reshape(n, k, -1).astype(np.int64), 2).reshape(y.shape))
    assert np.array_equal(arg // w // 2, np.broadcast_to(np.arange(p)[:, None], arg.shape)) and np.array_equal(arg % w // 2, np.broadcast_to(np.arange(q), arg.shape))
    want = orc.fused_conv(x[:1], prm, dict(l, pool=None), None, bf16=(dt == "bf16"))[0]
    covered = np.s_[..., :2 * p, :2 * q]                    # pixels that no window covers are not stored
    assert rel_err(pre[:1][covered], want[covered]) <= TOL[dt]


@pytest.mark.parametrize("c,ldx,k,hw,n,s,res,pool", [(64, 64, 128, 9, 3, 1, False, None), (96, 256, 40, 7, 2, 1, True, None), (32, 96, 128, 12, 5, 1, False, "avg"),
                                                     (256, 256, 33, 11, 9, 2, False, None), (1056, 1088, 128, 7, 2, 1, False, None)])
def test_preact_fp32_small_tiles(sol, c, ldx, k, hw, n, s, res, pool):  # noqa: F811
    """Pre-activated 1x1 convolutions in fp32 on the small-tile kernel (no tile asked for) against 64 bits and the register-staged kernel:
    prefixes of a wider tensor (what lies behind is not looked at), strides, pools, ragged channels."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(c + k)
    x = torch.randn((n, hw, hw, ldx), generator=gen, device="cuda:0")
    x[..., c:] = float("nan")
    w = torch.randn((k, c, 1, 1), generator=gen, device="cuda:0") / c ** 0.5
    ps, ph = torch.rand(c, generator=gen, device="cuda:0") + 0.5, torch.rand(c, generator=gen, device="cuda:0") - 0.5
    cd = sol.ConvDesc(k, c, 1, 1, s, s, 0, 0)
    wp = sol.sol_pack_conv_weights(cd, sol.F32, w)
    ho = (hw - 1) // s + 1
    r = torch.randn((n, ho, ho, k), generator=gen, device="cuda:0") if res else None
    pd = sol.pool_desc(wl.pool_desc(pool, 2, 2, 0)) if pool else None
    run = lambda: sol.sol_conv2d_preact_fused(x, cd, wp, ps, ph, residual=r, channels=c, pool=pd)  # noqa: E731
    y = run()
    assert sol.sol_debug_conv_kernel() == "direct"
    sol.sol_debug_set_conv_tile(5)
    try:
        staged = run()
    finally:
        sol.sol_debug_set_conv_tile(0)
    t = (x[..., :c].double() * ps.double() + ph.double()).relu()[:, ::s, ::s]
    want = t.reshape(-1, c) @ w.double().reshape(k, c).T
    want = want.reshape(n, ho, ho, k) + (r.double() if res else 0)
    if pool:
        h2 = ho // 2 * 2
        want = want[:, :h2, :h2].reshape(n, ho // 2, 2, ho // 2, 2, k).mean((2, 4))
    for got in (y, staged):
        assert rel_err(got.cpu().numpy(), want.cpu().numpy()) <= TOL["f32"]
