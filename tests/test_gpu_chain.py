"""fp32 training forward on few pixels (`conv_chain_kernel`): every convolution output bit for bit that of the ring kernel's 64x64 tile,
whose order of summation it repeats."""
import pytest
import torch

from paper_2003_10688_amd import sol
from paper_2003_10688_amd import workloads as wl

pytestmark = pytest.mark.gpu
RING_64x64 = 24


# channels in, layers, batch, image: more than one 64-pixel tile (so that walks start at different chunks), remainders of pixels and of
# channels (odd ones too), strides, 5x5 and 1x1 filters, one chunk per tap, few and many stages, a bias and a residual without BN
@pytest.mark.parametrize("cin,spec,n,hw", [
    (32, [dict(cout=64, k=3), dict(cout=96, k=3, s=2), dict(cout=128, k=1, p=0)], 3, 13),
    (64, [dict(cout=128, k=3), dict(cout=33, k=3), ], 2, 17),
    (64, [dict(cout=128, k=1, s=2, p=0), dict(cout=160, k=5)], 5, 9),
    (96, [dict(cout=71, k=3, bn=False)], 1, 5),
    (128, [dict(cout=128, k=3, bn=False), dict(cout=128, k=3, bn=False, res=0)], 7, 6),
    (512, [dict(cout=512, k=3), dict(cout=512, k=3)], 9, 4),
    (32, [dict(cout=32, k=3)], 1, 1),
    (32, [dict(cout=64, k=3), dict(cout=64, k=3)], 4, 43),      # 1852 blocks: the four-stage ring
])
def test_same_bits_as_the_ring_kernel(cin, spec, n, hw):
    layers = [wl.conv(**s) for s in spec] + [wl.gap(), wl.linear(5)]
    net = sol.Network(layers, (n, cin, hw, hw), sol.F32, flags=sol.NET_TRAINING)
    net.set_params(wl.make_params(layers, cin, 11, False, 0.1))
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(n)
    x = torch.randn((n, hw, hw, cin), generator=gen, device="cuda:0")
    got = {}
    for tile in (0, RING_64x64):
        net.set_tiles({i: tile for i in range(len(spec))})
        y = net.forward(x).clone()
        got[tile] = [y] + [(net.layer_preact(i) if l["bn"] else net.layer_output(i)).clone() for i, l in enumerate(layers) if l["kind"] == "conv"]
    for a, b in zip(got[0], got[RING_64x64]):
        assert torch.equal(a, b)


@pytest.mark.parametrize("cin,spec,n,hw,kernel", [
    (32, dict(cout=64, k=3), 3, 13, "chain"), (64, dict(cout=96, k=3, s=2), 3, 13, "chain"), (96, dict(cout=128, k=1, p=0), 3, 7, "chain"),
    (128, dict(cout=33, k=3), 2, 17, "chain"), (64, dict(cout=160, k=5), 5, 5, "chain"), (512, dict(cout=512, k=3), 9, 4, "chain"),
    (64, dict(cout=64, k=3), 4, 43, "chain"), (64, dict(cout=64, k=3), 5, 43, ""),        # 1852 and 2312 blocks of 16 x 16
    (48, dict(cout=64, k=3), 3, 13, ""), (64, dict(cout=32, k=3), 3, 13, ""), (64, dict(cout=64, k=1, p=0), 3, 13, "")])
def test_which_kernel(cin, spec, n, hw, kernel):
    """The layers that the ring kernel's 64x64 tile with 128-byte stages would run, of up to 2048 blocks; a tile asked for is used."""
    layers = [wl.conv(**spec), wl.gap()]
    net = sol.Network(layers, (n, cin, hw, hw), sol.F32, flags=sol.NET_TRAINING)
    net.set_params(wl.make_params(layers, cin, 11, False, 0.1))
    x = torch.ones((n, hw, hw, cin), device="cuda:0")
    net.forward(x)
    assert sol.sol_debug_conv_kernel() == kernel
    net.set_tiles({0: 5})
    net.forward(x)
    torch.cuda.synchronize()
    assert sol.sol_debug_conv_kernel() == ""
