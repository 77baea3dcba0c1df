"""The parameter update and the packed copies it writes (`update_batch_kernel`): after a step, a network computes, bit for bit, what a
fresh network does whose parameters are set to the updated masters; the update itself against v <- mu v + g, w <- w - lr v."""
import numpy as np
import pytest
import torch

from paper_2003_10688_amd import sol
from paper_2003_10688_amd import workloads as wl

pytestmark = pytest.mark.gpu
KEYS = {"w": sol.NT_W, "gamma": sol.NT_GAMMA, "beta": sol.NT_BETA, "bias": sol.NT_BIAS}

# filters and channels around a block's tile: whole 32 x 32 and 64 x 64 tiles, remainders that are and are not whole 16-byte groups,
# runs that do not start on 16 bytes (odd channels x 9 taps), 49 and 400 taps (a tile of few channels, of one channel)
LISTS = {
    "tiles": [wl.conv(64, 3), wl.conv(96, 3), wl.conv(128, 1, p=0), wl.gap(), wl.linear(64)],
    "remainders": [wl.conv(40, 3), wl.conv(72, 3), wl.conv(100, 1, p=0), wl.gap(), wl.linear(10)],
    "odd": [wl.conv(7, 3), wl.conv(33, 3), wl.conv(65, 1, p=0), wl.gap(), wl.linear(9)],
    "few_tiles": [wl.conv(40, 3), wl.conv(64, 11, p=5), wl.conv(48, 7), wl.conv(24, 1, p=0), wl.gap(), wl.linear(12)],   # cut into smaller ones
    "large_filters": [wl.conv(36, 7), wl.conv(12, 5), wl.conv(35, 20, p=9), wl.gap(), wl.linear(11)],
}


def make(layers, dt, params):
    net = sol.Network(layers, (4, 3, 14, 14), dt, flags=sol.NET_TRAINING)
    net.set_params(params)
    return net


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", list(LISTS))
def test_update_and_packed_copies(name, dtype):
    layers, dt = LISTS[name], sol.F32 if dtype == "f32" else sol.BF16
    rng = np.random.default_rng(7)
    params = wl.make_params(layers, 3, 7, dtype == "bf16")
    x = sol.to_device_nhwc(rng.standard_normal((4, 3, 14, 14)).astype(np.float32), dt)
    labels = torch.tensor([0, 3, 5, 8], dtype=torch.int32, device="cuda:0")
    net = make(layers, dt, params)
    trained = [(i, k) for i, l in enumerate(layers) if l["kind"] in ("conv", "linear")
               for k in (("w", "gamma", "beta") if l["kind"] == "conv" and l["bn"] else ("w", "bias"))]
    vel = {t: 0.0 for t in trained}
    for step in range(2):
        net.forward(x)
        net.backward(x, labels)
        before = {t: net.tensor(t[0], KEYS[t[1]]).double() for t in trained}
        grad = {t: net.tensor(t[0], KEYS[t[1]] + sol.NT_GRAD_W).double() for t in trained}
        net.sgd_step(0.125, 0.5)
        for t in trained:
            vel[t] = 0.5 * vel[t] + grad[t]
            got, want = net.tensor(t[0], KEYS[t[1]]).double(), before[t] - 0.125 * vel[t]
            # one rounding of the velocity (times lr) and one of the weight
            assert ((got - want).abs() <= 2.0 ** -23 * (want.abs() + 0.125 * vel[t].abs() * 2 + before[t].abs())).all(), (t, step)
    new = [dict(p) for p in params]
    for i, k in trained:
        new[i][k] = net.tensor(i, KEYS[k]).cpu().numpy().reshape(np.shape(params[i][k]))
    fresh = make(layers, dt, new)
    outs = []
    for n in (net, fresh):
        y = n.forward(x).clone()
        n.backward(x, labels)
        outs.append([y] + [n.layer_grad(i).clone() for i in range(len(layers))] + [n.tensor(i, KEYS[k] + sol.NT_GRAD_W).clone() for i, k in trained])
    for a, b in zip(*outs):
        assert torch.equal(a, b)
