"""Workloads the library's speed is judged on: layer lists of the benchmark, run through the public entry points.

Every case is one call (or one training step) as a program that uses the library makes it: a network planned once and run
on inputs that lie on the GPU, or one fused layer on its own.  Sizes are those of the benchmark configurations and of the
tests, plus batches and image sizes that divide nothing.
"""
from __future__ import annotations

import math

import torch

from paper_2003_10688_amd import sol
from paper_2003_10688_amd import workloads as wl

DEVICE = "cuda:0"
NETS = {"cnn5": wl.small_cnn_layers, "resnet18": wl.resnet18_layers, "resnet50": wl.resnet50_layers, "separable": wl.separable_layers,
        "squeezenet": wl.squeezenet_layers, "densenet121": wl.densenet_layers}
CLASSES = 1000
LR, MOMENTUM = 1e-4, 0.9     # fine-tuning: two steps on, two correct implementations still see nearly the same weights


def case(path, net, dtype, batch, hw, tune=False):
    """path: layer = one fused convolution block, infer = forward pass, train = forward + backward + SGD step.
    hw: image height and width (mlp3: number of features).  tune: the plan is auto-tuned, as the benchmark does it."""
    return {"path": path, "net": net, "dtype": dtype, "batch": batch, "hw": hw, "tune": tune}


def listed():
    return [
        # one fused convolution + BN + ReLU + max-pool block on one small image: the smallest call, all latency
        {"name": "block_f32_b1", **case("layer", "block", "f32", 1, 32)},
        # a small CIFAR-sized classifier in full precision: few short launches
        {"name": "cnn5_f32_b64", **case("infer", "cnn5", "f32", 64, 32)},
        # serving one image at a time: latency through some fifty dependent layers
        {"name": "resnet50_bf16_b1", **case("infer", "resnet50", "bf16", 1, 224)},
        # offline inference at the benchmark's batch, auto-tuned like the benchmark
        {"name": "resnet50_bf16_b64", **case("infer", "resnet50", "bf16", 64, 224, tune=True)},
        # whatever images and however many happened to be queued: nothing divides a tile
        {"name": "resnet18_bf16_b13_odd", **case("infer", "resnet18", "bf16", 13, 193)},
        # full precision inference, for users who validate against fp32
        {"name": "resnet50_f32_b8", **case("infer", "resnet50", "f32", 8, 224)},
        # the other convolutional families of the benchmark: depthwise, concatenating, densely connected
        {"name": "separable_bf16_b64", **case("infer", "separable", "bf16", 64, 224)},
        {"name": "squeezenet_bf16_b64", **case("infer", "squeezenet", "bf16", 64, 224)},
        {"name": "densenet121_bf16_b64", **case("infer", "densenet121", "bf16", 64, 224)},
        # linear layers whose weights do not fit any cache
        {"name": "mlp3_bf16_b64", **case("infer", "mlp3", "bf16", 64, 8192)},
        # training at the benchmark's size, and a small full-precision one with odd sizes
        {"name": "train_resnet18_bf16_b32", **case("train", "resnet18", "bf16", 32, 224)},
        {"name": "train_resnet18_f32_b9_odd", **case("train", "resnet18", "f32", 9, 113)},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["block", "cnn5", "mlp3", "train", "train", "net", "net", "net", "net", "net", "net"])
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    if kind == "block":
        return case("layer", "block", dtype, _log_int(rng, 1, 256), _log_int(rng, 16, 64))
    if kind == "cnn5":
        return case("infer", "cnn5", dtype, _log_int(rng, 1, 256), rng.randint(24, 48))
    if kind == "mlp3":       # feature counts are multiples of 8, as the library stores rows of 16 bytes
        return case("infer", "mlp3", dtype, _log_int(rng, 1, 128), 8 * _log_int(rng, 64, 1024 if dtype == "bf16" else 512))
    if kind == "train":      # enough pixels per channel in the last stage for its batch statistics to mean something
        return case("train", "resnet18", dtype, rng.randint(8, 32 if dtype == "bf16" else 12), rng.randint(96, 224 if dtype == "bf16" else 160))
    net = rng.choice(["resnet18", "resnet50", "resnet50", "separable", "squeezenet", "densenet121"])
    return case("infer", net, dtype, _log_int(rng, 1, 64 if dtype == "bf16" else 8), rng.randint(64, 224), tune=rng.random() < 0.2)


def _layers(c):
    if c["net"] == "block":
        return wl.single_block_layers()
    if c["net"] == "mlp3":
        return wl.mlp_layers(c["hw"])
    return NETS[c["net"]]()


def _in_shape(c):
    return (c["batch"], c["hw"], 1, 1) if c["net"] == "mlp3" else (c["batch"], 3, c["hw"], c["hw"])


def _params(layers, cin, gen, bf16):
    """Parameters in framework layout with the distributions of the workload module, drawn on the GPU."""
    def normal(*shape):
        return torch.randn(shape, generator=gen, device=DEVICE)

    def uniform(lo, hi, n):
        return torch.rand(n, generator=gen, device=DEVICE) * (hi - lo) + lo

    def host(t):
        return t.cpu().numpy()

    chans, out = wl.layer_channels(layers, cin), []
    for i, l in enumerate(layers):
        src = l.get("src", -1)
        c = cin if src == -1 and i == 0 else chans[i - 1 if src == -1 else src]
        p = {}
        if l["kind"] in ("conv", "linear"):
            if l["kind"] == "conv":
                shape = (l["cout"], 1 if l["dw"] else c, l["kh"], l["kw"])
            else:
                shape = (l["out"], c)
            w = normal(*shape) * math.sqrt(2.0 / math.prod(shape[1:]))
            p["w"] = host(w.to(torch.bfloat16).float() if bf16 else w)
            p["bias"] = host(0.1 * normal(shape[0]))
        for pre, on, n in (("", l.get("bn"), l.get("cout")), ("pre_", l.get("pre_bn"), c)):
            if on:
                p.update({pre + "gamma": host(uniform(0.5, 1.5, n)), pre + "beta": host(uniform(-0.1, 0.1, n)),
                          pre + "mean": host(0.1 * normal(n)), pre + "var": host(uniform(0.5, 1.5, n)), "eps": 1e-5})
        out.append(p)
    return out


def prepare(c, seed):
    """Inputs and what a program keeps between calls: the packed layer, or the planned network with its parameters."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    layers, shape = _layers(c), _in_shape(c)
    dt = sol.BF16 if c["dtype"] == "bf16" else sol.F32
    params = _params(layers, shape[1], gen, dt == sol.BF16)
    n, ch, h, w = shape
    x = torch.randn((n, h, w, ch), generator=gen, device=DEVICE).to(sol.torch_dtype(dt))
    if c["path"] == "layer":
        l, p = layers[0], params[0]
        cd = sol.ConvDesc(l["cout"], ch, l["kh"], l["kw"], l["sh"], l["sw"], l["ph"], l["pw"])
        scale, shift = sol.sol_fold_bn(l["cout"], *(sol.dev_f32(p[k]) for k in ("gamma", "beta", "mean", "var", "bias")), p["eps"])
        return {"path": "layer", "x": x, "cd": cd, "w": sol.sol_pack_conv_weights(cd, dt, sol.dev_f32(p["w"])), "scale": scale,
                "shift": shift, "pool": sol.pool_desc(l["pool"])}
    net = sol.Network(layers, shape, dt, flags=sol.NET_TRAINING if c["path"] == "train" else 0)
    net.set_params(params)
    if c["tune"]:
        net.autotune(x)
    s = {"path": c["path"], "net": net, "x": x}
    if c["path"] == "train":
        s["labels"] = torch.randint(0, CLASSES, (n,), generator=gen, device=DEVICE, dtype=torch.int32)
        # views of the updated weights, and in fp32 of the weight gradients, inside the parameter buffer (in bf16 the gradients
        # of two correct implementations differ by up to 0.25, see tolerance(): nothing to compare)
        s["trained"] = [net.tensor(i, which) for i, l in enumerate(layers) if l["kind"] in ("conv", "linear")
                        for which in ((sol.NT_W,) if dt == sol.BF16 else (sol.NT_W, sol.NT_GRAD_W))]
    return s


def run(s):
    if s["path"] == "layer":
        return sol.sol_conv2d_fused(s["x"], s["cd"], s["w"], s["scale"], s["shift"], act=sol.ACT_RELU, pool=s["pool"])[0]
    y = s["net"].forward(s["x"])
    if s["path"] == "infer":
        return y
    loss = s["net"].backward(s["x"], s["labels"])
    s["net"].sgd_step(LR, MOMENTUM)
    return [y, loss, *s["trained"]]


def _shapes(layers, shape):
    """(input shape, convolution output extent, output shape) of every layer."""
    size = lambda n, k, s, p: (n + 2 * p - k) // s + 1  # noqa: E731
    got = []
    for i, l in enumerate(layers):
        src = l.get("src", -1)
        x = shape if src == -1 and i == 0 else got[i - 1 if src == -1 else src][2]
        n, c, h, w = x
        conv = (h, w)
        if l["kind"] == "conv":
            c, h, w = l["cout"], size(h, l["kh"], l["sh"], l["ph"]), size(w, l["kw"], l["sw"], l["pw"])
            conv = (h, w)
        if l.get("pool"):
            p = l["pool"]
            h, w = size(h, p["kh"], p["sh"], p["ph"]), size(w, p["kw"], p["sw"], p["pw"])
        elif l["kind"] in ("gap", "linear"):
            c, h, w = l.get("out", c), 1, 1
        elif l["kind"] == "concat":
            c += got[l["res"]][2][1]
        got.append((x, conv, (n, c, h, w)))
    return got


def work(c):
    """Contractions of the pass; the network's input, output and parameters once (activations between the layers and the
    gradients of activations are not counted).  Training: three contractions per layer (two for the first), weights and
    velocities read and written, gradients written."""
    layers, esize = _layers(c), 2 if c["dtype"] == "bf16" else 4
    shapes = _shapes(layers, _in_shape(c))
    flops = weights = vectors = 0
    first = True
    for l, (x, conv, y) in zip(layers, shapes):
        if l["kind"] not in ("conv", "linear"):
            continue
        taps = l.get("kh", 1) * l.get("kw", 1) * (1 if l.get("dw") else x[1])
        f = 2 * x[0] * conv[0] * conv[1] * y[1] * taps
        flops += f * (1 if c["path"] != "train" else 2 if first else 3)
        first = False
        weights += taps * y[1]
        vectors += 2 * y[1]
    nbytes = esize * (math.prod(shapes[0][0]) + math.prod(shapes[-1][2]))
    if c["path"] == "train":
        return {"bytes": nbytes + 4 * 5 * (weights + vectors), "flops": flops}
    return {"bytes": nbytes + esize * weights + 4 * vectors, "flops": flops}


def tolerance(c):
    """Four times what the library's own kernels of different summation orders differ by from one another (three steps of
    training included: logits 0.009 in bf16, gradients 0.006 in fp32).  Gradients differ by far more than sums do: a
    rounding of relative size d puts about 0.4 d of the ReLU decisions on the other side of zero, each of them a whole
    term, so an activation gradient moves by the square root of that per layer."""
    bf16 = c["dtype"] == "bf16"
    if c["path"] == "train":
        return {"rel": 0.03}
    return {"rel": 0.017 if bf16 else 5e-6}
