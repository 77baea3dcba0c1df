"""CPU-only checks of the C ABI: the library loads, exports every symbol the header declares, and its
host-side logic (argument validation, shape inference, buffer planning) behaves -- no kernel runs."""
import ctypes as C
import os
import re

import pytest

from paper_2003_10688_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def sol():
    from paper_2003_10688_amd import sol as s

    if not os.path.exists(s.LIB_PATH):
        from paper_2003_10688_amd import build

        build.build(verbose=False)
    s.lib()
    return s


def test_exports_every_declared_symbol(sol):
    hdr = open(os.path.join(ROOT, "include", "sol.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    names = set(re.findall(r"\b(sol_[a-z0-9_]+)\s*\(", hdr))
    assert {"sol_conv2d_fused", "sol_linear", "sol_pool", "sol_network_forward", "sol_network_create"} <= names
    for n in sorted(names):
        assert hasattr(sol.lib(), n), f"{n} declared in include/sol.h but not exported"
    assert b"gfx950" in sol.lib().sol_version()


def test_out_size_and_packed_bytes(sol):
    assert sol.sol_out_size(224, 7, 2, 3) == 112 and sol.sol_out_size(112, 3, 2, 1) == 56
    assert sol.sol_out_size(5, 2, 2, 0) == 2 and sol.sol_out_size(7, 3, 1, 1) == 7
    assert sol.sol_packed_weight_bytes(sol.ConvDesc(64, 3, 7, 7, 2, 2, 3, 3), sol.BF16) == 64 * 192 * 2   # 147 -> 192
    assert sol.sol_packed_weight_bytes(sol.ConvDesc(64, 3, 7, 7, 2, 2, 3, 3), sol.F32) == 64 * 160 * 4    # 147 -> 160
    assert sol.sol_packed_weight_bytes(sol.ConvDesc(256, 64, 1, 1, 1, 1, 0, 0), sol.BF16) == 256 * 64 * 2


def _status(sol, fn, *args):
    return fn(*args)


def test_validation_rejects_before_launch(sol):
    L = sol.lib()
    xd = sol.TensorDesc(1, 8, 8, 16, sol.F32)
    cd = sol.ConvDesc(8, 16, 3, 3, 1, 1, 1, 1)
    null = C.c_void_p(0)
    fake = C.c_void_p(0x1000)          # never dereferenced: validation fails first
    call = lambda xd_, x, cd_, w, y, pool=None: L.sol_conv2d_fused(  # noqa: E731
        C.byref(xd_), x, C.byref(cd_), w, null, null, null, 0, C.byref(pool) if pool else None, y, null, null, null)
    assert call(xd, null, cd, fake, fake) == 1                                            # NULL x
    assert b"NULL" in L.sol_last_error()
    assert call(xd, fake, sol.ConvDesc(8, 4, 3, 3, 1, 1, 1, 1), fake, fake) == 2           # cin mismatch
    assert call(xd, fake, sol.ConvDesc(8, 16, 3, 3, 0, 1, 1, 1), fake, fake) == 2          # zero stride
    assert call(sol.TensorDesc(1, 8, 8, 16, 7), fake, cd, fake, fake) == 3                 # dtype
    assert call(xd, C.c_void_p(0x1004), cd, fake, fake) == 4                               # alignment
    assert call(xd, fake, cd, fake, fake, sol.PoolDesc(sol.POOL_MAX, 3, 3, 2, 2, 1, 1, 1)) == 6   # unfusable pool
    assert call(sol.TensorDesc(1, 2, 2, 16, 0), fake, sol.ConvDesc(8, 16, 5, 5, 1, 1, 0, 0), fake, fake) == 2  # filter > input
    big = sol.TensorDesc(65536, 512, 512, 16, sol.BF16)                                    # >= 2^31 elements
    assert call(big, fake, cd, fake, fake) == 6
    assert L.sol_pool(C.byref(xd), fake, C.byref(sol.PoolDesc(sol.POOL_MAX, 2, 2, 2, 2, 2, 2, 1)), fake, null, null) == 2
    assert L.sol_linear(4, 0, 3, 0, fake, fake, null, 0, fake, null) == 2


def _create(sol, layers, shape, dt, flags=0):
    h = C.c_void_p(0)
    n, c, hh, ww = shape
    st = sol.lib().sol_network_create(sol.make_layer_array(layers), len(layers), C.byref(sol.TensorDesc(n, hh, ww, c, dt)),
                                      flags, C.byref(h))
    return st, h


def test_planner_shapes_and_buffers(sol):
    L = sol.lib()
    wk = wl.config(3)
    st, h = _create(sol, wk.layers, wk.in_shape, sol.BF16)
    assert st == 0
    d = sol.TensorDesc()
    assert L.sol_network_output_desc(h, -1, C.byref(d)) == 0 and (d.n, d.h, d.w, d.c) == (64, 1, 1, 1000)
    assert L.sol_network_output_desc(h, 0, C.byref(d)) == 0 and (d.n, d.h, d.w, d.c) == (64, 112, 112, 64)
    assert L.sol_network_output_desc(h, 1, C.byref(d)) == 0 and (d.n, d.h, d.w, d.c) == (64, 56, 56, 64)
    assert L.sol_network_output_desc(h, len(wk.layers) - 3, C.byref(d)) == 0 and (d.n, d.h, d.w, d.c) == (64, 7, 7, 2048)
    assert L.sol_network_num_layers(h) == len(wk.layers)
    ws = L.sol_network_workspace_bytes(h)
    biggest = 64 * 56 * 56 * 256 * 2                      # largest live activation
    assert 2 * biggest <= ws <= 5 * biggest               # buffers are reused, not one per layer
    pb = L.sol_network_param_bytes(h)
    assert 25.5e6 * 2 <= pb <= 25.5e6 * 2 * 1.1           # ~25.5 M bf16 weights plus scale/shift
    st2, h2 = _create(sol, wk.layers, wk.in_shape, sol.BF16, sol.NET_KEEP_ACTIVATIONS)
    assert st2 == 0 and L.sol_network_workspace_bytes(h2) > 4 * ws
    L.sol_network_destroy(h)
    L.sol_network_destroy(h2)


def test_planner_rejects_bad_graphs(sol):
    bad_res = [wl.conv(8, 3), wl.conv(16, 3, res=0)]                       # residual channel mismatch
    assert _create(sol, bad_res, (1, 3, 8, 8), sol.F32)[0] == 2
    fwd_ref = [wl.conv(8, 3, src=1), wl.conv(8, 3)]                        # src must be an earlier layer
    assert _create(sol, fwd_ref, (1, 3, 8, 8), sol.F32)[0] == 2
    lin = [wl.conv(8, 3), wl.linear(4)]                                    # linear needs [n,1,1,c]
    assert _create(sol, lin, (1, 3, 8, 8), sol.F32)[0] == 6
    assert _create(sol, [wl.conv(8, 9, p=0)], (1, 3, 4, 4), sol.F32)[0] == 2   # filter larger than input
    st, h = _create(sol, wl.small_cnn_layers(), (64, 3, 32, 32), sol.F32)
    assert st == 0
    # forward without bound parameters / workspace is refused, nothing is launched
    fake = C.c_void_p(0x1000)
    assert sol.lib().sol_network_forward(h, fake, fake, fake, C.c_size_t(1 << 30), None) == 5
    sol.lib().sol_network_destroy(h)


def test_plan_tile_api_validates(sol):
    """Per-layer kernel/tile ids (set by the auto-tune, restorable by the caller) are range-checked on the host."""
    L = sol.lib()
    st, h = _create(sol, wl.small_cnn_layers(), (8, 3, 32, 32), sol.F32)
    assert st == 0
    t = C.c_int(-1)
    assert L.sol_network_layer_tile(h, 0, C.byref(t)) == 0 and t.value == 0          # heuristic until tuned
    assert L.sol_network_set_layer_tile(h, 1, 21) == 0
    assert L.sol_network_layer_tile(h, 1, C.byref(t)) == 0 and t.value == 21
    assert L.sol_network_set_layer_tile(h, 99, 21) == 2 and L.sol_network_set_layer_tile(h, 0, 1000) == 2
    assert L.sol_network_layer_tile(None, 0, C.byref(t)) == 1
    fake = C.c_void_p(0x1000)
    assert L.sol_network_autotune(None, fake, fake, fake, C.c_size_t(0), 3, None) == 1
    assert L.sol_network_autotune(h, fake, fake, fake, C.c_size_t(1 << 30), 0, None) == 2     # reps out of range
    L.sol_network_destroy(h)


def test_plan_fuses_stem_and_pool_only_when_it_may(sol):
    """The depth-first stem + max-pool pair is a plan-time decision taken on the host: bf16 7x7/2 stem with 64
    filters and ReLU whose only consumer is a 3x3/2 pad-1 max-pool layer, and no kept activations."""
    L = sol.lib()
    t = C.c_int(-1)

    def fused(layers, shape, dt, flags=0):
        st, h = _create(sol, layers, shape, dt, flags)
        assert st == 0
        r = []
        for i in range(len(layers)):
            assert L.sol_network_layer_fused_into(h, i, C.byref(t)) == 0
            r.append(t.value)
        assert L.sol_network_layer_fused_into(h, len(layers), C.byref(t)) == 2
        ws = L.sol_network_workspace_bytes(h)
        L.sol_network_destroy(h)
        return r, ws

    wk = wl.config(3)
    n = len(wk.layers)
    r, ws = fused(wk.layers, wk.in_shape, sol.BF16)
    # the pool runs inside the stem's launch; the projection shortcut of every stage's first bottleneck (a 1x1
    # convolution without activation, read only as a residual) runs inside the launch of the 1x1 convolution that adds it
    want = list(range(n))
    want[1] = 0
    shortcuts = [l["res"] for l in wk.layers if l["kind"] == "conv" and l.get("res", -1) >= 0 and wk.layers[l["res"]]["act"] == "none"]
    assert len(shortcuts) == 4 and shortcuts[0] == 4
    for j in shortcuts:
        want[j] = j + 1
    # the identity bottlenecks of stages 0 and 1 (mid widths 64 / 128, enough pixels at batch 64) run as one
    # depth-first launch: their first two convolutions are produced by the launch of the third
    ends = [i for i, l in enumerate(wk.layers) if l["kind"] == "conv" and l.get("res", -1) >= 0 and wk.layers[l["res"]]["act"] != "none"
            and l["cout"] in (256, 512)]
    assert len(ends) == 5
    for i in ends:
        want[i - 2] = want[i - 1] = i
    # the last 1x1 convolution of an identity bottleneck of stage 2 (256 -> 1024 channels at 14x14) and the first 1x1
    # convolution of the next bottleneck (1024 -> 256, and 1024 -> 512 into the last stage) run as one expand-reduce launch:
    # five pairs
    starts = [i for i, l in enumerate(wk.layers[:-1]) if l["kind"] == "conv" and l["cout"] == 1024 and l.get("res", -1) >= 0
              and wk.layers[l["res"]]["act"] != "none" and wk.layers[i + 1]["kind"] == "conv" and wk.layers[i + 1]["cout"] in (256, 512)
              and wk.layers[i + 1]["kh"] == 1]
    assert len(starts) == 5
    for i in starts:
        want[i + 1] = i
    assert r == want
    st_, h_ = _create(sol, wk.layers, wk.in_shape, sol.BF16, 0)
    bs = C.c_int(-2)
    assert [L.sol_network_layer_xr(h_, i, C.byref(bs)) or bs.value for i in starts] == [1] * 5
    assert L.sol_network_layer_xr(h_, 0, C.byref(bs)) == 0 and bs.value == -1
    assert L.sol_network_set_layer_xr(h_, starts[0], 0) == 0 and L.sol_network_layer_xr(h_, starts[0], C.byref(bs)) == 0 and bs.value == 0
    assert L.sol_network_layer_fused_into(h_, starts[0] + 1, C.byref(t)) == 0 and t.value == starts[0] + 1
    assert L.sol_network_set_layer_xr(h_, 0, 1) == 6 and L.sol_network_set_layer_xr(h_, 0, 0) == 0
    assert L.sol_network_set_layer_xr(h_, starts[0], 1) == 0
    assert [L.sol_network_layer_block(h_, i, C.byref(bs)) or bs.value for i in ends] == [1] * 5
    assert L.sol_network_layer_block(h_, 0, C.byref(bs)) == 0 and bs.value == -1
    assert L.sol_network_set_layer_block(h_, ends[0], 0) == 0 and L.sol_network_layer_block(h_, ends[0], C.byref(bs)) == 0 and bs.value == 0
    assert L.sol_network_layer_fused_into(h_, ends[0] - 1, C.byref(t)) == 0 and t.value == ends[0] - 1
    assert L.sol_network_set_layer_block(h_, 0, 1) == 6 and L.sol_network_set_layer_block(h_, 0, 0) == 0
    L.sol_network_destroy(h_)
    r_keep, ws_keep = fused(wk.layers, wk.in_shape, sol.BF16, sol.NET_KEEP_ACTIVATIONS)
    assert r_keep == list(range(n)) and ws_keep > ws
    assert fused(wk.layers, wk.in_shape, sol.BF16, sol.NET_TRAINING)[0] == list(range(n))
    assert fused(wk.layers, wk.in_shape, sol.F32)[0] == [0, 0] + list(range(2, n))         # fp32: the stem pair alone
    stem, pool = wl.conv(64, 7, 2, 3), wl.pool("max", 3, 2, 1)
    tail = [wl.conv(8, 1)]
    assert fused([stem, pool] + tail, (2, 3, 40, 40), sol.BF16)[0] == [0, 0, 2]
    assert fused([stem, pool], (2, 3, 40, 40), sol.BF16)[0] == [0, 0]                      # the pool is the network output
    assert fused([stem, wl.pool("max", 2, 2, 0)] + tail, (2, 3, 40, 40), sol.BF16)[0] == [0, 1, 2]
    assert fused([stem, wl.pool("avg", 3, 2, 1)] + tail, (2, 3, 40, 40), sol.BF16)[0] == [0, 1, 2]
    assert fused([wl.conv(32, 7, 2, 3), pool] + tail, (2, 3, 40, 40), sol.BF16)[0] == [0, 1, 2]
    assert fused([wl.conv(64, 7, 2, 3, act="none"), pool] + tail, (2, 3, 40, 40), sol.BF16)[0] == [0, 1, 2]
    # a second consumer of the stem's output keeps it alive: no fusion
    assert fused([stem, pool, wl.conv(8, 1, src=0)], (2, 3, 40, 40), sol.BF16)[0] == [0, 1, 2]
    assert L.sol_network_layer_fused_into(None, 0, C.byref(t)) == 1


@pytest.mark.parametrize("k", [3, 7])
@pytest.mark.parametrize("pad", [0, 1])
def test_plan_leaves_a_pre_activated_stem_alone(sol, k, pad):
    """The stem + pool kernel has no BN + ReLU on its input side: such a convolution and its pool stay two launches, as two layers and as one."""
    L = sol.lib()
    t, pool = C.c_int(-1), wl.pool("max", 3, 2, pad)
    for dt in (sol.F32, sol.BF16):
        for pre, want in ((False, 0), (True, 1)):
            st, h = _create(sol, [wl.conv(64, k, 2, k // 2, pre_bn=pre), pool, wl.conv(8, 1)], (2, 3, 40, 40), dt)
            assert st == 0 and L.sol_network_layer_fused_into(h, 1, C.byref(t)) == 0 and t.value == want
            L.sol_network_destroy(h)
        ws = []
        for pre in (False, True):                          # the pool inside the layer: apart from it, the convolution's output needs a buffer
            st, h = _create(sol, [wl.conv(64, k, 2, k // 2, pre_bn=pre, pool=wl.pool_desc("max", 3, 2, pad)), wl.conv(8, 1)], (2, 3, 40, 40), dt)
            assert st == 0
            ws.append(L.sol_network_workspace_bytes(h))
            L.sol_network_destroy(h)
        assert ws[1] >= ws[0] + 2 * 64 * 20 * 20 * (2 if dt == sol.BF16 else 4)


# tiles that add up a reduction alike (tests/test_gpu_grad_order.py): split over waves, staged in registers, ring kernel by pixels x bytes
SUM_ORDERS = {"split": (81, 82, 83, 84, 85), "staged": tuple(range(1, 9)), "64x64": (15, 18, 33), "64x128": (24, 26), "128x64": (11, 12, 14, 16, 25, 32),
              "128x128": (21, 22, 23)}
# (batch, channels of the gradient, of the layer's input, filter): the order, and from which square image on it is
GRADIENT_ORDERS = {
    (1, 64, 64, 3): {2: "split", 111: "64x128"}, (1, 128, 64, 1): {2: "split", 74: "64x128", 111: "64x64"},
    (1, 256, 256, 3): {2: "split", 75: "64x128", 111: "128x128"}, (1, 512, 512, 3): {2: "split", 55: "64x128", 78: "128x128"},
    (1, 64, 256, 1): {2: "split", 23: "64x128", 55: "64x64", 78: "64x128", 111: "128x128"},
    (9, 64, 64, 3): {2: "split", 37: "64x128"}, (9, 128, 64, 1): {2: "split", 25: "64x128", 37: "64x64"},
    (9, 128, 128, 3): {2: "split", 32: "64x128", 53: "128x128"}, (9, 256, 256, 3): {2: "split", 25: "64x128", 37: "128x128", 86: "128x64"},
    (9, 512, 512, 3): {2: "split", 19: "64x128", 26: "128x128", 61: "128x64"}, (9, 512, 256, 1): {2: "split", 19: "64x128", 37: "128x128", 86: "128x64"},
    (9, 64, 256, 1): {2: "split", 8: "64x128", 19: "64x64", 26: "64x128", 37: "128x128", 86: "128x64"},
    (9, 64, 32, 3): {2: "split", 37: "staged"}, (9, 48, 64, 3): {2: "64x64"},
    (32, 128, 64, 1): {2: "split", 13: "64x128", 20: "64x64"}, (32, 128, 128, 3): {2: "split", 17: "64x128", 28: "128x128", 64: "128x64"},
    (32, 64, 256, 1): {2: "split", 5: "64x128", 10: "64x64", 14: "64x128", 20: "128x128", 46: "128x64"},
}


def test_order_of_fp32_data_gradients_is_pinned(sol):
    """The order in which an fp32 data gradient adds up decides its last bits, and through them where a training run ends: it must not
    move when the estimates of times do."""
    for (n, c, k, f), pins in GRADIENT_ORDERS.items():
        want = None
        for hw in range(2, 113):
            want = pins.get(hw, want)
            t = sol.sol_debug_choose_conv_tile(sol.TensorDesc(n, hw, hw, c, sol.F32), sol.ConvDesc(k, c, f, f, 1, 1, f // 2, f // 2), gradient=True)
            assert t in SUM_ORDERS[want], (n, c, k, f, hw, t)
    for hw in range(2, 80):                                 # bf16: the fastest estimate
        xd, cd = sol.TensorDesc(9, hw, hw, 128, sol.BF16), sol.ConvDesc(64, 128, 3, 3, 1, 1, 1, 1)
        assert sol.sol_debug_choose_conv_tile(xd, cd, gradient=True) == sol.sol_debug_choose_conv_tile(xd, cd)


def test_concat_planning_and_validation(sol):
    """Channel concatenation layers: shapes, refusals, and which producers the plan lets write in place."""
    L = sol.lib()
    c, cat = wl.conv, wl.concat
    fire = wl.fire_layers(1, 0, 8, 16)
    layers = [c(16, 3)] + fire + [c(8, 1, p=0)]
    st, h = _create(sol, layers, (2, 3, 12, 12), sol.BF16)
    assert st == 0
    d = sol.TensorDesc()
    assert L.sol_network_output_desc(h, 4, C.byref(d)) == 0 and (d.n, d.h, d.w, d.c) == (2, 12, 12, 32)
    t = C.c_int(-1)
    assert L.sol_network_concat_in_place(h, 4, C.byref(t)) == 0 and t.value == 2
    assert L.sol_network_concat_in_place(h, 3, C.byref(t)) == 2            # not a concatenation
    assert L.sol_network_concat_in_place(h, 99, C.byref(t)) == 2 and L.sol_network_concat_in_place(None, 4, C.byref(t)) == 1
    ws = L.sol_network_workspace_bytes(h)
    L.sol_network_destroy(h)
    st, h = _create(sol, layers, (2, 3, 12, 12), sol.BF16, sol.NET_KEEP_ACTIVATIONS)
    assert st == 0 and L.sol_network_concat_in_place(h, 4, C.byref(t)) == 0 and t.value == 0
    assert L.sol_network_workspace_bytes(h) > ws                         # the expand outputs exist twice when everything is kept
    L.sol_network_destroy(h)
    assert _create(sol, layers, (2, 3, 12, 12), sol.BF16, sol.NET_TRAINING)[0] == 6                     # inference only
    assert _create(sol, [c(8, 3), cat(0, 0)], (1, 3, 8, 8), sol.F32)[0] == 2                            # one layer twice
    assert _create(sol, [c(8, 3), c(8, 3, s=2, src=0), cat(0, 1)], (1, 3, 8, 8), sol.F32)[0] == 2       # extents differ
    assert _create(sol, [c(8, 3), cat(0, 2), c(8, 3)], (1, 3, 8, 8), sol.F32)[0] == 2                   # names a later layer
    assert _create(sol, [cat(-1, 0)], (1, 3, 8, 8), sol.F32)[0] == 2                                    # nothing to join


def test_depthwise_planning_and_validation(sol):
    """Depthwise layers: shape inference keeps the channel count, parameters are [taps][c] + scale/shift, bad
    descriptors are refused on the host."""
    L = sol.lib()
    assert L.sol_packed_dw_weight_bytes(32, 3, 3, sol.BF16) == 32 * 9 * 2
    assert L.sol_packed_dw_weight_bytes(8, 5, 3, sol.F32) == 8 * 15 * 4 and L.sol_packed_dw_weight_bytes(0, 3, 3, sol.F32) == 0
    assert L.sol_packed_dw_weight_bytes(3, 3, 3, sol.BF16) == 64                     # 54 bytes, rounded up to 16
    wk = wl.config(6)
    st, h = _create(sol, wk.layers, wk.in_shape, sol.BF16)
    assert st == 0
    d = sol.TensorDesc()
    assert L.sol_network_output_desc(h, 1, C.byref(d)) == 0 and (d.n, d.h, d.w, d.c) == (64, 112, 112, 32)    # depthwise s1
    assert L.sol_network_output_desc(h, 3, C.byref(d)) == 0 and (d.n, d.h, d.w, d.c) == (64, 56, 56, 64)      # depthwise s2
    assert L.sol_network_output_desc(h, -1, C.byref(d)) == 0 and (d.n, d.h, d.w, d.c) == (64, 1, 1, 1000)
    # 4.2 M parameters: pointwise + classifier weights dominate, 9 values per channel for the depthwise layers
    assert 4.2e6 * 2 <= L.sol_network_param_bytes(h) <= 4.2e6 * 2 * 1.15
    L.sol_network_destroy(h)
    assert _create(sol, [wl.conv(24, 3, dw=True)], (2, 16, 8, 8), sol.BF16)[0] == 2                            # channel count must be kept
    assert _create(sol, [wl.conv(16, 3, dw=True, pool=wl.pool_desc("max", 2, 2, 0))], (2, 16, 8, 8), sol.BF16)[0] == 6
    assert _create(sol, [wl.conv(16, 3, dw=True), wl.gap(), wl.linear(4)], (2, 16, 8, 8), sol.BF16, sol.NET_TRAINING)[0] == 6
    xd = sol.TensorDesc(1, 8, 8, 16, sol.BF16)
    fake, null = C.c_void_p(0x1000), C.c_void_p(0)
    call = lambda cd, x=fake, w=fake, y=fake: L.sol_dwconv2d_fused(C.byref(xd), x, C.byref(cd), w, null, null, null, 0, y, null)  # noqa: E731
    assert call(sol.ConvDesc(32, 16, 3, 3, 1, 1, 1, 1)) == 2                          # cout != channels
    assert call(sol.ConvDesc(16, 16, 3, 3, 1, 1, 1, 1), w=null) == 1                  # NULL weights
    assert call(sol.ConvDesc(16, 16, 3, 3, 1, 1, 1, 1), x=C.c_void_p(0x1008)) == 4    # misaligned x
    assert call(sol.ConvDesc(16, 16, 11, 11, 1, 1, 0, 0)) == 2                        # filter larger than the input


def test_no_kernel_spills_registers():
    """The compiler's per-kernel resource report of the last build (written by paper_2003_10688_amd/build.py): no kernel
    of the library may use scratch memory (spilled registers travel through HBM: the stage-3 3x3 kernels once wrote
    5.7x their output that way), and none may exceed the 160 KB of LDS of a compute unit."""
    import json

    from paper_2003_10688_amd import build as b

    path = b.RESOURCES
    if not os.path.exists(path):
        pytest.skip("no build report (run __graft_entry__.build())")
    with open(path) as f:
        res = json.load(f)
    assert len(res) > 100
    spills = {k: v["scratch_bytes_per_lane"] for k, v in res.items() if v.get("scratch_bytes_per_lane", 0) != 0}
    assert not spills, spills
    assert all(v.get("lds_bytes", 0) <= 160 * 1024 for v in res.values())


@pytest.mark.parametrize("dt,late", [("f32", "pointwise"), ("bf16", "pointwise"), ("bf16", "dense")])
def test_dense_chain_buffer_outlives_its_last_reader(sol, dt, late):
    """The joins of a dense block share one buffer.  A layer that reads an inner join after everything has read the last one
    (on its own, or inside the launch of the 3x3 convolution behind it) still finds it: no other output takes its place."""
    L, c = sol.lib(), wl.conv
    layers = [c(64, 1, p=0), c(128, 1, p=0, src=0, pre_bn=True), c(32, 3, bn=False, act="none"), wl.concat(0, 2),
              c(128, 1, p=0, src=3, pre_bn=True), c(32, 3, bn=False, act="none"), wl.concat(3, 5)]
    if late == "dense":
        layers += [c(128, 1, p=0, src=3, pre_bn=True), c(256, 1, p=0, src=6), c(64, 1, p=0), c(128, 1, p=0, src=9), c(32, 3, src=7), c(8, 1, p=0, src=10)]
    else:
        layers += [c(256, 1, p=0, src=6), c(64, 1, p=0), c(128, 1, p=0, src=8), c(64, 1, p=0, src=3), c(8, 1, p=0, src=9)]
    d = sol.BF16 if dt == "bf16" else sol.F32
    st, h = _create(sol, layers, (2, 64, 14, 14), d)
    assert st == 0
    last = max(i for i in range(len(layers) - 1) if layers[i].get("src", -1) == (7 if late == "dense" else 3))   # launches the late read
    es, got = 2 if dt == "bf16" else 4, {}
    for i in range(6, last):
        p, od, into = C.c_void_p(), sol.TensorDesc(), C.c_int()
        assert L.sol_network_layer_fused_into(h, i, C.byref(into)) == 0
        if into.value != i:
            continue
        assert L.sol_network_layer_output(h, i, C.c_void_p(1 << 40), C.byref(p)) == 0
        assert L.sol_network_output_desc(h, i, C.byref(od)) == 0
        got[i] = (p.value, p.value + od.n * od.h * od.w * od.c * es)
    for i in range(7, last):
        if i in got:
            assert got[i][0] >= got[6][1] or got[i][1] <= got[6][0], f"layer {i} is written over the block's buffer"
    L.sol_network_destroy(h)


def _dense_net(sol, shape, c=64):
    layers = [wl.conv(c, 1, p=0), wl.conv(128, 1, p=0, src=0, pre_bn=True), wl.conv(32, 3, bn=False, act="none"), wl.concat(0, 2),
              wl.conv(8, 1, p=0, bn=False, act="none")]
    st, h = _create(sol, layers, shape, sol.BF16)
    assert st == 0
    return h


@pytest.mark.parametrize("shape,c,fused", [((64, 64, 56, 56), 64, 1), ((64, 64, 104, 104), 64, 1), ((64, 64, 105, 105), 64, 0), ((64, 64, 144, 144), 96, 1),
                                           ((16, 64, 149, 149), 96, 0), ((8, 64, 183, 183), 64, 0), ((1, 64, 144, 144), 64, 1), ((1, 64, 176, 176), 64, 0)])
def test_dense_layer_one_launch_or_two(sol, shape, c, fused):
    """Wide images, whose tiles are mostly halo, keep the two launches; the choice can be set both ways, and only a pass that
    stores the 1x1 convolution's output needs the buffer for it."""
    L, h, v = sol.lib(), _dense_net(sol, shape, c), C.c_int()

    def state():
        assert L.sol_network_layer_dense(h, 2, C.byref(v)) == 0
        d = v.value
        assert L.sol_network_layer_fused_into(h, 1, C.byref(v)) == 0 and v.value == (2 if d else 1)
        return d

    assert state() == fused
    assert L.sol_network_layer_dense(h, 1, C.byref(v)) == 0 and v.value == -1
    assert L.sol_network_set_layer_dense(h, 1, 1) == 6
    n, _, hh, ww = shape
    buf, need = n * hh * ww * 128 * 2, L.sol_network_workspace_bytes(h)
    fake = C.c_void_p(0x1000)
    for f in (0, 1):
        assert L.sol_network_set_layer_dense(h, 2, f) == 0 and state() == f
        # parameters are not set: a workspace that is large enough is refused for that, a smaller one for its size
        for size, what in ((need, "parameters"), (need - buf, "parameters" if f else "workspace"), (need - buf - (buf + 255) // 256 * 256, "workspace")):
            assert L.sol_network_forward(h, fake, fake, fake, C.c_size_t(size), None) == 5
            assert what in L.sol_last_error().decode(), (f, size)
    L.sol_network_destroy(h)


def test_dense_layer_tile_runs_two_launches(sol):
    """A tile set for either convolution of a dense layer is used: the pair runs one by one until both are automatic again."""
    L, h, v = sol.lib(), _dense_net(sol, (4, 64, 14, 14)), C.c_int()

    def state():
        assert L.sol_network_layer_dense(h, 2, C.byref(v)) == 0
        return v.value

    assert state() == 1
    for layer in (1, 2):
        assert L.sol_network_set_layer_tile(h, layer, 5) == 0 and state() == 0
        assert L.sol_network_set_layer_tile(h, 3 - layer, 0) == 0 and state() == 0
        assert L.sol_network_set_layer_tile(h, layer, 0) == 0 and state() == 1
    assert L.sol_network_set_layer_tile(h, 0, 5) == 0 and state() == 1       # any other layer's tile leaves it alone
    L.sol_network_destroy(h)


@pytest.mark.parametrize("n,hw,c,s,k,fused", [
    (1, 7, 32, 1, 192, 1), (1, 7, 32, 1, 256, 0), (1, 14, 32, 1, 2048, 0), (16, 112, 32, 1, 1024, 1), (4, 56, 64, 1, 1024, 0), (64, 56, 64, 1, 128, 1),
    (1, 7, 128, 1, 128, 1), (1, 7, 128, 1, 256, 0), (64, 28, 256, 1, 256, 1), (1, 28, 256, 1, 256, 0), (64, 14, 512, 1, 512, 1), (1, 7, 512, 1, 64, 0),
    (1, 14, 64, 2, 192, 0), (64, 56, 128, 2, 256, 1), (1, 7, 256, 2, 64, 0), (64, 28, 256, 2, 128, 1), (4, 14, 512, 2, 64, 0), (64, 28, 256, 2, 2048, 0)])
def test_depthwise_pair_one_launch_or_two(sol, n, hw, c, s, k, fused):
    """A depthwise convolution and the 1x1 behind it run as one launch where their tiles are many for the output channels that each
    has to pass; few tiles with many output channels keep the two launches (one was up to five times slower)."""
    layers = [wl.conv(c, 3, s=s, dw=True), wl.conv(k, 1, p=0), wl.conv(8, 1, p=0)]
    st, h = _create(sol, layers, (n, c, hw, hw), sol.BF16)
    v = C.c_int()
    assert st == 0 and sol.lib().sol_network_layer_dwpw(h, 1, C.byref(v)) == 0
    sol.lib().sol_network_destroy(h)
    assert v.value == fused


@pytest.mark.parametrize("n,hw,c,e1,e3,fused", [
    (1, 13, 64, 64, 64, 1), (1, 13, 64, 256, 256, 0), (64, 55, 64, 64, 64, 1), (80, 55, 64, 64, 64, 0), (8, 55, 64, 128, 128, 1), (64, 55, 64, 128, 128, 0),
    (1, 27, 256, 128, 128, 1), (1, 27, 512, 128, 128, 0), (16, 27, 128, 128, 128, 1), (64, 27, 128, 128, 128, 0), (1, 13, 512, 256, 256, 0)])
def test_fire_module_one_launch_or_not(sol, n, hw, c, e1, e3, fused):
    """A fire module runs as one launch where its tile's path is short -- few input and output channels -- and its tiles are few; wide
    modules of few tiles were up to 1.5 times slower that way."""
    layers = [wl.conv(c, 1, p=0), wl.conv(32, 1, p=0), wl.conv(e1, 1, p=0, src=1), wl.conv(e3, 3, src=1), wl.concat(2, 3), wl.conv(8, 1, p=0)]
    st, h = _create(sol, layers, (n, 64, hw, hw), sol.BF16)
    v = C.c_int()
    assert st == 0 and sol.lib().sol_network_layer_fire(h, 3, C.byref(v)) == 0
    sol.lib().sol_network_destroy(h)
    assert v.value == fused


@pytest.mark.parametrize("first", [0, 1])
def test_fire_module_of_one_join_only(sol, first):
    """Expands that different joins of one dense chain take are no module: the layer that reads the earlier join (here layer 4) runs
    between them.  The same expands under one join of a chain are one."""
    L, c, cat, v = sol.lib(), wl.conv, wl.concat, C.c_int()
    head = [c(64, 1, p=0), c(32, 1, p=0, src=0), c(64, 1, p=0, src=1)]
    join = cat(0, 2) if first == 0 else cat(2, 0)
    apart = head + [join, c(64, 1, p=0, src=3), c(64, 3, src=1), cat(3, 5), c(64, 1, p=0, src=6, res=4), c(8, 1, p=0)]
    one = head + [c(64, 3, src=1), cat(2, 3), c(64, 1, p=0, src=4), cat(4, 5), c(8, 1, p=0)]
    for layers, expand, state in ((apart, 5, -1), (one, 3, 1)):
        st, h = _create(sol, layers, (1, 64, 8, 8), sol.BF16)
        assert st == 0
        assert L.sol_network_layer_fire(h, expand, C.byref(v)) == 0 and v.value == state
        for i in (1, 2):
            assert L.sol_network_layer_fused_into(h, i, C.byref(v)) == 0 and v.value == (expand if state == 1 else i)
        L.sol_network_destroy(h)


def test_layer_output_only_of_stored_layers(sol):
    """A layer without a tensor of its own in the workspace has no address (it used to be another layer's)."""
    L, c = sol.lib(), wl.conv
    layers = [c(64, 7, 2, 3, bn=False), wl.pool("max", 3, 2, 1),                              # stem + pool in one launch
              c(64, 1, p=0), c(64, 1, p=0, src=1, act="none"), c(64, 1, p=0, src=2, res=3),  # projection shortcut inside the expand
              c(32, 3), c(32, 3, src=4), wl.concat(5, 6), c(128, 1, p=0, src=7, pre_bn=True), c(32, 3), c(8, 1, p=0)]
    own = {0: False, 3: False, 5: False, 6: False}
    for flags in (0, sol.NET_KEEP_ACTIVATIONS):
        st, h = _create(sol, layers, (2, 3, 64, 64), sol.BF16, flags)
        assert st == 0, L.sol_last_error()
        ws, seen = 1 << 40, []
        for i in range(len(layers) - 1):
            p = C.c_void_p()
            st = L.sol_network_layer_output(h, i, C.c_void_p(ws), C.byref(p))
            assert st == (0 if flags or own.get(i, True) else 6), (flags, i, st)
            if st == 0:
                assert ws <= p.value < ws + L.sol_network_workspace_bytes(h)
                seen.append(p.value)
        assert not flags or len(set(seen)) == len(seen)
        L.sol_network_destroy(h)


def test_small_tile_refusal_names_its_condition(sol):
    """32 bf16 channels are 64 bytes: a small tile forced on them is refused with the rule that they miss."""
    fake, null = C.c_void_p(0x1000), C.c_void_p(0)
    sol.sol_debug_set_conv_tile(81)
    try:
        st = sol.lib().sol_conv2d_fused(C.byref(sol.TensorDesc(1, 8, 8, 32, sol.BF16)), fake, C.byref(sol.ConvDesc(32, 32, 3, 3, 1, 1, 1, 1)), fake, null,
                                        null, null, 0, None, fake, null, null, null)
    finally:
        sol.sol_debug_set_conv_tile(0)
    assert st == 6 and "multiples of 128 bytes" in sol.lib().sol_last_error().decode()
