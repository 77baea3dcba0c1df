"""The weight-streaming linear kernel (up to 128 rows, long reductions) against the CPU checker: row and feature tiles with
remainders, reductions that end inside a 128-byte stage or give the eight waves unequal shares, with and without bias."""
import numpy as np
import pytest

import oracle as orc
from paper_2003_10688_amd import workloads as wl
from test_gpu_parity import TOL, rel_err, sol  # noqa: F401  (sol: the module fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows,kin,out", [
    (1, 2048, 10),        # one row, one ragged feature tile
    (16, 2056, 33),       # a full 16-row block; the last stage holds 16 (bf16) or 32 (fp32) bytes
    (17, 2112, 1000),     # two row blocks, the second nearly empty
    (33, 3000, 130),      # four row blocks; last stage 112 (bf16) or 96 (fp32) bytes
    (64, 2048, 4104),     # 32-feature tiles with a remainder
    (65, 2088, 72),       # two row tiles sharing their weights
    (128, 2048, 4100),    # both at their largest
    (128, 2048, 6656),    # bf16: many rows for the reduction, the eight-wave ring kernel's
    (1, 2048, 4104),      # up to 16 and up to 32 rows on 32-feature tiles (more than 4096 features), with remainders of all three
    (16, 2056, 8200),
    (17, 2056, 4104),
    (32, 2112, 4100),
    (64, 2048, 12800),    # the first width of one row tile that is
])
def test_linear_stream(sol, dt, rows, kin, out):  # noqa: F811
    rng = np.random.default_rng([rows, kin, out])
    d = sol.BF16 if dt == "bf16" else sol.F32
    x, w, b = rng.standard_normal((rows, kin)), rng.standard_normal((out, kin)) / np.sqrt(kin), rng.standard_normal(out)
    if dt == "bf16":
        x, w = wl.to_bf16_grid(x), wl.to_bf16_grid(w)
    cd = sol.ConvDesc(out, kin, 1, 1, 1, 1, 0, 0)
    wp = sol.sol_pack_conv_weights(cd, d, sol.dev_f32(w.reshape(out, kin, 1, 1)))
    for bias, act in ((b, sol.ACT_RELU), (None, sol.ACT_NONE)):
        y = sol.sol_linear(sol.to_device_nhwc(x, d), wp, None if bias is None else sol.dev_f32(bias), out, act)
        want = orc.linear(x, w, np.zeros(out) if bias is None else bias)
        if act == sol.ACT_RELU:
            want = np.maximum(want, 0)
        assert rel_err(sol.to_host_nchw(y).reshape(rows, out), want) <= TOL[dt]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows,kin,out", [(65, 4096, 40), (128, 2304, 600), (128, 2048, 6656)])
def test_linear_equal_rows_equal_bits(sol, dt, rows, kin, out):  # noqa: F811
    """A row's sums run in one order wherever it stands: the rows of the second row tile repeat those of the first."""
    rng = np.random.default_rng([rows, kin, out])
    d = sol.BF16 if dt == "bf16" else sol.F32
    x = rng.standard_normal((64, kin))[np.arange(rows) % 64]
    cd = sol.ConvDesc(out, kin, 1, 1, 1, 1, 0, 0)
    wp = sol.sol_pack_conv_weights(cd, d, sol.dev_f32((rng.standard_normal((out, kin)) / np.sqrt(kin)).reshape(out, kin, 1, 1)))
    y = sol.to_host_nchw(sol.sol_linear(sol.to_device_nhwc(x, d), wp, None, out, sol.ACT_NONE)).reshape(rows, out)
    assert np.array_equal(y[64:], y[:rows - 64])
