"""dx of first layers at stride 1 (csrc/taps_dx.hip): every channel count and filter size it takes, channels of dy that end inside a step of 32,
images narrower than a strip, strips and segments that end early, paddings from none to more than the filter reaches; the mask, the prepared
filter, and infinities and NaN opposite padding."""
import numpy as np
import pytest
import torch

from paper_1512_01274_amd import inputs as gen
from tests import util

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad
DIMS = [
    (2, 3, 33, 61, 64, 3, 3, 1, 1),        # two strips and one column, 9 steps
    (1, 1, 5, 30, 8, 3, 3, 1, 0),          # one strip exactly, fewer channels than a step
    (3, 2, 4, 7, 40, 3, 3, 1, 2),
    (1, 4, 70, 95, 128, 3, 3, 1, 1),
    (1, 3, 1, 1, 16, 3, 3, 1, 1),
    (1, 1, 29, 57, 96, 5, 5, 1, 2),
    (2, 2, 11, 28, 24, 5, 5, 1, 0),
    (1, 3, 40, 30, 72, 5, 5, 1, 2),
    (1, 4, 9, 65, 128, 5, 5, 1, 3),
    (40, 3, 12, 10, 32, 3, 3, 1, 1),
    (1, 3, 6, 9, 16, 3, 3, 1, 5),          # rows and columns of dy that lie outside dx altogether
]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


@pytest.fixture(autouse=True)
def forced(monkeypatch):
    monkeypatch.setenv("MXC_FORCE_VARIANT", "taps_dx")


@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("dims", DIMS)
def test_dx(mxc, oracle, dims, layout):
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="bf16", dist="normal")
    run = util.Runner(mxc, dims, "bf16", layout)
    a = (*dims, run.dt, run.lay)
    dx = torch.full((N * C * H * W + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
    mxc.mxc_conv2d_bwd_data(*a, run._in(dy), run._in(w), dx, run._ws(mxc.MXC_BWD_DATA))
    assert mxc.mxc_last_variant() == "bwd_data:smallc+taps_dx"
    assert bool((dx[-64:] == 7.0).all())
    ref = oracle.conv2d_bwd_data(dy, w, x.shape, st, pad)
    den = oracle.conv2d_bwd_data(np.abs(dy), np.abs(w), x.shape, st, pad)
    assert np.all(np.abs(run._out(dx[:-64], x.shape) - ref) <= util.tight_bound(ref, den, "bf16", True)), dims
    prepared = run._ws(mxc.MXC_BWD_DATA_FILTER)
    mxc.mxc_conv2d_bwd_data_prepare_filter(*a, run._in(w), prepared)
    again, masked = (torch.full((N * C * H * W,), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    mxc.mxc_conv2d_bwd_data_prepared(*a, run._in(dy), prepared, None, again, run._ws(mxc.MXC_BWD_DATA_PREPARED))
    assert torch.equal(again, dx[:-64])
    mxc.mxc_conv2d_bwd_data_relu(*a, run._in(dy), run._in(w), run._in(x), masked, run._ws(mxc.MXC_BWD_DATA_RELU))
    assert torch.equal(masked, torch.where(run._in(x).reshape(-1) > 0, again, torch.zeros_like(again)))


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("R", [3, 5])
def test_taps_outside_are_left_out(mxc, bad, R):
    """A filter row that holds no finite value reaches dx only from dy rows that exist: dx's last rows lie under its first row
    alone where dy has no row."""
    dims = (1, 3, 9, 34, 16, R, R, 1, 0)
    N, C, H, W, K, _, S, st, pad = dims
    x, w, dy = gen.random_case(5, *dims, dtype="bf16", dist="normal")
    worse = w.copy()
    worse[:, :, 0, :] = bad
    run = util.Runner(mxc, dims, "bf16", "nhwc")
    out = []
    for f in (w, worse):
        dx = torch.empty(N * C * H * W, dtype=torch.bfloat16, device="cuda")
        mxc.mxc_conv2d_bwd_data(*dims, run.dt, run.lay, run._in(dy), run._in(f), dx, run._ws(mxc.MXC_BWD_DATA))
        out.append(dx.view(H, W, C))
    first_outside = H - R + 1              # rows from here on have no dy row under the filter's row 0
    assert torch.equal(out[0][first_outside:], out[1][first_outside:])
    assert not bool(torch.isfinite(out[1][:first_outside]).any())
