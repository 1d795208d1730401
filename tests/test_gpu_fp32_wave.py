"""fp32 layers of whole 16-byte chunks of channels (the wave kernels of fp32.hip), every shape of them: ragged rows, columns and
reductions, steps in one tap and across taps, 1x1 filters, strides with residue classes no tap reaches, one and several
pixel ranges of dw, infinities and NaN opposite padding; NCHW problems on NHWC copies, planes of whole and of broken groups of
four pixels."""
import numpy as np
import pytest
import torch

from paper_1512_01274_amd import inputs as gen
from tests import util

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad
DIMS = [
    (2, 20, 9, 11, 36, 3, 3, 1, 1),
    (1, 48, 13, 7, 64, 5, 3, 1, 2),
    (3, 16, 7, 7, 132, 1, 1, 1, 0),
    (5, 4, 6, 5, 8, 1, 1, 2, 0),           # classes of dx that no tap reaches, fewer pixels than the first steps
    (2, 24, 12, 11, 40, 3, 3, 2, 1),
    (40, 8, 3, 3, 12, 2, 2, 1, 0),         # images of fewer pixels than a step
]
RANGES = [(40, 8, 12, 9, 12, 3, 3, 2, 1), (24, 12, 20, 21, 20, 3, 3, 1, 1), (60, 36, 13, 14, 36, 1, 1, 1, 0)]      # pixels enough for several ranges
LAYOUTS = ["nhwc", "nchw"]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


def _names(dw):
    from paper_1512_01274_amd import mxc as m
    return [n for n in m.mxc_tile_names(6) if ("_dw_" in n) == dw]


def _case(dims):
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="f32", dist="normal")
    return np.maximum(x, 0.0).astype(np.float32), w, dy


@pytest.mark.parametrize("dims", DIMS + [(2, 12, 8, 9, 30, 3, 3, 1, 1)])       # filters that are no multiple of 4: forward only
@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("name", _names(False))
def test_forward(mxc, oracle, monkeypatch, name, layout, dims):
    monkeypatch.setenv("MXC_FORCE_VARIANT", name)
    N, C, H, W, K, R, S, st, pad = dims
    x, w, _ = _case(dims)
    bias = np.linspace(-1.0, 1.0, K).astype(np.float32)
    run = util.Runner(mxc, dims, "f32", layout)
    y = torch.full((N * K * run.P * run.Q + 64,), 7.0, device="cuda")
    mxc.mxc_conv2d_fwd_bias_act(*dims, run.dt, run.lay, run._in(x), run._in(w), torch.from_numpy(bias).cuda(), 1, y, run._ws(mxc.MXC_FWD))
    assert mxc.mxc_last_variant().split(":")[-1] == name
    assert bool((y[-64:] == 7.0).all())
    ref, den = oracle.conv2d_fwd_bias_act(x, w, bias, True, st, pad)
    got = run._out(y[:-64], (N, K, run.P, run.Q))
    assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "f32", False)), dims


def _copies(dims, layout):
    """whether dx of an NCHW problem can run on copies: the filter's copy has to fit where dx's would lie"""
    N, C, H, W, K, R, S, st, pad = dims
    return layout == "nhwc" or R * S == 1 or K * C * R * S <= N * C * H * W


@pytest.mark.parametrize("dims", DIMS + [(3, 20, 9, 12, 12, 3, 3, 1, 1)])
@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("name", _names(False))
def test_masked_input_gradient(mxc, oracle, monkeypatch, name, layout, dims):
    monkeypatch.setenv("MXC_FORCE_VARIANT", name)
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = _case(dims)
    run = util.Runner(mxc, dims, "f32", layout)
    dx = torch.full((N * C * H * W + 64,), 7.0, device="cuda")
    mxc.mxc_conv2d_bwd_data_relu(*dims, run.dt, run.lay, run._in(dy), run._in(w), run._in(x), dx, run._ws(mxc.MXC_BWD_DATA_RELU))
    assert (mxc.mxc_last_variant().split(":")[-1] == name) == _copies(dims, layout)
    assert bool((dx[-64:] == 7.0).all())
    ref, den = oracle.conv2d_bwd_data_relu(dy, w, x, st, pad)
    got = run._out(dx[:-64], (N, C, H, W))
    assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "f32", False)), dims
    assert np.all(got[x <= 0] == 0)
    if layout == "nchw":                   # the prepared filter is a copy of the caller's: the same kernel, the same bits
        a = (*dims, run.dt, run.lay)
        plain, prepared = (torch.empty(N * C * H * W, device="cuda") for _ in range(2))
        mxc.mxc_conv2d_bwd_data(*a, run._in(dy), run._in(w), plain, run._ws(mxc.MXC_BWD_DATA))
        pw = run._ws(mxc.MXC_BWD_DATA_FILTER)
        mxc.mxc_conv2d_bwd_data_prepare_filter(*a, run._in(w), pw)
        mxc.mxc_conv2d_bwd_data_prepared(*a, run._in(dy), pw, None, prepared, run._ws(mxc.MXC_BWD_DATA_PREPARED))
        assert torch.equal(plain, prepared)


@pytest.mark.parametrize("ranges", [1, 3])
@pytest.mark.parametrize("dims", DIMS + RANGES)
@pytest.mark.parametrize("name", _names(True))
def test_weight_gradient(mxc, oracle, monkeypatch, name, dims, ranges):
    monkeypatch.setenv("MXC_FORCE_WGRAD", f"{name}/{ranges}")
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = _case(dims)
    run = util.Runner(mxc, dims, "f32", "nhwc")
    if dims in RANGES:                     # of fewer pixels the plan, which the ranges are limited to, has one or two
        assert mxc.mxc_conv2d_workspace_bytes(mxc.MXC_BWD_WEIGHT, *dims, run.dt, run.lay) >= 3 * 4 * w.size
    dw = torch.full((w.size + 64,), 7.0, device="cuda")
    mxc.mxc_conv2d_bwd_weight(*dims, run.dt, run.lay, run._in(x), run._in(dy), dw, run._ws(mxc.MXC_BWD_WEIGHT))
    assert mxc.mxc_last_variant().split(":")[-1] == name
    assert bool((dw[-64:] == 7.0).all())
    ref = oracle.conv2d_bwd_weight(x, dy, w.shape, st, pad)
    den = oracle.conv2d_bwd_weight(np.abs(x), np.abs(dy), w.shape, st, pad)
    got = dw[:-64].double().cpu().numpy().reshape(K, R, S, C).transpose(0, 3, 1, 2)
    assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "f32", False)), dims


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_taps_outside_are_left_out(mxc, monkeypatch, bad, layout):
    """A filter tap that holds no finite value meets the image only where it lies inside: the first rows of a padded layer
    must not see the filter's first row, whatever kernel sums them."""
    dims = (2, 16, 6, 7, 20, 3, 3, 1, 1)
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = _case(dims)
    run = util.Runner(mxc, dims, "f32", layout)
    a = (*dims, run.dt, run.lay)
    clean, worse = w.copy(), w.copy()
    worse[:, :, 0, :] = bad
    xp = np.maximum(x, 0.1)
    for name in _names(False):
        monkeypatch.setenv("MXC_FORCE_VARIANT", name)
        y = [torch.empty(N * K * H * W, device="cuda") for _ in range(2)]
        for f, out in zip((clean, worse), y):
            mxc.mxc_conv2d_fwd(*a, run._in(xp), run._in(f), out, run._ws(mxc.MXC_FWD))
        y = [t.view(N, H, W, K) if layout == "nhwc" else t.view(N, K, H, W).permute(0, 2, 3, 1) for t in y]
        first = [t[:, 0] for t in y]
        assert bool(torch.isfinite(first[1]).all()) and torch.allclose(first[0], first[1], rtol=1e-5, atol=1e-5)
        assert not bool(torch.isfinite(y[1][:, 1:]).any())
    if layout == "nchw":
        return
    # dy's first row does not meet the filter's first row in dw: its pixels there lie outside x
    bad_dy = dy.copy()
    bad_dy[:, :, 0, :] = bad
    for name in _names(True):
        monkeypatch.setenv("MXC_FORCE_WGRAD", f"{name}/1")
        dw = [torch.empty(K * C * R * S, device="cuda") for _ in range(2)]
        for g, out in zip((dy, bad_dy), dw):
            mxc.mxc_conv2d_bwd_weight(*a, run._in(xp), run._in(g), out, run._ws(mxc.MXC_BWD_WEIGHT))
        top = dw[1].view(K, R, S, C)[:, 0]
        assert bool(torch.isfinite(top).all())
