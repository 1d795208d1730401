"""bf16 NCHW problems whose result the wave kernel stores straight to its planes: every shape of the kernel, planes of whole and of
broken groups of four pixels, images that end inside a tile, channel counts that are no multiple of 8, bias, ReLU and mask."""
import numpy as np
import pytest
import torch

from paper_1512_01274_amd import inputs as gen
from tests import util

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad
DIMS = [
    (2, 24, 6, 10, 40, 3, 3, 1, 1),
    (3, 32, 7, 7, 72, 1, 1, 1, 0),
    (7, 16, 3, 3, 16, 3, 3, 1, 1),         # a group of four pixels spans two images
    (1, 64, 13, 9, 136, 3, 3, 1, 1),
    (5, 21, 8, 8, 32, 3, 3, 1, 0),
    (2, 40, 1, 1, 24, 1, 1, 1, 0),         # planes of one pixel
]
FORWARD = DIMS + [(2, 24, 9, 11, 35, 3, 3, 2, 1), (1, 3, 14, 12, 16, 3, 3, 2, 1)]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


def _names():
    from paper_1512_01274_amd import mxc as m
    return m.mxc_tile_names(4)


@pytest.mark.parametrize("dims", FORWARD)
@pytest.mark.parametrize("name", _names())
def test_forward(mxc, oracle, monkeypatch, name, dims):
    monkeypatch.setenv("MXC_FORCE_VARIANT", name)
    N, C, H, W, K, R, S, st, pad = dims
    x, w, _ = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="bf16", dist="normal")
    bias = np.linspace(-1.0, 1.0, K).astype(np.float32)
    run = util.Runner(mxc, dims, "bf16", "nchw")
    y = torch.full((N * K * run.P * run.Q + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
    mxc.mxc_conv2d_fwd_bias_act(*dims, run.dt, run.lay, run._in(x), run._in(w), torch.from_numpy(bias).cuda(), 1, y, run._ws(mxc.MXC_FWD))
    assert mxc.mxc_last_variant().endswith(name)
    assert bool((y[-64:] == 7.0).all())
    ref, den = oracle.conv2d_fwd_bias_act(x, w, bias, True, st, pad)
    assert np.all(np.abs(run._out(y[:-64], (N, K, run.P, run.Q)) - ref) <= util.tight_bound(ref, den, "bf16", True)), dims


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("name", [n for n in _names() if "16x16" not in n])
def test_input_gradient(mxc, oracle, monkeypatch, name, dims):
    monkeypatch.setenv("MXC_FORCE_VARIANT", name)
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="bf16", dist="normal")
    run = util.Runner(mxc, dims, "bf16", "nchw")
    a = (*dims, run.dt, run.lay)
    dx, masked, prepared = (torch.full((N * C * H * W + 64,), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(3))
    mxc.mxc_conv2d_bwd_data(*a, run._in(dy), run._in(w), dx, run._ws(mxc.MXC_BWD_DATA))
    assert mxc.mxc_last_variant().endswith(name)
    ref = oracle.conv2d_bwd_data(dy, w, x.shape, st, pad)
    den = oracle.conv2d_bwd_data(np.abs(dy), np.abs(w), x.shape, st, pad)
    assert np.all(np.abs(run._out(dx[:-64], x.shape) - ref) <= util.tight_bound(ref, den, "bf16", True)), dims
    mxc.mxc_conv2d_bwd_data_relu(*a, run._in(dy), run._in(w), run._in(x), masked, run._ws(mxc.MXC_BWD_DATA_RELU))
    pw = run._ws(mxc.MXC_BWD_DATA_FILTER)
    mxc.mxc_conv2d_bwd_data_prepare_filter(*a, run._in(w), pw)
    mxc.mxc_conv2d_bwd_data_prepared(*a, run._in(dy), pw, None, prepared, run._ws(mxc.MXC_BWD_DATA_PREPARED))
    assert torch.equal(prepared, dx)
    assert torch.equal(masked[:-64], torch.where(run._in(x).reshape(-1) > 0, dx[:-64], torch.zeros_like(dx[:-64])))
    assert all(bool((t[-64:] == 7.0).all()) for t in (dx, masked, prepared))
