"""bf16 channel counts that are no multiple of 8 run on the matrix cores with zero-padded copies: every combination of
ragged C and K, each pass, both layouts, plain, grouped and with a prepared filter, at one and several tiles."""
import numpy as np
import pytest
import torch

from paper_1512_01274_amd import inputs as gen
from tests import util

pytestmark = pytest.mark.gpu

SHAPES = [
    (2, 30, 13, 11, 50, 3, 3, 2, 1),
    (3, 5, 9, 9, 7, 5, 5, 1, 2),
    (1, 16, 8, 9, 129, 1, 1, 1, 0),       # columns one past a tile
    (2, 71, 10, 7, 24, 3, 3, 1, 1),
    (1, 3, 20, 18, 13, 3, 3, 1, 1),       # first layers: few channels, ragged K
    (1, 3, 35, 35, 9, 11, 11, 4, 2),
    (2, 100, 6, 6, 66, 1, 1, 2, 0),       # residue classes no tap reaches
    (40, 515, 1, 1, 1001, 1, 1, 1, 0),    # FullyConnected-shaped, long reduction
]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("dims", SHAPES)
def test_ragged_channels(mxc, oracle, dims, layout):
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="bf16", dist="normal")
    run = util.Runner(mxc, dims, "bf16", layout)
    bias = np.linspace(-1.0, 1.0, K).astype(np.float32)

    def check(name, got, ref, den, rounded=True):
        assert "direct" not in mxc.mxc_last_variant(), (name, dims, mxc.mxc_last_variant())
        assert util.metric(got, ref, den) <= util.TOL["bf16"], (name, dims)
        assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "bf16", rounded)), (name, dims)

    new = lambda n: torch.full((n,), float("nan"), dtype=torch.bfloat16, device="cuda")
    y = new(N * K * run.P * run.Q)
    mxc.mxc_conv2d_fwd_bias_act(*dims, run.dt, run.lay, run._in(x), run._in(w), torch.from_numpy(bias).cuda(), 1, y, run._ws(mxc.MXC_FWD))
    check("fwd", run._out(y, (N, K, run.P, run.Q)), *oracle.conv2d_fwd_bias_act(x, w, bias, True, st, pad))

    ref, den = oracle.conv2d_bwd_data_relu(dy, w, x, st, pad)
    dx = new(N * C * H * W)
    mxc.mxc_conv2d_bwd_data_relu(*dims, run.dt, run.lay, run._in(dy), run._in(w), run._in(x), dx, run._ws(mxc.MXC_BWD_DATA_RELU))
    check("bwd_data", run._out(dx, (N, C, H, W)), ref, den)
    prepared = mxc.alloc_workspace(mxc.mxc_conv2d_workspace_bytes(mxc.MXC_BWD_DATA_FILTER, *dims, run.dt, run.lay))
    mxc.mxc_conv2d_bwd_data_prepare_filter(*dims, run.dt, run.lay, run._in(w), prepared)
    again = new(N * C * H * W)
    mxc.mxc_conv2d_bwd_data_prepared(*dims, run.dt, run.lay, run._in(dy), prepared, run._in(x), again, run._ws(mxc.MXC_BWD_DATA_PREPARED_RELU))
    torch.cuda.synchronize()
    assert torch.equal(again.view(torch.int16), dx.view(torch.int16)), dims

    ref = oracle.conv2d_bwd_weight(x, dy, w.shape, st, pad)
    den = oracle.conv2d_bwd_weight(np.abs(x), np.abs(dy), w.shape, st, pad)
    check("bwd_weight", run.bwd_weight(x, dy), ref, den, rounded=False)
