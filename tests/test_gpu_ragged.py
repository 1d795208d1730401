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


# On either side of the lines between one thread per result and the padded path (NHWC): heads, several results per pixel and
# tap, strided, first layers; dw of few and many multiply-adds, of few pixels (one range, no summing launch) and more
SMALL = [
    ((128, 512, 1, 1, 10, 1, 1, 1, 0), True, False),
    ((8, 512, 1, 1, 10, 1, 1, 1, 0), True, True),
    ((128, 512, 1, 1, 2, 1, 1, 1, 0), True, True),
    ((128, 513, 1, 1, 2, 1, 1, 1, 0), True, False),
    ((24, 72, 1, 1, 39, 1, 1, 1, 0), True, True),
    ((24, 72, 1, 1, 41, 1, 1, 1, 0), False, True),
    ((300, 64, 1, 1, 100, 1, 1, 1, 0), False, False),
    ((1, 64, 28, 28, 1, 3, 3, 1, 1), True, True),
    ((3, 16, 9, 7, 6, 3, 3, 1, 1), True, False),
    ((3, 16, 9, 7, 7, 3, 3, 1, 1), False, False),
    ((2, 24, 11, 10, 12, 3, 3, 2, 1), True, False),
    ((2, 3, 12, 13, 10, 3, 3, 1, 1), True, True),
    ((2, 3, 12, 13, 11, 3, 3, 1, 1), False, True),
    ((4, 64, 65, 65, 4, 3, 3, 1, 1), False, False),
]


@pytest.mark.parametrize("dims,dx_direct,dw_direct", SMALL)
def test_small_ragged_gradients(mxc, oracle, dims, dx_direct, dw_direct):
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="bf16", dist="normal")
    run = util.Runner(mxc, dims, "bf16", "nhwc")
    a = (*dims, run.dt, run.lay)
    ref, den = oracle.conv2d_bwd_data_relu(dy, w, x, st, pad)
    bound = util.tight_bound(ref, den, "bf16", True)
    dx = torch.full((N * C * H * W,), 7.0, dtype=torch.bfloat16, device="cuda")
    mxc.mxc_conv2d_bwd_data_relu(*a, run._in(dy), run._in(w), run._in(x), dx, run._ws(mxc.MXC_BWD_DATA_RELU))
    assert ("direct" in mxc.mxc_last_variant()) == dx_direct, mxc.mxc_last_variant()
    assert np.all(np.abs(run._out(dx, x.shape) - ref) <= bound)
    prepared = mxc.alloc_workspace(mxc.mxc_conv2d_workspace_bytes(mxc.MXC_BWD_DATA_FILTER, *a))
    mxc.mxc_conv2d_bwd_data_prepare_filter(*a, run._in(w), prepared)
    again = torch.full_like(dx, 7.0)
    mxc.mxc_conv2d_bwd_data_prepared(*a, run._in(dy), prepared, run._in(x), again, run._ws(mxc.MXC_BWD_DATA_PREPARED_RELU))
    assert torch.equal(again.view(torch.int16), dx.view(torch.int16))

    ref = oracle.conv2d_bwd_weight(x, dy, w.shape, st, pad)
    den = oracle.conv2d_bwd_weight(np.abs(x), np.abs(dy), w.shape, st, pad)
    guard = torch.full((w.size + 4096,), 7.0, device="cuda")
    mxc.mxc_conv2d_bwd_weight(*a, run._in(x), run._in(dy), guard, run._ws(mxc.MXC_BWD_WEIGHT))
    assert ("direct" in mxc.mxc_last_variant()) == dw_direct, mxc.mxc_last_variant()
    got = guard[:w.size].double().cpu().numpy().reshape(K, R, S, C).transpose(0, 3, 1, 2)
    assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "bf16", False)) and bool((guard[w.size:] == 7.0).all())
    dw = torch.full((w.size,), 7.0, dtype=torch.bfloat16, device="cuda")
    mxc.mxc_conv2d_bwd_weight_bf16(*a, run._in(x), run._in(dy), dw, run._ws(mxc.MXC_BWD_WEIGHT_BF16))
    got = util.to_host_f64(dw).reshape(K, R, S, C).transpose(0, 3, 1, 2)
    assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "bf16", True))
