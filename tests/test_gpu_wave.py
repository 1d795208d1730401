"""The implicit GEMM of small problems (wave.hip), every shape of it: ragged rows, columns and reductions, reductions of whole and
of broken 32-element steps, 1x1 filters, strides, bias and ReLU, the masked input gradient from the filter in place and from a
prepared one."""
import numpy as np
import pytest
import torch

from paper_1512_01274_amd import inputs as gen
from tests import util

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad
DIMS = [
    (2, 64, 9, 11, 40, 3, 3, 1, 1),        # whole steps in both passes' taps (C) and broken ones (K)
    (1, 24, 13, 7, 96, 5, 3, 1, 2),        # unequal filter sides, C below a step
    (3, 32, 7, 7, 64, 1, 1, 1, 0),         # 1x1: one tap, every pixel inside
    (5, 8, 6, 5, 8, 1, 1, 1, 1),           # 1x1 with padding, reduction shorter than a step
    (1, 264, 5, 6, 24, 2, 2, 1, 0),        # long reduction, few rows
    (17, 16, 8, 8, 136, 3, 3, 1, 1),       # several row and column tiles of every shape
]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


def _names():
    from paper_1512_01274_amd import mxc as m
    return m.mxc_tile_names(4)


def _case(dims):
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="bf16", dist="normal")
    return np.maximum(x, 0.0).astype(np.float32), w, dy


def _forward(mxc, oracle, dims, name):
    N, C, H, W, K, R, S, st, pad = dims
    x, w, _ = _case(dims)
    bias = np.linspace(-1.0, 1.0, K).astype(np.float32)
    run = util.Runner(mxc, dims, "bf16", "nhwc")
    y = torch.full((N * K * run.P * run.Q + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")
    mxc.mxc_conv2d_fwd_bias_act(*dims, run.dt, run.lay, run._in(x), run._in(w), torch.from_numpy(bias).cuda(), 1, y, run._ws(mxc.MXC_FWD))
    assert mxc.mxc_last_variant().split(":")[-1].split("+")[-1] == name
    assert bool(torch.isnan(y[-64:]).all())
    ref, den = oracle.conv2d_fwd_bias_act(x, w, bias, True, st, pad)
    got = run._out(y[:-64], (N, K, run.P, run.Q))
    assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "bf16", True)), dims


@pytest.mark.parametrize("dims", DIMS + [(2, 40, 12, 11, 50, 3, 3, 2, 1), (4, 3, 20, 18, 24, 3, 3, 1, 1), (2, 3, 33, 30, 16, 7, 7, 2, 3)])
@pytest.mark.parametrize("name", _names())
def test_forward(mxc, oracle, monkeypatch, name, dims):
    monkeypatch.setenv("MXC_FORCE_VARIANT", name)
    _forward(mxc, oracle, dims, name)


@pytest.mark.parametrize("dims", DIMS + [(2, 40, 9, 10, 30, 3, 3, 1, 1)])
@pytest.mark.parametrize("name", _names()[1:])
def test_masked_input_gradient(mxc, oracle, monkeypatch, name, dims):
    monkeypatch.setenv("MXC_FORCE_VARIANT", name)
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = _case(dims)
    run = util.Runner(mxc, dims, "bf16", "nhwc")
    a = (*dims, run.dt, run.lay)
    dx = torch.full((N * C * H * W + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")
    mxc.mxc_conv2d_bwd_data_relu(*a, run._in(dy), run._in(w), run._in(x), dx, run._ws(mxc.MXC_BWD_DATA_RELU))
    assert mxc.mxc_last_variant().split(":")[-1] == name
    assert bool(torch.isnan(dx[-64:]).all())
    ref, den = oracle.conv2d_bwd_data_relu(dy, w, x, st, pad)
    got = run._out(dx[:-64], (N, C, H, W))
    assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "bf16", True)), dims
    assert np.all(got[x <= 0] == 0)
    # from the re-packed filter: the same sums in the same order
    prepared = mxc.alloc_workspace(mxc.mxc_conv2d_workspace_bytes(mxc.MXC_BWD_DATA_FILTER, *a))
    mxc.mxc_conv2d_bwd_data_prepare_filter(*a, run._in(w), prepared)
    again = torch.full_like(dx, float("nan"))
    mxc.mxc_conv2d_bwd_data_prepared(*a, run._in(dy), prepared, run._in(x), again, run._ws(mxc.MXC_BWD_DATA_PREPARED_RELU))
    torch.cuda.synchronize()
    assert torch.equal(again[:-64].view(torch.int16), dx[:-64].view(torch.int16)), dims


def test_chosen_by_size(mxc, oracle, monkeypatch):
    """Which kernel a problem gets by itself: a small one this, a large one the planned tiles."""
    monkeypatch.delenv("MXC_FORCE_VARIANT", raising=False)
    for dims, wave in (((1, 64, 13, 13, 64, 3, 3, 1, 1), True), ((64, 256, 28, 28, 256, 3, 3, 1, 1), False)):
        N, C, H, W, K, R, S, st, pad = dims
        x = torch.zeros(N, H, W, C, dtype=torch.bfloat16, device="cuda")
        w = torch.zeros(K, R, S, C, dtype=torch.bfloat16, device="cuda")
        y = torch.empty(N, H, W, K, dtype=torch.bfloat16, device="cuda")
        a = (*dims, mxc.MXC_BF16, mxc.MXC_NHWC)
        mxc.mxc_conv2d_fwd(*a, x, w, y, mxc.alloc_workspace(mxc.mxc_conv2d_workspace_bytes(mxc.MXC_FWD, *a)))
        assert ("igemm_wave" in mxc.mxc_last_variant()) == wave, mxc.mxc_last_variant()
