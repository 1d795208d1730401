"""Backward-weight of small problems (wave_dw.hip), every shape of it, as one range of pixels and as several: ragged filters,
columns and pixels, 1x1 filters read linearly, strides, first layers' packings, padded channels, KCRS and bf16 results."""
import numpy as np
import pytest
import torch

from paper_1512_01274_amd import inputs as gen
from tests import util

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad
DIMS = [
    (2, 40, 9, 11, 72, 3, 3, 1, 1),
    (3, 136, 7, 7, 24, 1, 1, 1, 0),        # 1x1: pixels in a row
    (5, 16, 6, 5, 40, 1, 1, 2, 0),         # ... strided, fewer pixels than the waves' first steps
    (1, 24, 13, 70, 16, 5, 3, 1, 2),       # unequal filter sides
    (1, 8, 3, 4, 8, 2, 2, 1, 0),           # six pixels
    (40, 16, 3, 3, 32, 3, 3, 1, 1),        # images of fewer pixels than a step
    (6, 30, 12, 13, 50, 3, 3, 1, 1),       # padded channels on both sides
    (2, 3, 37, 33, 16, 7, 7, 2, 3),        # space-to-depth columns
    (2, 3, 20, 18, 24, 3, 3, 1, 1),        # rows of four channels per pixel
]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


def _names():
    from paper_1512_01274_amd import mxc as m
    return m.mxc_tile_names(5)


@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("ranges", [1, 3])
@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("name", _names())
def test_weight_gradient(mxc, oracle, monkeypatch, name, dims, ranges, layout):
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="bf16", dist="normal")
    run = util.Runner(mxc, dims, "bf16", layout)
    a = (*dims, run.dt, run.lay)
    monkeypatch.setenv("MXC_FORCE_WGRAD", f"{name}/{ranges}")
    ref = oracle.conv2d_bwd_weight(x, dy, w.shape, st, pad)
    den = oracle.conv2d_bwd_weight(np.abs(x), np.abs(dy), w.shape, st, pad)
    for dtype, call, op in ((torch.float32, mxc.mxc_conv2d_bwd_weight, mxc.MXC_BWD_WEIGHT), (torch.bfloat16, mxc.mxc_conv2d_bwd_weight_bf16, mxc.MXC_BWD_WEIGHT_BF16)):
        dw = torch.full((w.size + 64,), 7.0, dtype=dtype, device="cuda")
        call(*a, run._in(x), run._in(dy), dw, run._ws(op))
        assert name in mxc.mxc_last_variant()
        assert bool((dw[w.size:] == 7.0).all())
        got = dw[:w.size].double().cpu().numpy()
        got = got.reshape(K, R, S, C).transpose(0, 3, 1, 2) if layout == "nhwc" else got.reshape(w.shape)
        assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "bf16", dtype == torch.bfloat16)), dims


def test_chosen_by_size(mxc, monkeypatch):
    """Which kernel a problem gets by itself: a small one this, a large one the planned tiles."""
    monkeypatch.delenv("MXC_FORCE_WGRAD", raising=False)
    for dims, wave in (((1, 64, 13, 13, 64, 3, 3, 1, 1), True), ((64, 256, 28, 28, 256, 3, 3, 1, 1), False)):
        N, C, H, W, K, R, S, st, pad = dims
        x = torch.zeros(N, H, W, C, dtype=torch.bfloat16, device="cuda")
        dy = torch.zeros(N, H, W, K, dtype=torch.bfloat16, device="cuda")
        dw = torch.empty(K, R, S, C, device="cuda")
        a = (*dims, mxc.MXC_BF16, mxc.MXC_NHWC)
        mxc.mxc_conv2d_bwd_weight(*a, x, dy, dw, mxc.alloc_workspace(mxc.mxc_conv2d_workspace_bytes(mxc.MXC_BWD_WEIGHT, *a)))
        assert ("wgrad_wave" in mxc.mxc_last_variant()) == wave, mxc.mxc_last_variant()
