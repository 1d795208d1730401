"""Backward-weight by the kernel whose taps of a filter row share their pixels: every shape, as one range of pixels and as several: ragged
channels on both sides, images narrower and shorter than the filter, stages that span many images, filters of other heights than widths,
padded channels, KCRS and bf16 results."""
import numpy as np
import pytest
import torch

from paper_1512_01274_amd import inputs as gen
from tests import util

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, pad: Q = W where S = 2*pad + 1, or S = 3 without padding
DIMS = [
    (6, 40, 9, 11, 72, 3, 3, 1),
    (3, 24, 7, 7, 136, 5, 5, 2),
    (9, 72, 5, 1, 40, 5, 5, 2),            # no tap but the middle column's meets a pixel
    (2, 8, 3, 2, 8, 3, 3, 1),              # twelve pixels
    (37, 96, 8, 8, 200, 3, 3, 1),
    (5, 16, 6, 37, 48, 1, 3, 1),           # P = H + 2
    (3, 48, 8, 5, 16, 5, 3, 1),            # P = H - 2
    (60, 32, 1, 3, 264, 3, 5, 2),          # a stage of 128 pixels is some 14 images
    (6, 30, 12, 13, 50, 3, 3, 1),          # padded channels on both sides
    (1, 64, 9, 150, 64, 5, 5, 2),
    (3, 40, 9, 11, 72, 3, 3, 0),           # no padding: positions of x without dy
    (2, 64, 4, 150, 48, 3, 3, 0),
    (37, 96, 8, 8, 200, 5, 3, 0),
    (5, 16, 5, 3, 24, 3, 3, 0),            # one column of dy
]
# first layers in space-to-depth form
FIRST = [(3, 3, 43, 39, 40, 11, 11, 4, 2), (2, 1, 64, 67, 16, 11, 11, 4, 2), (6, 4, 35, 50, 96, 5, 5, 2, 2)]


def _names():
    from paper_1512_01274_amd import mxc as m
    return [n.removeprefix("wgrad_run_") for n in m.mxc_tile_names(9)]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("ranges", [1, 4])
@pytest.mark.parametrize("name,dims", [(n, d) for n in _names() for d in DIMS + FIRST if not (n in ("96x64", "192x64") and d[6] == 5 and len(d) == 8)])      # (sums of 3*5 blocks do not fit)
def test_weight_gradient(mxc, oracle, monkeypatch, name, dims, ranges, layout):
    N, C, H, W, K, R, S, pad = dims[:7] + dims[-1:]
    full = dims if len(dims) == 9 else (*dims[:7], 1, pad)
    st = full[7]
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *full, dtype="bf16", dist="normal")
    run = util.Runner(mxc, full, "bf16", layout)
    a = (*full, run.dt, run.lay)
    monkeypatch.setenv("MXC_FORCE_WGRAD", f"wgrad_run_{name}/{ranges}")
    ref = oracle.conv2d_bwd_weight(x, dy, w.shape, st, pad)
    den = oracle.conv2d_bwd_weight(np.abs(x), np.abs(dy), w.shape, st, pad)
    for dtype, call, op in ((torch.float32, mxc.mxc_conv2d_bwd_weight, mxc.MXC_BWD_WEIGHT), (torch.bfloat16, mxc.mxc_conv2d_bwd_weight_bf16, mxc.MXC_BWD_WEIGHT_BF16)):
        dw = torch.full((w.size + 64,), 7.0, dtype=dtype, device="cuda")
        call(*a, run._in(x), run._in(dy), dw, run._ws(op))
        assert mxc.mxc_last_variant().endswith("wgrad_run_" + name)
        assert bool((dw[w.size:] == 7.0).all())
        got = dw[:w.size].double().cpu().numpy()
        got = got.reshape(K, R, S, C).transpose(0, 3, 1, 2) if layout == "nhwc" else got.reshape(w.shape)
        assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "bf16", dtype == torch.bfloat16)), dims


@pytest.mark.filterwarnings("ignore:invalid value")
def test_infinities_beside_the_borders(mxc, oracle, monkeypatch):
    """An infinite x at a row's end is not multiplied with what lies outside dy: results whose window does not hold it stay finite."""
    full = (3, 16, 5, 6, 16, 3, 3, 1, 1)
    x, w, dy = gen.random_case(5, *full, dtype="bf16", dist="normal")
    x[1, 2, 2, 5] = np.inf
    x[2, 3, 4, 0] = np.inf
    run = util.Runner(mxc, full, "bf16", "nhwc")
    monkeypatch.setenv("MXC_FORCE_WGRAD", "wgrad_run_64x64/1")
    got, ref = run.bwd_weight(x, dy), oracle.conv2d_bwd_weight(x, dy, w.shape, 1, 1)
    assert np.array_equal(np.isfinite(got), np.isfinite(ref)) and not np.isfinite(ref).all() and np.isfinite(ref[:, 2, :, 0]).any()
    full = (3, 16, 6, 8, 16, 3, 3, 1, 0)
    x, w, dy = gen.random_case(6, *full, dtype="bf16", dist="normal")
    x[1, 2, 5, 7] = np.inf
    run = util.Runner(mxc, full, "bf16", "nhwc")
    got, ref = run.bwd_weight(x, dy), oracle.conv2d_bwd_weight(x, dy, w.shape, 1, 0)
    assert np.array_equal(np.isfinite(got), np.isfinite(ref)) and not np.isfinite(ref).all() and np.isfinite(ref[:, 2]).any()


def test_chosen(mxc):
    """A layer far from the line between the kernels, in the pixel ranges that the plan gives it: whole numbers, exact in any order."""
    dims = (64, 64, 28, 28, 96, 5, 5, 1, 2)
    a = (*dims, mxc.MXC_BF16, mxc.MXC_NHWC)
    g = torch.Generator(device="cuda").manual_seed(2)
    x, dy = (torch.randint(-2, 3, (64, 28, 28, n), generator=g, device="cuda").float() for n in (64, 96))      # sums below 2^18
    dw = torch.empty(96, 5, 5, 64, device="cuda")
    mxc.mxc_conv2d_bwd_weight(*a, x.bfloat16(), dy.bfloat16(), dw, mxc.alloc_workspace(mxc.mxc_conv2d_workspace_bytes(mxc.MXC_BWD_WEIGHT, *a)))
    assert "wgrad_run_" in mxc.mxc_last_variant()
    padded, rows = torch.nn.functional.pad(x, (0, 0, 2, 2, 2, 2)), dy.reshape(-1, 96).T.contiguous()
    for r in range(5):
        for s in range(5):
            assert torch.equal(dw[:, r, s], rows @ padded[:, r:r + 28, s:s + 28].reshape(-1, 64)), (r, s)


def test_padded_channels_of_one_range(mxc, oracle):
    """A large dw of few pixels with channels that are padded: the wave kernel, which stores it in place without another pass."""
    dims = (4, 491, 14, 14, 300, 3, 3, 1, 1)
    x, w, dy = gen.random_case(9, *dims, dtype="bf16", dist="normal")
    run = util.Runner(mxc, dims, "bf16", "nhwc")
    got = run.bwd_weight(x, dy)
    assert "wgrad_run_" not in mxc.mxc_last_variant()
    ref, den = (oracle.conv2d_bwd_weight(f(x), f(dy), w.shape, 1, 1) for f in (lambda t: t, np.abs))
    assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "bf16", False))
