"""Input gradients of strided first layers that the streaming and the window kernel store straight into the image: odd and even channels,
widths and padding (element and pair stores), filter sizes with and without a remainder, grids that end before the image
does (which take the separate un-packing), and a padded channel count of dy."""
import numpy as np
import pytest
import torch

from paper_1512_01274_amd import inputs as gen
from tests import util

pytestmark = pytest.mark.gpu

SHAPES = [
    (2, 3, 43, 48, 16, 11, 11, 4, 2),
    (3, 3, 20, 26, 8, 3, 3, 2, 1),
    (1, 3, 33, 37, 24, 7, 7, 2, 3),
    (2, 4, 31, 40, 16, 7, 7, 2, 3),
    (2, 1, 24, 25, 16, 5, 5, 2, 2),
    (1, 2, 30, 22, 12, 5, 6, 4, 0),
    (2, 3, 27, 28, 8, 4, 4, 4, 0),        # rows and columns no block covers
    (70, 3, 9, 10, 16, 3, 3, 2, 0),       # row tiles that span images
]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


@pytest.mark.parametrize("kernel", ["igemm_stream", "igemm_window"])
@pytest.mark.parametrize("dims", SHAPES)
def test_image_store(mxc, oracle, monkeypatch, dims, kernel):
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="bf16", dist="normal")
    run = util.Runner(mxc, dims, "bf16", "nhwc")
    monkeypatch.setenv("MXC_FORCE_VARIANT", kernel)
    dx = torch.full((N * C * H * W,), float("nan"), dtype=torch.bfloat16, device="cuda")
    mxc.mxc_conv2d_bwd_data(*dims, run.dt, run.lay, run._in(dy), run._in(w), dx, run._ws(mxc.MXC_BWD_DATA))
    if kernel == "igemm_stream" or K % 16 == 0:
        assert mxc.mxc_last_variant().endswith("s2d+" + kernel), mxc.mxc_last_variant()
    ref = oracle.conv2d_bwd_data(dy, w, x.shape, st, pad)
    den = oracle.conv2d_bwd_data(np.abs(dy), np.abs(w), x.shape, st, pad)
    got = run._out(dx, (N, C, H, W))
    assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "bf16", True)), dims
    prepared = mxc.alloc_workspace(mxc.mxc_conv2d_workspace_bytes(mxc.MXC_BWD_DATA_FILTER, *dims, run.dt, run.lay))
    mxc.mxc_conv2d_bwd_data_prepare_filter(*dims, run.dt, run.lay, run._in(w), prepared)
    again = torch.full_like(dx, float("nan"))
    mxc.mxc_conv2d_bwd_data_prepared(*dims, run.dt, run.lay, run._in(dy), prepared, None, again, run._ws(mxc.MXC_BWD_DATA_PREPARED))
    torch.cuda.synchronize()
    assert torch.equal(again.view(torch.int16), dx.view(torch.int16)), dims
