"""The tiled kernel's order of the reduction (all taps of a block of channels before the next block) where the last block of channels
is not whole: forward, and dx with the filter as it lies (transposed tiles) and re-packed, split and unsplit, narrow tiles."""
import numpy as np
import pytest
import torch

from tests import util

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


@pytest.mark.parametrize("tile", ["igemm_128x64_k64s2_w4", "igemm_128x64_k64s2_w4/3", "igemm_256x64_k32s3_w4", "igemm_128x32_k64s2_w4"])
@pytest.mark.parametrize("C", [296, 440])
def test_blocks_that_are_not_whole(mxc, oracle, monkeypatch, tile, C):
    monkeypatch.setenv("MXC_FORCE_VARIANT", tile)
    N, H, W, K = 17, 32, 31, 24                            # 16864 pixels
    rng = np.random.default_rng(C)
    few = rng.integers(-3, 4, (2, C, H, W)).astype(np.float32)         # small integers: exact in bf16 and in every order
    w = rng.integers(-2, 3, (K, C, 3, 3)).astype(np.float32)
    x = np.concatenate([few, np.zeros((N - 2, C, H, W), np.float32)])
    dims = (N, C, H, W, K, 3, 3, 1, 1)
    run = util.Runner(mxc, dims, "bf16", "nhwc")
    y = run._out(run.fwd(x, w, return_tensor=True), (N, K, H, W))
    ref = oracle.conv2d_fwd(few, w, 1, 1)
    assert np.all(np.abs(y[:2] - ref) <= 2.0 ** -8 * np.abs(ref)), "forward"       # the one rounding to bf16
    assert not y[2:].any()
    # dx of the layer that goes the other way: dy has C channels
    dims = (N, K, H, W, C, 3, 3, 1, 1)
    run = util.Runner(mxc, dims, "bf16", "nhwc")
    a = (*dims, run.dt, run.lay)
    wt = np.ascontiguousarray(w.transpose(1, 0, 2, 3))
    ref = oracle.conv2d_bwd_data(few, wt, (2, K, H, W), 1, 1)
    dx, prepared = (torch.full((N * K * H * W,), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    mxc.mxc_conv2d_bwd_data(*a, run._in(x), run._in(wt), dx, run._ws(mxc.MXC_BWD_DATA))
    pw = run._ws(mxc.MXC_BWD_DATA_FILTER)
    mxc.mxc_conv2d_bwd_data_prepare_filter(*a, run._in(wt), pw)
    mxc.mxc_conv2d_bwd_data_prepared(*a, run._in(x), pw, None, prepared, run._ws(mxc.MXC_BWD_DATA_PREPARED))
    got = run._out(dx, (N, K, H, W))
    assert np.all(np.abs(got[:2] - ref) <= 2.0 ** -8 * np.abs(ref)), "dx"
    assert not got[2:].any()
    assert torch.equal(dx, prepared)
