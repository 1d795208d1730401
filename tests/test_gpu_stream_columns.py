"""The streaming kernel's column tiles of 96 (one staging pass of 64 columns and one of 32), whole and ragged, one to three of them, with bias,
ReLU and mask, from the filter as it lies and re-packed; and 1x1 layers that the library gives to it by itself.  Whole numbers: exact in any order."""
import pytest
import torch

from tests import util

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, pad: dx has C columns, forward K
DIMS = [(3, 72, 9, 7, 72, 1, 0), (2, 96, 11, 13, 96, 1, 0), (5, 192, 10, 9, 160, 1, 0), (1, 288, 5, 5, 264, 1, 0), (2, 24, 8, 9, 80, 3, 1), (90, 184, 17, 16, 136, 1, 0)]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


def check(mxc, dims, fwd=None, dx=None):
    """fwd, dx: whether the streaming kernel runs that pass (None: whichever); the other kernels are those of igemm.hip and wave.hip."""
    def by(streams):
        name = mxc.mxc_last_variant()
        assert "igemm_" in name and streams in (None, "igemm_stream" in name), name

    N, C, H, W, K, R, pad = dims
    run = util.Runner(mxc, (N, C, H, W, K, R, R, 1, pad), "bf16", "nhwc")
    a = (*run.dims, run.dt, run.lay)
    g = torch.Generator(device="cuda").manual_seed(N * C + H)

    def ints(*shape):      # one in eight is not zero: sums stay below 2^8, exact in bf16 too
        return torch.randint(-1, 2, shape, generator=g, device="cuda").float() * (torch.rand(shape, generator=g, device="cuda") < 0.125)

    x, w, dy, mask, bias = ints(N, H, W, C), ints(K, R, R, C), ints(N, H, W, K), ints(N, H, W, C), ints(K)
    pads = lambda t: torch.nn.functional.pad(t, (0, 0, pad, pad, pad, pad))  # noqa: E731
    y_want, dx_want = bias.expand(N, H, W, K).clone(), torch.zeros(N, H, W, C, device="cuda")
    for r in range(R):
        for s in range(R):
            y_want += (pads(x)[:, r:r + H, s:s + W].reshape(-1, C) @ w[:, r, s].T.contiguous()).view(N, H, W, K)
            dx_want += (pads(dy)[:, 2 * pad - r:2 * pad - r + H, 2 * pad - s:2 * pad - s + W].reshape(-1, K) @ w[:, r, s].contiguous()).view(N, H, W, C)
    assert float(y_want.abs().max()) <= 256 and float(dx_want.abs().max()) <= 256
    wants = [v.bfloat16() for v in (y_want.clamp(min=0), dx_want, torch.where(mask > 0, dx_want, torch.zeros_like(dx_want)), dx_want)]
    x, w, dy, mask = x.bfloat16(), w.bfloat16(), dy.bfloat16(), mask.bfloat16()
    y, plain, masked, prepared = (torch.full((want.numel() + 64,), 7.0, dtype=torch.bfloat16, device="cuda") for want in wants)
    mxc.mxc_conv2d_fwd_bias_act(*a, x, w, bias, 1, y, run._ws(mxc.MXC_FWD))
    by(fwd)
    mxc.mxc_conv2d_bwd_data(*a, dy, w, plain, run._ws(mxc.MXC_BWD_DATA))
    by(dx)
    mxc.mxc_conv2d_bwd_data_relu(*a, dy, w, mask, masked, run._ws(mxc.MXC_BWD_DATA_RELU))
    pw = run._ws(mxc.MXC_BWD_DATA_FILTER)
    mxc.mxc_conv2d_bwd_data_prepare_filter(*a, w, pw)
    mxc.mxc_conv2d_bwd_data_prepared(*a, dy, pw, None, prepared, run._ws(mxc.MXC_BWD_DATA_PREPARED))
    by(dx)
    for got, want in zip((y, plain, masked, prepared), wants):
        assert torch.equal(got[:-64], want.reshape(-1)) and bool((got[-64:] == 7.0).all())


@pytest.mark.parametrize("dims", DIMS)
def test_tiles_of_96_columns(mxc, monkeypatch, dims):
    monkeypatch.setenv("MXC_FORCE_VARIANT", "igemm_stream")
    check(mxc, dims, True, True)


def test_chosen(mxc):
    check(mxc, (211, 80, 57, 57, 224, 1, 0), True, True)


# rows of 480 and 416 bytes that two column tiles share, one stage, from 120 MB on (forward, dx); three stages against tiles of 256 columns
@pytest.mark.parametrize("dims,fwd,dx", [((140, 32, 66, 66, 240, 1, 0), False, None), ((140, 240, 66, 66, 24, 1, 0), None, False), ((130, 208, 79, 79, 48, 1, 0), None, False),
                                         ((168, 416, 37, 37, 192, 1, 0), None, False), ((183, 160, 39, 39, 416, 1, 0), False, None)])
def test_left_to_the_tiles(mxc, monkeypatch, dims, fwd, dx):
    """Layers that run 1.1 to 1.3 times as long on the streaming kernel."""
    monkeypatch.delenv("MXC_FORCE_VARIANT", raising=False)
    check(mxc, dims, fwd, dx)
