"""Forward and dx by the kernel whose taps of a filter row share their pixels: every tile at ragged last rows and columns, channel blocks that
are not whole, padded channels, images narrower than the filter, filters of other heights than widths, and the mask, bias and ReLU.  Whole numbers, so
results are exact in any order."""
import pytest
import torch
import torch.nn.functional as F

from tests import util

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, pad: Q = W where S = 2*pad + 1
DIMS = [(3, 40, 9, 7, 24, 3, 3, 1), (2, 8, 11, 13, 104, 5, 5, 2), (1, 16, 1, 1, 8, 3, 3, 1), (5, 72, 1, 2, 40, 5, 5, 2), (4, 32, 16, 24, 264, 3, 3, 1),
        (2, 24, 6, 37, 200, 1, 3, 1), (3, 48, 8, 5, 16, 5, 3, 1), (2, 64, 9, 12, 136, 3, 5, 2), (37, 96, 8, 8, 64, 3, 3, 1),
        # channels that are no multiple of 8, on copies padded with zeros: columns without a filter row, a bias or a result (NCHW both, NHWC the input's)
        (3, 30, 9, 11, 50, 3, 3, 1), (2, 13, 8, 13, 99, 5, 5, 2), (4, 250, 6, 7, 72, 3, 3, 1), (3, 72, 5, 9, 250, 3, 3, 1)]


def _tiles():
    from paper_1512_01274_amd import mxc as m
    return [n.removeprefix("igemm_run_") for n in m.mxc_tile_names(8)]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("tile,dims", [(t, d) for t in _tiles() for d in DIMS if not (t == "256x256" and d[6] == 5)])      # (the filter rows of five taps do not fit)
def test_forward_and_dx(mxc, monkeypatch, tile, dims, layout):
    N, C, H, W, K, R, S, pad = dims
    name = "igemm_run_" + tile
    runs = lambda columns: mxc.mxc_last_variant().endswith(name) or (layout == "nhwc" and columns % 8 != 0)  # noqa: E731  (results in place: whole 16 bytes)
    monkeypatch.setenv("MXC_FORCE_VARIANT", name)
    run = util.Runner(mxc, (N, C, H, W, K, R, S, 1, pad), "bf16", layout)
    a = (*run.dims, run.dt, run.lay)
    g = torch.Generator(device="cuda").manual_seed(N * C + H)

    def ints(*shape, most=1):      # sums of up to 72*25 products: most are zero, the rest stay below 2^8, exact in bf16 too
        v = torch.randint(-most, most + 1, shape, generator=g, device="cuda").double()
        return v * (torch.rand(shape, generator=g, device="cuda") < 0.25)

    x, w, dy, mask, bias = ints(N, C, H, W), ints(K, C, R, S), ints(N, K, run.P, run.Q), ints(N, C, H, W), ints(K, most=3)
    y_want = F.conv2d(x.cpu(), w.cpu(), bias.cpu(), padding=pad).clamp_(min=0).cuda()
    dx_want = F.conv_transpose2d(dy.cpu(), w.cpu(), padding=pad).cuda()
    assert dx_want.shape == x.shape and float(y_want.max()) <= 256 and float(dx_want.abs().max()) <= 256
    put = lambda t: (t if layout == "nchw" else t.permute(0, 2, 3, 1)).contiguous().bfloat16()  # noqa: E731
    x, w, dy, mask = put(x), put(w), put(dy), put(mask)
    wants = (put(y_want), put(dx_want), put(torch.where((mask if layout == "nchw" else mask.permute(0, 3, 1, 2)) > 0, dx_want, torch.zeros_like(dx_want))),
             put(dx_want))
    y, dx, masked, prepared = (torch.full((want.numel() + 64,), 7.0, dtype=torch.bfloat16, device="cuda") for want in wants)
    mxc.mxc_conv2d_fwd_bias_act(*a, x, w, bias.float(), 1, y, run._ws(mxc.MXC_FWD))
    assert runs(K), mxc.mxc_last_variant()
    mxc.mxc_conv2d_bwd_data(*a, dy, w, dx, run._ws(mxc.MXC_BWD_DATA))
    assert runs(C), mxc.mxc_last_variant()
    mxc.mxc_conv2d_bwd_data_relu(*a, dy, w, mask, masked, run._ws(mxc.MXC_BWD_DATA_RELU))
    pw = run._ws(mxc.MXC_BWD_DATA_FILTER)
    mxc.mxc_conv2d_bwd_data_prepare_filter(*a, w, pw)
    mxc.mxc_conv2d_bwd_data_prepared(*a, dy, pw, None, prepared, run._ws(mxc.MXC_BWD_DATA_PREPARED))
    for got, want in zip((y, dx, masked, prepared), wants):
        assert torch.equal(got[:-64], want.reshape(-1)) and bool((got[-64:] == 7.0).all())


def test_chosen(mxc):
    """A layer far from the line between the kernels gets it, in every call that has to give the same bits."""
    dims = (64, 64, 28, 28, 96, 5, 5, 1, 2)
    run = util.Runner(mxc, dims, "bf16", "nhwc")
    a = (*run.dims, run.dt, run.lay)
    g = torch.Generator(device="cuda").manual_seed(1)
    dy = torch.randn(64, 28, 28, 96, generator=g, device="cuda").bfloat16()
    w = torch.randn(96, 5, 5, 64, generator=g, device="cuda").bfloat16()
    dx, again = (torch.empty(64, 28, 28, 64, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    mxc.mxc_conv2d_bwd_data(*a, dy, w, dx, run._ws(mxc.MXC_BWD_DATA))
    assert "igemm_run_" in mxc.mxc_last_variant()
    pw = run._ws(mxc.MXC_BWD_DATA_FILTER)
    mxc.mxc_conv2d_bwd_data_prepare_filter(*a, w, pw)
    mxc.mxc_conv2d_bwd_data_prepared(*a, dy, pw, None, again, run._ws(mxc.MXC_BWD_DATA_PREPARED))
    assert torch.equal(dx, again)
    ref = F.conv_transpose2d(dy.cpu().permute(0, 3, 1, 2).float(), w.cpu().permute(0, 3, 1, 2).float(), padding=2).permute(0, 2, 3, 1)
    assert float((dx.cpu().float() - ref).norm() / ref.norm()) < 2.0 ** -8      # the rounding of the result
