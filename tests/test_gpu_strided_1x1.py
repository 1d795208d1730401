"""dx of 1x1 filters at stride 2 by the tiles that write the zeros no tap reaches with their results: odd image sides, ragged last tiles and
columns, padding, the filter as it lies and re-packed, the mask, both layouts.  Whole numbers, so results are exact in any order."""
import pytest
import torch

from tests import util

pytestmark = pytest.mark.gpu

TILES = ["igemm_128x128_k64s2_w4", "igemm_256x256_k64s2_w8", "igemm_128x64_k64s2_w4", "igemm_128x32_k64s2_w4", "igemm_64x128_k64s3_w4",
         "igemm_256x256_k64s2_w8+igemm_128x64_k64s2_w4", "igemm_192x128_k64s3_w8"]     # two launches; a tile that leaves the zeros to a launch of their own
# N, C, H, W, K, pad
DIMS = [(3, 40, 9, 7, 24, 0), (2, 136, 8, 11, 72, 0), (1, 8, 1, 1, 8, 0), (5, 64, 1, 10, 64, 0), (2, 48, 13, 6, 32, 2), (40, 264, 30, 41, 40, 0)]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("tile", TILES)
def test_dx(mxc, monkeypatch, tile, dims, layout):
    monkeypatch.setenv("MXC_FORCE_VARIANT", tile)
    N, C, H, W, K, pad = dims
    run = util.Runner(mxc, (N, C, H, W, K, 1, 1, 2, pad), "bf16", layout)
    a = (*run.dims, run.dt, run.lay)
    g = torch.Generator(device="cuda").manual_seed(N * C + H)
    ints = lambda *shape: torch.randint(-2, 3, shape, generator=g, device="cuda").float()  # noqa: E731  (sums below 2^9: exact in bf16 too)
    dy, w, mask = ints(N, run.P, run.Q, K), ints(K, C), ints(N, H, W, C)
    mask[:, 1::2] = float("nan")           # of pixels no tap reaches: zeros all the same
    grid = torch.zeros(N, H + 2 * pad, W + 2 * pad, C, device="cuda")
    grid[:, :2 * run.P:2, :2 * run.Q:2] = (dy.reshape(-1, K) @ w).view(N, run.P, run.Q, C)
    want = grid[:, pad:pad + H, pad:pad + W]
    put = lambda t: (t if layout == "nhwc" else t.permute(0, 3, 1, 2)).contiguous().bfloat16()  # noqa: E731
    dy, w, mask, wants = put(dy), w.bfloat16(), put(mask), (put(want), put(torch.where(mask > 0, want, torch.zeros_like(want))))
    dx, masked, prepared = (torch.full((N * C * H * W + 64,), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(3))
    mxc.mxc_conv2d_bwd_data(*a, dy, w, dx, run._ws(mxc.MXC_BWD_DATA))
    mxc.mxc_conv2d_bwd_data_relu(*a, dy, w, mask, masked, run._ws(mxc.MXC_BWD_DATA_RELU))
    assert tile.split("+")[0] in mxc.mxc_last_variant()
    pw = run._ws(mxc.MXC_BWD_DATA_FILTER)
    mxc.mxc_conv2d_bwd_data_prepare_filter(*a, w, pw)
    mxc.mxc_conv2d_bwd_data_prepared(*a, dy, pw, None, prepared, run._ws(mxc.MXC_BWD_DATA_PREPARED))
    for got, expect in ((dx, wants[0]), (masked, wants[1]), (prepared, wants[0])):
        assert torch.equal(got[:-64], expect.reshape(-1)) and bool((got[-64:] == 7.0).all())
