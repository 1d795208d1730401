"""fp32 on the matrix cores: every tile shape of the fp32 kernel, both layouts, all three passes, against the oracle on
the shapes its address arithmetic distinguishes (channel counts with and without aligned fours, ragged row and column
tiles, strides with several and with unreached residue classes, padding beyond the filter, several pixel ranges)."""
import os

import numpy as np
import pytest
import torch

from paper_1512_01274_amd import inputs as gen
from tests import util

pytestmark = pytest.mark.gpu

SHAPES = [
    (2, 16, 16, 16, 32, 3, 3, 1, 1),
    (1, 5, 13, 9, 7, 5, 3, 1, 2),         # nothing is a multiple of 4, R != S
    (3, 36, 11, 10, 132, 3, 3, 2, 1),     # four residue classes, columns past one 128-wide tile
    (2, 20, 9, 9, 33, 1, 1, 2, 0),        # three classes no tap reaches
    (1, 3, 30, 31, 70, 11, 11, 4, 2),     # 121 taps, sixteen classes
    (5, 130, 7, 6, 40, 1, 1, 1, 1),       # padding beyond the filter
]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


def _tiles():
    from paper_1512_01274_amd import mxc as m
    return m.mxc_tile_names(3)


@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("dims", SHAPES)
@pytest.mark.parametrize("tile", _tiles())
def test_every_fp32_tile(mxc, oracle, monkeypatch, tile, dims, layout):
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="f32", dist="normal")
    run = util.Runner(mxc, dims, "f32", layout)
    bias = np.linspace(-1.0, 1.0, K).astype(np.float32)
    monkeypatch.setenv("MXC_FORCE_VARIANT", tile)

    def check(name, got, ref, den):
        assert mxc.mxc_last_variant() == f"{name}:{tile}"
        assert util.metric(got, ref, den) <= util.TOL["f32"], (name, dims)
        assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "f32", False)), (name, dims)

    y = torch.full((N * K * run.P * run.Q,), float("nan"), device="cuda")
    mxc.mxc_conv2d_fwd_bias_act(*dims, run.dt, run.lay, run._in(x), run._in(w), torch.from_numpy(bias).cuda(), 1, y, run._ws(mxc.MXC_FWD))
    ref, den = oracle.conv2d_fwd_bias_act(x, w, bias, True, st, pad)
    check("fwd", run._out(y, (N, K, run.P, run.Q)), ref, den)

    dx = torch.full((N * C * H * W,), float("nan"), device="cuda")
    mxc.mxc_conv2d_bwd_data_relu(*dims, run.dt, run.lay, run._in(dy), run._in(w), run._in(x), dx, run._ws(mxc.MXC_BWD_DATA_RELU))
    ref, den = oracle.conv2d_bwd_data_relu(dy, w, x, st, pad)
    check("bwd_data", run._out(dx, (N, C, H, W)), ref, den)

    ref = oracle.conv2d_bwd_weight(x, dy, w.shape, st, pad)
    den = oracle.conv2d_bwd_weight(np.abs(x), np.abs(dy), w.shape, st, pad)
    for splits in (1, 3):
        monkeypatch.setenv("MXC_FORCE_WGRAD", f"{tile}/{splits}")
        check("bwd_weight", run.bwd_weight(x, dy), ref, den)
