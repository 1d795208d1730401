"""Backward-data through a ReLU mask in the epilogues of the streaming and the window kernel, and every tile shape on
strided problems (all residue classes in one launch): ragged rows and columns, several column tiles, the general store
path, classes no tap reaches."""
import numpy as np
import pytest
import torch

from paper_1512_01274_amd import inputs as gen
from tests import util

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


def _tiles():
    from paper_1512_01274_amd import mxc as m
    return m.mxc_tile_names(0)


def _check(mxc, oracle, dims, seed, expect):
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = gen.random_case((hash(dims) + seed) & 0xFFFF, *dims, dtype="bf16", dist="normal")
    run = util.Runner(mxc, dims, "bf16", "nhwc")
    dx = torch.full((N * C * H * W,), float("nan"), dtype=torch.bfloat16, device="cuda")
    mxc.mxc_conv2d_bwd_data_relu(*dims, run.dt, run.lay, run._in(dy), run._in(w), run._in(x), dx, run._ws(mxc.MXC_BWD_DATA_RELU))
    assert mxc.mxc_last_variant().split(":")[-1].split("_inplace")[0] == expect, mxc.mxc_last_variant()
    ref, den = oracle.conv2d_bwd_data_relu(dy, w, x, st, pad)
    got = run._out(dx, (N, C, H, W))
    assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "bf16", True)), dims
    assert np.all(got[x <= 0] == 0)


@pytest.mark.parametrize("dims", [(3, 64, 20, 22, 64, 3, 3, 1, 1), (2, 136, 9, 35, 16, 3, 3, 1, 1), (1, 24, 5, 5, 48, 5, 3, 1, 2), (70, 32, 4, 33, 32, 3, 3, 1, 0)])
def test_masked_window(mxc, oracle, monkeypatch, dims):
    monkeypatch.setenv("MXC_FORCE_VARIANT", "igemm_patch_masked")
    _check(mxc, oracle, dims, 1, "igemm_patch_masked")


@pytest.mark.parametrize("dims", [(3, 64, 19, 17, 64, 1, 1, 1, 0), (2, 200, 13, 15, 24, 1, 1, 1, 0), (5, 32, 9, 9, 128, 1, 1, 1, 0), (2, 40, 12, 11, 40, 1, 1, 2, 0)])
def test_masked_stream(mxc, oracle, monkeypatch, dims):
    monkeypatch.setenv("MXC_FORCE_VARIANT", "igemm_stream")
    _check(mxc, oracle, dims, 2, "igemm_stream")


@pytest.mark.parametrize("dims", [(2, 72, 17, 19, 64, 3, 3, 2, 1), (3, 24, 13, 14, 40, 1, 1, 2, 0), (1, 20, 22, 15, 16, 5, 3, 3, 1), (1, 264, 9, 8, 72, 2, 2, 4, 0)])
@pytest.mark.parametrize("tile", _tiles())
def test_strided_classes(mxc, oracle, monkeypatch, tile, dims):
    monkeypatch.setenv("MXC_FORCE_VARIANT", tile)
    _check(mxc, oracle, dims, 3, tile)


# filters read in place as transposed tiles: taps with channels that fill stages or straddle them, column remainders, a
# reduction shorter than one stage, split and whole reductions
@pytest.mark.parametrize("dims", [(2, 72, 9, 11, 64, 3, 3, 1, 1), (1, 136, 7, 9, 24, 5, 3, 1, 2), (2, 8, 13, 12, 8, 1, 1, 1, 0), (1, 264, 8, 9, 192, 3, 3, 1, 0)])
@pytest.mark.parametrize("splits", ["/1", "/2"])
@pytest.mark.parametrize("tile", ["igemm_128x128_k64s2_w4", "igemm_256x256_k64s2_w8", "igemm_128x64_k64s2_w4", "igemm_128x32_k64s2_w4", "igemm_64x128_k64s3_w4"])
def test_in_place_filter(mxc, oracle, monkeypatch, tile, splits, dims):
    monkeypatch.setenv("MXC_FORCE_VARIANT", tile + splits)
    _check(mxc, oracle, dims, 4, tile)


# the streaming kernel transposes the filter on its way into LDS: one and several taps, reductions that end inside a stage,
# one and two column tiles with remainders, channels of dy that are padding
@pytest.mark.parametrize("dims", [(3, 64, 19, 17, 192, 1, 1, 1, 0), (2, 8, 13, 15, 8, 1, 1, 1, 0), (1, 136, 9, 8, 72, 1, 1, 1, 0), (2, 24, 12, 11, 24, 3, 3, 1, 1),
                                  (2, 40, 10, 9, 20, 3, 2, 1, 1)])
def test_stream_filter_in_place(mxc, oracle, monkeypatch, dims):
    monkeypatch.setenv("MXC_FORCE_VARIANT", "igemm_stream")
    _check(mxc, oracle, dims, 5, "igemm_stream")
