"""The split reduction of backward-weight where dw's order differs from the filter matrix's or many splits meet a small
dw: first layers' packings, padded channels and KCRS results, at split counts on both sides of the kernel's two widths."""
import numpy as np
import pytest
import torch

from paper_1512_01274_amd import inputs as gen
from tests import util

pytestmark = pytest.mark.gpu

SHAPES = [
    (4, 3, 67, 67, 24, 11, 11, 4, 2),     # space-to-depth columns, taps past the filter dropped
    (4, 3, 40, 33, 16, 3, 3, 1, 1),       # rows of four channels per pixel, one of them padding
    (3, 1, 45, 45, 8, 7, 7, 2, 3),
    (6, 30, 30, 31, 50, 3, 3, 1, 1),      # padded channels on both sides
    (6, 16, 33, 40, 24, 3, 3, 1, 1),      # same order in NHWC
]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("splits", [1, 2, 31, 32, 70])
@pytest.mark.parametrize("dims", SHAPES)
def test_dw_of_any_split_count(mxc, oracle, monkeypatch, dims, splits, layout):
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="bf16", dist="normal")
    run = util.Runner(mxc, dims, "bf16", layout)
    monkeypatch.setenv("MXC_FORCE_WGRAD", f"wgrad_64x64_p64s2_w4/{splits}")
    got = run.bwd_weight(x, dy)
    assert "wgrad_64x64" in mxc.mxc_last_variant()
    ref = oracle.conv2d_bwd_weight(x, dy, w.shape, st, pad)
    den = oracle.conv2d_bwd_weight(np.abs(x), np.abs(dy), w.shape, st, pad)
    assert np.all(np.abs(got - ref) <= util.tight_bound(ref, den, "bf16", False)), dims
