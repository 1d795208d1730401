"""Infinities and NaN in one operand where the other one has padding: a tap outside the image is left out of the sum, so
that a border result which does not use a non-finite value stays what it is.  Every fp32 tile in the three passes, and the
gradients of bf16 layers of ragged K, both layouts, against the oracle (which walks the taps inside): NaN and infinities at
the same places with the same signs, finite results within the usual bound."""
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
    (1, 3, 30, 31, 70, 11, 11, 4, 2),     # 121 taps, sixteen classes
    (5, 130, 7, 6, 40, 1, 1, 1, 1),       # border results without a single tap
    (2, 24, 9, 8, 20, 2, 3, 1, 0),        # no padding: the input gradient has taps outside dy all the same
]


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


def _tiles():
    from paper_1512_01274_amd import mxc as m
    return m.mxc_tile_names(3)


def plant(a, seed):
    """a with an infinity of each sign and a NaN: one at the first element, one at the last, one in between"""
    b = a.copy()
    rng = np.random.Generator(np.random.Philox(key=seed))
    at = [0, b.size - 1, int(rng.integers(0, b.size))]
    for i, v in zip(at, rng.permutation([np.inf, -np.inf, np.nan])):
        b.flat[i] = v
    return b


def finite_abs(a):
    return np.abs(np.where(np.isfinite(a), a, 0)).astype(np.float32)


def check(got, ref, den, dtype, rounded, what):
    assert np.array_equal(np.isnan(got), np.isnan(ref)), (what, int(np.isnan(got).sum()), int(np.isnan(ref).sum()))
    inf = np.isinf(ref)
    assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], ref[inf]), what
    ok = np.isfinite(ref)
    assert np.all(np.abs(got[ok] - ref[ok]) <= util.tight_bound(ref[ok], den[ok], dtype, rounded)), what


@pytest.mark.filterwarnings("ignore:invalid value")
@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("dims", SHAPES)
@pytest.mark.parametrize("tile", _tiles())
def test_fp32(mxc, oracle, monkeypatch, tile, dims, layout):
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="f32", dist="normal")
    w_bad, dy_bad = plant(w, 1), plant(dy, 2)
    run = util.Runner(mxc, dims, "f32", layout)
    monkeypatch.setenv("MXC_FORCE_VARIANT", tile)
    check(run.fwd(x, w_bad), oracle.conv2d_fwd(x, w_bad, st, pad), oracle.conv2d_fwd(np.abs(x), finite_abs(w_bad), st, pad), "f32", False,
          ("fwd", dims))
    dx = torch.full((N * C * H * W,), float("nan"), device="cuda")
    mxc.mxc_conv2d_bwd_data_relu(*dims, run.dt, run.lay, run._in(dy), run._in(w_bad), run._in(x), dx, run._ws(mxc.MXC_BWD_DATA_RELU))
    ref = np.where(x > 0, oracle.conv2d_bwd_data(dy, w_bad, x.shape, st, pad), 0.0)
    check(run._out(dx, x.shape), ref, oracle.conv2d_bwd_data(np.abs(dy), finite_abs(w_bad), x.shape, st, pad), "f32", False, ("bwd_data", dims))
    ref = oracle.conv2d_bwd_weight(x, dy_bad, w.shape, st, pad)
    den = oracle.conv2d_bwd_weight(np.abs(x), finite_abs(dy_bad), w.shape, st, pad)
    for splits in (1, 3):
        monkeypatch.setenv("MXC_FORCE_WGRAD", f"{tile}/{splits}")
        check(run.bwd_weight(x, dy_bad), ref, den, "f32", False, ("bwd_weight", dims, splits))


# fp32 layers of whole 16-byte chunks of channels, of which the wave kernels store results straight to NHWC or to planes and sum what
# is NaN once more over the taps inside: unequal sides, residue classes of dx (some without a tap, planes of broken groups of four
# pixels), no padding, several pixel ranges of dw
CHUNKS = [
    (2, 16, 16, 16, 32, 3, 3, 1, 1),
    (2, 20, 13, 9, 12, 5, 3, 1, 2),
    (3, 36, 21, 18, 24, 3, 3, 2, 1),
    (5, 132, 7, 6, 40, 1, 1, 1, 1),       # border results without a single tap
    (4, 8, 9, 10, 16, 1, 1, 2, 0),        # three of four classes of dx without a tap
    (2, 24, 9, 8, 20, 2, 3, 1, 0),
    (40, 8, 12, 9, 12, 3, 3, 2, 1),       # pixels enough for several ranges in dw, here and below
    (24, 12, 20, 21, 20, 3, 3, 1, 1),
]


@pytest.mark.filterwarnings("ignore:invalid value")
@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("dims", CHUNKS)
def test_fp32_wave(mxc, oracle, monkeypatch, dims, layout):
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="f32", dist="normal")
    w_bad, dy_bad = plant(w, 5), plant(dy, 6)
    run = util.Runner(mxc, dims, "f32", layout)
    fwd = oracle.conv2d_fwd(x, w_bad, st, pad), oracle.conv2d_fwd(np.abs(x), finite_abs(w_bad), st, pad)
    dx = [(f, g, np.where(x > 0, oracle.conv2d_bwd_data(g, f, x.shape, st, pad), 0.0), oracle.conv2d_bwd_data(finite_abs(g), finite_abs(f), x.shape, st, pad))
          for f, g in ((w_bad, dy), (w, dy_bad))]
    names = mxc.mxc_tile_names(6)
    for name in (n for n in names if "_dw_" not in n):
        monkeypatch.setenv("MXC_FORCE_VARIANT", name)
        check(run.fwd(x, w_bad), *fwd, "f32", False, ("fwd", name, dims))
        assert mxc.mxc_last_variant().endswith(name)
        for f, g, ref, den in dx:
            got = torch.full((N * C * H * W,), 7.0, device="cuda")
            mxc.mxc_conv2d_bwd_data_relu(*dims, run.dt, run.lay, run._in(g), run._in(f), run._in(x), got, run._ws(mxc.MXC_BWD_DATA_RELU))
            assert mxc.mxc_last_variant().endswith(name)
            check(run._out(got, x.shape), ref, den, "f32", False, ("bwd_data", name, dims))
    if layout == "nchw":                  # dw of planes has no wave kernel
        return
    ref, den = oracle.conv2d_bwd_weight(x, dy_bad, w.shape, st, pad), oracle.conv2d_bwd_weight(np.abs(x), finite_abs(dy_bad), w.shape, st, pad)
    for name in (n for n in names if "_dw_" in n):
        for ranges in (1, 3) if dims in CHUNKS[-2:] else (1,):
            monkeypatch.setenv("MXC_FORCE_WGRAD", f"{name}/{ranges}")
            assert mxc.mxc_conv2d_workspace_bytes(mxc.MXC_BWD_WEIGHT, *dims, run.dt, run.lay) >= ranges * 4 * w.size or ranges == 1
            check(run.bwd_weight(x, dy_bad), ref, den, "f32", False, ("bwd_weight", name, dims, ranges))
            assert mxc.mxc_last_variant().endswith(name)


# bf16 layers of ragged K: general, several classes, strided and unstrided first layers (their packings have empty places
# in the filter, too), channels of both tensors ragged, no padding
RAGGED = [
    (2, 30, 13, 11, 50, 3, 3, 2, 1),
    (3, 16, 9, 9, 70, 5, 5, 1, 2),
    (1, 3, 20, 18, 13, 3, 3, 1, 1),
    (2, 3, 35, 35, 9, 11, 11, 4, 2),
    (2, 2, 17, 16, 130, 2, 2, 2, 0),
    (4, 40, 10, 7, 100, 3, 3, 1, 0),
    (2, 100, 6, 6, 66, 1, 1, 2, 1),
    (1, 8, 290, 301, 9, 3, 3, 1, 1),      # more pixels than one lane adds up
]


@pytest.mark.filterwarnings("ignore:invalid value")
@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("dims", RAGGED)
def test_bf16_ragged_k_gradients(mxc, oracle, dims, layout):
    N, C, H, W, K, R, S, st, pad = dims
    x, w, dy = gen.random_case(hash(dims) & 0xFFFF, *dims, dtype="bf16", dist="normal")
    w_bad, dy_bad = plant(w, 3), plant(dy, 4)
    run = util.Runner(mxc, dims, "bf16", layout)
    a = (*dims, run.dt, run.lay)
    prepared = mxc.alloc_workspace(mxc.mxc_conv2d_workspace_bytes(mxc.MXC_BWD_DATA_FILTER, *a))
    for f, g in ((w_bad, dy), (w, dy_bad)):
        ref, den = oracle.conv2d_bwd_data(g, f, x.shape, st, pad), oracle.conv2d_bwd_data(finite_abs(g), finite_abs(f), x.shape, st, pad)
        check(run.bwd_data(g, f), ref, den, "bf16", True, ("bwd_data", dims))
        mxc.mxc_conv2d_bwd_data_prepare_filter(*a, run._in(f), prepared)
        dx = torch.full((N * C * H * W,), 7.0, dtype=torch.bfloat16, device="cuda")
        mxc.mxc_conv2d_bwd_data_prepared(*a, run._in(g), prepared, run._in(x), dx, run._ws(mxc.MXC_BWD_DATA_PREPARED_RELU))
        check(run._out(dx, x.shape), np.where(x > 0, ref, 0.0), den, "bf16", True, ("bwd_data prepared, masked", dims))
    ref = oracle.conv2d_bwd_weight(x, dy_bad, w.shape, st, pad)
    den = oracle.conv2d_bwd_weight(np.abs(x), finite_abs(dy_bad), w.shape, st, pad)
    check(run.bwd_weight(x, dy_bad), ref, den, "bf16", False, ("bwd_weight", dims))
    dw = torch.full((w.size,), 7.0, dtype=torch.bfloat16, device="cuda")
    mxc.mxc_conv2d_bwd_weight_bf16(*a, run._in(x), run._in(dy_bad), dw, run._ws(mxc.MXC_BWD_WEIGHT_BF16))
    got = util.to_host_f64(dw)
    got = util.nhwc_to_nchw(got.reshape(K, R, S, C)) if layout == "nhwc" else got.reshape(w.shape)
    check(got, ref, den, "bf16", True, ("bwd_weight_bf16", dims))
