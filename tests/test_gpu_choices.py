"""Which kernel a layer gets by itself, and what it computes on either side of each line between two: layers that grow from one image to
many, of which the first image holds small whole numbers (exact in bf16 and in sums of any order) and the others zeros, so that the
first image's results and the weight gradient stay the same bits whichever kernel ran."""
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


# dtype, layout, (C, H, W, K, R, S, stride, pad), batches, and for forward, dx and dw what the names of some batches' kernels hold and
# those of others do not ("": all do)
CHOICES = [
    ("bf16", "nhwc", (64, 28, 28, 72, 3, 3, 1, 1), (1, 4, 12, 24, 48, 96, 192, 320), ("igemm_wave", "igemm_wave", "wgrad_wave")),
    ("bf16", "nchw", (64, 28, 28, 72, 3, 3, 1, 1), (1, 4, 12, 24, 48, 96, 192, 320), ("igemm_wave", "igemm_wave", "wgrad_wave")),
    ("bf16", "nhwc", (128, 20, 22, 128, 3, 3, 2, 1), (1, 4, 12, 24, 48, 96, 192, 384), ("igemm_wave", "igemm_wave", "")),
    ("bf16", "nhwc", (3, 91, 91, 40, 5, 5, 1, 2), (1, 4, 16, 64, 131), ("igemm_wave", "taps_dx", "wgrad_wave")),
    ("f32", "nhwc", (32, 20, 22, 48, 3, 3, 1, 1), (1, 4, 12, 24, 48, 96, 192), ("f32_wave", "", "")),
    ("f32", "nhwc", (32, 20, 22, 48, 3, 3, 2, 1), (1, 4, 12, 24, 48, 96, 192), ("f32_wave", "f32_wave", "")),
    ("f32", "nhwc", (192, 13, 13, 384, 3, 3, 1, 1), (1, 48, 192), ("f32_wave", "f32_wave", "f32_wave")),
    ("f32", "nchw", (16, 16, 16, 32, 3, 3, 1, 1), (1, 4, 12, 24, 48, 96, 192), ("f32_wave", "f32_wave", "")),
]


def _walk(mxc, oracle, dtype, layout, shape, batches):
    """The kernels' names, batch by batch, in each pass; every result compared with the oracle's of the first image."""
    C, H, W, K, R, S, st, pad = shape
    P, Q = (H + 2 * pad - R) // st + 1, (W + 2 * pad - S) // st + 1
    rng = np.random.default_rng(C * K + st)
    x, w, dy = (rng.integers(-2, 3, d).astype(np.float32) for d in ((1, C, H, W), (K, C, R, S), (1, K, P, Q)))
    mask = rng.integers(0, 2, x.shape).astype(np.float32)
    want = oracle.conv2d_fwd(x, w, st, pad), oracle.conv2d_bwd_data(dy, w, x.shape, st, pad) * mask, oracle.conv2d_bwd_weight(x, dy, w.shape, st, pad)
    rounded = [torch.from_numpy(a).to(torch.bfloat16 if dtype == "bf16" and n < 2 else torch.float32).double().numpy() for n, a in enumerate(want)]
    names = ([], [], [])
    for n in batches:
        dims = (n, *shape)
        run = util.Runner(mxc, dims, dtype, layout)
        a = (*dims, run.dt, run.lay)

        def grown(first):
            t = torch.zeros(n, first.size, dtype=run.tdtype, device="cuda")
            t[0] = run._in(first).reshape(-1)
            return t

        out = [torch.full((size,), 7.0, dtype=t, device="cuda") for size, t in ((n * K * P * Q, run.tdtype), (n * x.size, run.tdtype), (w.size, torch.float32))]
        mxc.mxc_conv2d_fwd(*a, grown(x), run._in(w), out[0], run._ws(mxc.MXC_FWD))
        names[0].append(mxc.mxc_last_variant())
        mxc.mxc_conv2d_bwd_data_relu(*a, grown(dy), run._in(w), grown(mask), out[1], run._ws(mxc.MXC_BWD_DATA_RELU))
        names[1].append(mxc.mxc_last_variant())
        mxc.mxc_conv2d_bwd_weight(*a, grown(x), grown(dy), out[2], run._ws(mxc.MXC_BWD_WEIGHT))
        names[2].append(mxc.mxc_last_variant())
        for i, shape_i in enumerate(((1, K, P, Q), x.shape)):
            t = out[i].view(n, -1)
            assert np.array_equal(run._out(t[0], shape_i), rounded[i]), (n, names[i][-1])
            assert not bool(t[1:].any()), (n, names[i][-1])
        got = out[2].double().cpu().numpy()
        got = got.reshape(K, R, S, C).transpose(0, 3, 1, 2) if layout == "nhwc" else got.reshape(w.shape)
        assert np.array_equal(got, rounded[2]), (n, names[2][-1])
    return names


@pytest.mark.parametrize("dtype,layout,shape,batches,kernels", CHOICES)
def test_either_side_of_a_choice(mxc, oracle, monkeypatch, dtype, layout, shape, batches, kernels):
    monkeypatch.delenv("MXC_FORCE_VARIANT", raising=False)
    monkeypatch.delenv("MXC_FORCE_WGRAD", raising=False)
    names = _walk(mxc, oracle, dtype, layout, shape, batches)
    for got, kernel in zip(names, kernels):
        print(got)
        held = {kernel in name for name in got}
        assert held == ({True, False} if kernel else {True}), got


# Layers that the kernels sharing pixels among the taps of a filter row run 1.06 to 1.2 times as long as the kernel they leave it to: (N, C, H, W, K, R), the
# pass (0 forward, 1 dx with a mask, 2 dw).  Wave kernels of a few us and split reductions; dw in blocks of 128x32, and against tiles of 256x256.
LEFT = [((28, 32, 16, 15, 96, 3), 0), ((13, 512, 8, 14, 32, 3), 1), ((163, 384, 8, 8, 64, 5), 0), ((2, 480, 24, 24, 352, 5), 1),
        ((23, 16, 52, 52, 512, 3), 2), ((10, 80, 63, 63, 352, 3), 2), ((147, 80, 15, 15, 480, 3), 2), ((54, 352, 41, 10, 240, 5), 2)]


@pytest.mark.parametrize("dims,which", LEFT)
def test_left_by_the_run_kernels(mxc, oracle, monkeypatch, dims, which):
    monkeypatch.delenv("MXC_FORCE_VARIANT", raising=False)
    monkeypatch.delenv("MXC_FORCE_WGRAD", raising=False)
    N, C, H, W, K, R = dims
    name, = _walk(mxc, oracle, "bf16", "nhwc", (C, H, W, K, R, R, 1, R // 2), (N,))[which]
    assert "_run_" not in name, name


# 1x1 at stride 2, of whose dx three pixels in four are zeros: N, C, H, W, K and whether the wave kernel runs it (5x24x24 4.1 us where the
# other path takes 11.7; the last four with a mask 26.6, 67.7, 47.8 and 65.9 where the other path takes 15.7, 37.5, 30.1 and 50.5)
STRIDED_1X1 = [(1, 64, 14, 14, 128, True), (5, 32, 24, 24, 480, True), (8, 128, 28, 28, 256, True), (63, 216, 29, 29, 176, False), (146, 192, 42, 42, 176, False),
               (181, 64, 56, 56, 160, False), (170, 192, 48, 48, 24, False)]


def _dx_1x1(mxc, N, C, H, W, K, relu):
    """The kernel's name; results are zeros where no tap reaches whatever the mask holds there, and elsewhere the product of whole numbers."""
    run = util.Runner(mxc, (N, C, H, W, K, 1, 1, 2, 0), "bf16", "nhwc")
    g = torch.Generator(device="cuda").manual_seed(C * K + H)
    ints = lambda *shape: torch.randint(-2, 3, shape, generator=g, device="cuda").float()  # noqa: E731  (sums below 2^11: exact in fp32)
    dy, w, mask = ints(N, run.P, run.Q, K), ints(K, C), ints(N, H, W, C)
    want = torch.zeros(N, H, W, C, device="cuda")
    want[:, ::2, ::2] = (dy.reshape(-1, K) @ w).view(N, run.P, run.Q, C)
    if relu:
        mask[:, 1::2] = float("nan")
        want = torch.where(mask > 0, want, torch.zeros_like(want))
    a = (N, C, H, W, K, 1, 1, 2, 0, run.dt, run.lay)
    dx = torch.full((N, H, W, C), 7.0, dtype=torch.bfloat16, device="cuda")
    dy, w, mask = dy.bfloat16(), w.bfloat16(), mask.bfloat16()
    if relu:
        mxc.mxc_conv2d_bwd_data_relu(*a, dy, w, mask, dx, run._ws(mxc.MXC_BWD_DATA_RELU))
    else:
        mxc.mxc_conv2d_bwd_data(*a, dy, w, dx, run._ws(mxc.MXC_BWD_DATA))
    assert torch.equal(dx, want.bfloat16())
    return mxc.mxc_last_variant()


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("N,C,H,W,K,wave", STRIDED_1X1)
def test_strided_1x1(mxc, monkeypatch, N, C, H, W, K, wave, relu):
    monkeypatch.delenv("MXC_FORCE_VARIANT", raising=False)
    name = _dx_1x1(mxc, N, C, H, W, K, relu)
    assert ("wave" in name) == wave, name


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("N,C,H,W,K", [(12, 96, 16, 16, 448), (37, 24, 16, 16, 512), (6, 208, 14, 14, 416), (88, 24, 10, 10, 448)])
def test_strided_1x1_in_one_round(mxc, monkeypatch, N, C, H, W, K, relu):
    """Some 290 tiles of 32x32, those of zeros among them, are a second round of the 256 CUs: 7.1 us where half as many of 64x32 take 5.1."""
    monkeypatch.delenv("MXC_FORCE_VARIANT", raising=False)
    name = _dx_1x1(mxc, N, C, H, W, K, relu)
    assert "igemm_wave_" in name and "32x32" not in name, name
