"""Layers in turn, as a network runs them: what a thread keeps of one layer's plans must not show in another's results."""
import numpy as np
import pytest
import torch

from oracle import conv_oracle
from tests import util

pytestmark = pytest.mark.gpu

# alike but for channels that differ by multiples of 64, stride, filter or batch
LAYERS = [(2, 64, 14, 14, 64, 1, 1, 1, 0), (2, 128, 14, 14, 64, 1, 1, 1, 0), (2, 64, 14, 14, 128, 1, 1, 1, 0), (2, 192, 14, 14, 64, 1, 1, 1, 0),
          (2, 64, 14, 14, 64, 3, 3, 1, 1), (2, 128, 14, 14, 64, 3, 3, 2, 1), (4, 64, 14, 14, 64, 3, 3, 2, 1), (2, 64, 14, 14, 64, 3, 3, 2, 1)]


@pytest.fixture(scope="module")
def mxc():
    from paper_1512_01274_amd import mxc as m
    return m


@pytest.mark.parametrize("dtype,layout", [("bf16", "nhwc"), ("bf16", "nchw"), ("f32", "nhwc"), ("f32", "nchw")])
def test_layers_in_turn(mxc, dtype, layout):
    rng = np.random.Generator(np.random.Philox(key=11))
    jobs = []
    for dims in LAYERS:
        N, C, H, W, K, R, S, st, pad = dims
        P = (H + 2 * pad - R) // st + 1
        draw = lambda *shape: (rng.integers(-8, 9, shape) / 8.0).astype(np.float32)  # noqa: E731  (exact in bf16)
        jobs.append((util.Runner(mxc, dims, dtype, layout), draw(N, C, H, W), draw(K, C, R, S), draw(N, K, P, P), st, pad))
    first = {}
    for turn in range(3):
        for n, (run, x, w, dy, st, pad) in enumerate(jobs):
            got = [run.fwd(x, w, True), run.bwd_data(dy, w, True), run.bwd_weight(x, dy, True)]
            if turn > 0:
                assert all(torch.equal(a, b) for a, b in zip(got, first[n])), (turn, LAYERS[n])
                continue
            first[n] = got
            for name, fn, args in [("fwd", conv_oracle.conv2d_fwd, (x, w)), ("bwd_data", conv_oracle.conv2d_bwd_data, (dy, w, x.shape)),
                                   ("bwd_weight", conv_oracle.conv2d_bwd_weight, (x, dy, w.shape))]:
                ref, den = fn(*args, st, pad), fn(*(np.abs(a) if isinstance(a, np.ndarray) else a for a in args), st, pad)
                out = {"fwd": run.fwd, "bwd_data": run.bwd_data, "bwd_weight": run.bwd_weight}[name](*args[:2])
                assert (np.abs(out - ref) <= util.tight_bound(ref, den, dtype, dtype == "bf16" and name != "bwd_weight")).all(), (name, LAYERS[n])
    # searched once, whatever came in between
    before = mxc.mxc_plan_searches()
    for run, x, w, dy, _, _ in jobs:
        run.fwd(x, w), run.bwd_data(dy, w), run.bwd_weight(x, dy)
    assert mxc.mxc_plan_searches() == before


def test_last_plan_key_is_the_last_calls(mxc):
    """Forward and dx of layers in turn: the key is that of the layer just run, on the first turn (planned) and on the second (kept)."""
    layers = [(2, 3, 64, 64, 32, 7, 7, 2, 3), (2, 64, 14, 14, 64, 3, 3, 1, 1), (2, 3, 32, 32, 32, 3, 3, 1, 1), (2, 64, 9, 9, 96, 1, 1, 1, 0)]
    seen = []
    for _ in range(2):
        for dims in layers:
            run = util.Runner(mxc, dims, "bf16", "nhwc")
            run.fwd(np.zeros((run.N, run.C, run.H, run.W), np.float32), np.zeros((run.K, run.C, run.R, run.S), np.float32))
            seen.append(mxc.mxc_last_plan_key())
            assert seen[-1][:2] == (run.N * run.P * run.Q, run.K), dims
            if run.C > 4 or run.stride > 1:
                run.bwd_data(np.zeros((run.N, run.K, run.P, run.Q), np.float32), np.zeros((run.K, run.C, run.R, run.S), np.float32))
            if run.stride > 1:      # space-to-depth: 2x2 pixels of four values each, a 4x4 filter
                assert mxc.mxc_last_plan_key() == (run.N * 35 * 35, 16, 16 * run.K), dims
            elif run.C > 4:
                assert mxc.mxc_last_plan_key() == (run.N * run.H * run.W, run.C, run.R * run.S * run.K), dims
    assert seen[:len(layers)] == seen[len(layers):]
