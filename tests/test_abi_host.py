"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol the
header declares, validates arguments before touching the device, and answers workspace queries."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "mxc.h")


@pytest.fixture(scope="module")
def mxc():
    from paper_1512_01274_amd import mxc as m
    return m


def declared_symbols():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(mxc_[a-z0-9_]+)\s*\(", text)))


def test_header_symbols_are_exported(mxc):
    names = declared_symbols()
    assert {"mxc_conv2d_fwd", "mxc_conv2d_bwd_data", "mxc_conv2d_bwd_weight", "mxc_conv2d_workspace_bytes",
            "mxc_layout_convert", "mxc_status_string", "mxc_last_variant", "mxc_version"} <= set(names)
    lib = ctypes.CDLL(mxc.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), n
    for n in names:
        assert hasattr(mxc, n), f"binding lacks {n}"


def test_status_strings(mxc):
    seen = set()
    for code in range(0, 7):
        s = mxc.mxc_status_string(code)
        assert s and s != "unknown status" and s not in seen
        seen.add(s)
    assert mxc.mxc_status_string(99) == "unknown status"
    assert mxc.mxc_version() >= 100
    assert isinstance(mxc.mxc_last_variant(), str)


GOOD = (2, 16, 16, 16, 32, 3, 3, 1, 1)


@pytest.mark.parametrize("pos,val", [(0, 0), (1, -1), (2, 0), (3, 0), (4, 0), (5, 0), (6, -2), (7, 0), (8, -1),
                                     (5, 19), (6, 19)])
def test_shape_errors_before_any_pointer_use(mxc, pos, val):
    dims = list(GOOD)
    dims[pos] = val
    lib = mxc.raw()
    for fn in (lib.mxc_conv2d_fwd, lib.mxc_conv2d_bwd_data, lib.mxc_conv2d_bwd_weight):
        assert fn(*dims, mxc.MXC_F32, mxc.MXC_NCHW, None, None, None, None, 0, None) == mxc.MXC_ERR_SHAPE
    with pytest.raises(mxc.MxcError) as e:
        mxc.mxc_conv2d_workspace_bytes(mxc.MXC_FWD, *dims, mxc.MXC_F32, mxc.MXC_NCHW)
    assert e.value.status == mxc.MXC_ERR_SHAPE


def test_unsupported_and_null(mxc):
    lib = mxc.raw()
    assert lib.mxc_conv2d_fwd(*GOOD, 7, mxc.MXC_NCHW, None, None, None, None, 0, None) == mxc.MXC_ERR_UNSUPPORTED
    assert lib.mxc_conv2d_fwd(*GOOD, mxc.MXC_BF16, 5, None, None, None, None, 0, None) == mxc.MXC_ERR_UNSUPPORTED
    assert lib.mxc_conv2d_fwd(*GOOD, mxc.MXC_BF16, mxc.MXC_NHWC, None, None, None, None, 0, None) == mxc.MXC_ERR_NULL
    assert lib.mxc_conv2d_fwd(*GOOD, mxc.MXC_BF16, mxc.MXC_NHWC, 4096, 8192, None, None, 0, None) == mxc.MXC_ERR_NULL
    # misaligned (fake, never dereferenced) pointers are rejected before any launch
    assert lib.mxc_conv2d_bwd_data(*GOOD, mxc.MXC_BF16, mxc.MXC_NHWC, 4096, 8192 + 2, 16384, None, 0, None) \
        == mxc.MXC_ERR_ALIGN
    assert lib.mxc_layout_convert(1, 2, 3, 4, mxc.MXC_F32, 0, 1, None, None, None) == mxc.MXC_ERR_NULL
    assert lib.mxc_layout_convert(0, 2, 3, 4, mxc.MXC_F32, 0, 1, None, None, None) == mxc.MXC_ERR_SHAPE
    assert lib.mxc_layout_convert(1, 2, 3, 4, 9, 0, 1, None, None, None) == mxc.MXC_ERR_UNSUPPORTED
    assert lib.mxc_conv2d_workspace_bytes(9, *GOOD, 0, 0, ctypes.byref(ctypes.c_size_t())) == mxc.MXC_ERR_UNSUPPORTED
    assert lib.mxc_conv2d_workspace_bytes(0, *GOOD, 0, 0, None) == mxc.MXC_ERR_NULL


def test_workspace_query_is_consistent(mxc):
    for op in (mxc.MXC_FWD, mxc.MXC_BWD_DATA, mxc.MXC_BWD_WEIGHT):
        for dt in (mxc.MXC_F32, mxc.MXC_BF16):
            nchw = mxc.mxc_conv2d_workspace_bytes(op, *GOOD, dt, mxc.MXC_NCHW)
            nhwc = mxc.mxc_conv2d_workspace_bytes(op, *GOOD, dt, mxc.MXC_NHWC)
            assert nchw % 256 == 0 and nhwc % 256 == 0
            # NCHW needs room for the converted copies of all three tensors on top of the NHWC need
            assert nchw > nhwc
    # a call with too small a workspace is refused on the host, before any launch (fake aligned pointers)
    lib = mxc.raw()
    need = mxc.mxc_conv2d_workspace_bytes(mxc.MXC_FWD, *GOOD, mxc.MXC_F32, mxc.MXC_NCHW)
    assert lib.mxc_conv2d_fwd(*GOOD, mxc.MXC_F32, mxc.MXC_NCHW, 4096, 8192, 16384, 32768, need - 1, None) \
        == mxc.MXC_ERR_WORKSPACE


def test_workspace_query_over_random_shapes(mxc):
    """Host logic only: every pass answers the size query for a spread of shapes (all kernel families'
    geometry code runs in its dry mode), sizes are multiples of the carve-out alignment, and the
    grouped backward-data never needs less than the plain one."""
    import numpy as np
    rng = np.random.Generator(np.random.Philox(key=7))
    passes = (mxc.MXC_FWD, mxc.MXC_BWD_DATA, mxc.MXC_BWD_WEIGHT, mxc.MXC_BWD_DATA_RELU, mxc.MXC_BIAS_GRAD,
              mxc.MXC_BWD_DATA_FILTER, mxc.MXC_BWD_DATA_PREPARED, mxc.MXC_BWD_DATA_PREPARED_RELU)
    for _ in range(300):
        C = int(rng.choice([1, 2, 3, 4, 5, 8, 12, 16, 24, 64, 96, 192, 512]))
        K = int(rng.choice([1, 7, 8, 16, 40, 64, 96, 256, 520]))
        R = int(rng.choice([1, 2, 3, 5, 7, 11]))
        S = int(rng.choice([1, 2, 3, 5, 7, 11]))
        st = int(rng.integers(1, 5))
        pad = int(rng.integers(0, R + 1))
        H = int(rng.integers(max(1, R - 2 * pad), 64)) + R
        W = int(rng.integers(max(1, S - 2 * pad), 64)) + S
        N = int(rng.integers(1, 5))
        dims = (N, C, H, W, K, R, S, st, pad)
        for dt in (mxc.MXC_F32, mxc.MXC_BF16):
            for lay in (mxc.MXC_NCHW, mxc.MXC_NHWC):
                sizes = {p: mxc.mxc_conv2d_workspace_bytes(p, *dims, dt, lay) for p in passes}
                assert all(v % 256 == 0 and v < 2 ** 40 for v in sizes.values()), (dims, sizes)
                assert sizes[mxc.MXC_BWD_DATA_RELU] >= sizes[mxc.MXC_BWD_DATA], dims
                assert sizes[mxc.MXC_BIAS_GRAD] > 0
                # a prepared filter always has a size; with it, the call needs no more scratch than without
                assert sizes[mxc.MXC_BWD_DATA_FILTER] > 0, dims
                assert sizes[mxc.MXC_BWD_DATA_PREPARED] <= sizes[mxc.MXC_BWD_DATA], dims
                assert sizes[mxc.MXC_BWD_DATA_PREPARED_RELU] <= sizes[mxc.MXC_BWD_DATA_RELU], dims
                if dt == mxc.MXC_BF16:       # every bf16 path carves its filter forms out of the workspace
                    assert sizes[mxc.MXC_BWD_DATA_PREPARED] + sizes[mxc.MXC_BWD_DATA_FILTER] >= sizes[mxc.MXC_BWD_DATA], dims


def test_prepared_input_sizes_and_validation(mxc):
    """Host logic of the prepared-input calls: layers that read x as it is have an empty prepared form, first
    layers (C = 3) have one in each packing, with it a call needs no more scratch than without (the packed copy
    moved out of the workspace), NCHW is refused, and bad buffers are reported before any launch."""
    import ctypes as ct
    lib = mxc.raw()
    out = ct.c_size_t(0)
    q = lambda p, dims, dt=mxc.MXC_BF16, lay=mxc.MXC_NHWC: mxc.mxc_conv2d_workspace_bytes(p, *dims, dt, lay)
    plain = (2, 64, 14, 14, 32, 3, 3, 1, 1)
    assert q(mxc.MXC_INPUT_PREPARED, plain) == 0
    assert q(mxc.MXC_FWD_PREPARED_INPUT, plain) == q(mxc.MXC_FWD, plain)
    assert q(mxc.MXC_BWD_WEIGHT_PREPARED_INPUT, plain) == q(mxc.MXC_BWD_WEIGHT, plain)
    assert q(mxc.MXC_INPUT_PREPARED, plain, mxc.MXC_F32) == 0
    for dims in [(2, 3, 67, 67, 16, 11, 11, 4, 2), (2, 3, 30, 30, 16, 3, 3, 1, 1), (2, 20, 12, 12, 16, 3, 3, 1, 1)]:
        px = q(mxc.MXC_INPUT_PREPARED, dims)
        assert px > 0 and px % 256 == 0, dims
        assert q(mxc.MXC_FWD_PREPARED_INPUT, dims) + px == q(mxc.MXC_FWD, dims), dims
        assert q(mxc.MXC_BWD_WEIGHT_PREPARED_INPUT, dims) + px == q(mxc.MXC_BWD_WEIGHT, dims), dims
        assert q(mxc.MXC_BWD_WEIGHT_PREPARED_INPUT_BF16, dims) + px == q(mxc.MXC_BWD_WEIGHT_BF16, dims), dims
        for p in (mxc.MXC_INPUT_PREPARED, mxc.MXC_FWD_PREPARED_INPUT, mxc.MXC_BWD_WEIGHT_PREPARED_INPUT):
            assert lib.mxc_conv2d_workspace_bytes(p, *dims, mxc.MXC_BF16, mxc.MXC_NCHW, ct.byref(out)) == mxc.MXC_ERR_UNSUPPORTED
        big = 1 << 30
        assert lib.mxc_conv2d_prepare_input(*dims, 1, 1, 4096, None, big, None) == mxc.MXC_ERR_NULL
        assert lib.mxc_conv2d_prepare_input(*dims, 1, 1, 4096, 8192, px - 1, None) == mxc.MXC_ERR_WORKSPACE
        assert lib.mxc_conv2d_prepare_input(*dims, 1, 0, 4096, 8192, big, None) == mxc.MXC_ERR_UNSUPPORTED
        assert lib.mxc_conv2d_fwd_prepared_input(*dims, 1, 1, 4096, px - 1, 8192, None, 0, 16384, 32768, big, None) == mxc.MXC_ERR_WORKSPACE
        assert lib.mxc_conv2d_fwd_prepared_input(*dims, 1, 1, 4096, px, 8192, None, 2, 16384, 32768, big, None) == mxc.MXC_ERR_UNSUPPORTED
        assert lib.mxc_conv2d_bwd_weight_prepared_input(*dims, 1, 1, 4096, px - 1, 8192, 16384, 0, 32768, big, None) == mxc.MXC_ERR_WORKSPACE
        assert lib.mxc_conv2d_bwd_weight_prepared_input(*dims, 1, 1, 4096, px, 8192, 16384, 7, 32768, big, None) == mxc.MXC_ERR_UNSUPPORTED
        assert lib.mxc_conv2d_bwd_weight_prepared_input(*dims, 1, 1, None, px, 8192, 16384, 0, 32768, big, None) == mxc.MXC_ERR_NULL
    # the bf16 weight gradient exists for bf16 operands only
    assert lib.mxc_conv2d_workspace_bytes(mxc.MXC_BWD_WEIGHT_PREPARED_INPUT_BF16, *plain, mxc.MXC_F32, mxc.MXC_NHWC, ct.byref(out)) \
        == mxc.MXC_ERR_UNSUPPORTED


def test_transform_domain_forward_validation(mxc):
    """Host logic of the transform-domain forward: it exists for 3x3 stride-1 bf16 NHWC layers with channel counts
    that are multiples of 8, reports everything else as unsupported, and sizes its three workspace parts."""
    import ctypes as ct
    lib = mxc.raw()
    out = ct.c_size_t(0)
    ok = (2, 64, 14, 14, 32, 3, 3, 1, 1)
    T = 2 * 7 * 7
    need = mxc.mxc_conv2d_workspace_bytes(mxc.MXC_FWD_TRANSFORM, *ok, mxc.MXC_BF16, mxc.MXC_NHWC)
    assert need == 16 * 32 * 64 * 2 + 16 * T * 64 * 2 + 16 * T * 32 * 4       # U, V, M (each a multiple of 256 here)
    for bad in [(2, 64, 14, 14, 32, 5, 5, 1, 2), (2, 64, 14, 14, 32, 3, 3, 2, 1), (2, 60, 14, 14, 32, 3, 3, 1, 1),
                (2, 64, 14, 14, 36, 3, 3, 1, 1), (2, 64, 14, 14, 32, 1, 1, 1, 0)]:
        assert lib.mxc_conv2d_workspace_bytes(mxc.MXC_FWD_TRANSFORM, *bad, mxc.MXC_BF16, mxc.MXC_NHWC, ct.byref(out)) == mxc.MXC_ERR_UNSUPPORTED
        assert lib.mxc_conv2d_fwd_transform(*bad, mxc.MXC_BF16, mxc.MXC_NHWC, 4096, 8192, None, 0, 16384, 32768, 1 << 30, None) \
            == mxc.MXC_ERR_UNSUPPORTED
    for dt, lay in ((mxc.MXC_F32, mxc.MXC_NHWC), (mxc.MXC_BF16, mxc.MXC_NCHW)):
        assert lib.mxc_conv2d_workspace_bytes(mxc.MXC_FWD_TRANSFORM, *ok, dt, lay, ct.byref(out)) == mxc.MXC_ERR_UNSUPPORTED
    assert lib.mxc_conv2d_fwd_transform(*ok, 1, 1, 4096, 8192, None, 2, 16384, 32768, 1 << 30, None) == mxc.MXC_ERR_UNSUPPORTED
    assert lib.mxc_conv2d_fwd_transform(*ok, 1, 1, None, 8192, None, 0, 16384, 32768, 1 << 30, None) == mxc.MXC_ERR_NULL
    assert lib.mxc_conv2d_fwd_transform(*ok, 1, 1, 4096, 8192, 4098, 0, 16384, 32768, 1 << 30, None) == mxc.MXC_ERR_ALIGN
    assert lib.mxc_conv2d_fwd_transform(*ok, 1, 1, 4096, 8192, None, 0, 16384, 32768, need - 1, None) == mxc.MXC_ERR_WORKSPACE


def test_nchw_limits_are_reported_before_any_launch(mxc):
    """NCHW operands go through batched transposes with int row/column counts: what those cannot run is refused by the
    shape check itself (the size query sees it too), while the same problem in NHWC is accepted; batch and filter
    counts beyond 65535 are fine in both layouts."""
    import ctypes as ct
    out = ct.c_size_t(0)
    lib = mxc.raw()
    huge = (1, 1, 65536, 65536, 1, 1, 1, 1, 0)                # H*W = 2^32 elements per plane
    assert lib.mxc_conv2d_workspace_bytes(mxc.MXC_FWD, *huge, mxc.MXC_BF16, mxc.MXC_NCHW, ct.byref(out)) == mxc.MXC_ERR_SHAPE
    assert lib.mxc_conv2d_fwd(*huge, mxc.MXC_BF16, mxc.MXC_NCHW, 4096, 8192, 16384, None, 0, None) == mxc.MXC_ERR_SHAPE
    assert lib.mxc_conv2d_workspace_bytes(mxc.MXC_FWD, *huge, mxc.MXC_BF16, mxc.MXC_NHWC, ct.byref(out)) == mxc.MXC_OK
    many = (70000, 8, 4, 4, 70000, 1, 1, 1, 0)                # N and K beyond 65535
    for lay in (mxc.MXC_NCHW, mxc.MXC_NHWC):
        for p in (mxc.MXC_FWD, mxc.MXC_BWD_DATA, mxc.MXC_BWD_WEIGHT):
            assert lib.mxc_conv2d_workspace_bytes(p, *many, mxc.MXC_BF16, lay, ct.byref(out)) == mxc.MXC_OK


def test_grouped_entry_points_validate_on_the_host(mxc):
    lib = mxc.raw()
    big = 1 << 30
    # relu outside {0, 1}
    assert lib.mxc_conv2d_fwd_bias_act(*GOOD, 0, 0, 4096, 8192, None, 2, 16384, 32768, big, None) == mxc.MXC_ERR_UNSUPPORTED
    # misaligned bias
    assert lib.mxc_conv2d_fwd_bias_act(*GOOD, 0, 0, 4096, 8192, 4098, 1, 16384, 32768, big, None) == mxc.MXC_ERR_ALIGN
    # missing mask
    assert lib.mxc_conv2d_bwd_data_relu(*GOOD, 0, 0, 4096, 8192, None, 16384, 32768, big, None) == mxc.MXC_ERR_NULL
    # prepared filter: null buffer, buffer too small
    assert lib.mxc_conv2d_bwd_data_prepare_filter(*GOOD, 0, 0, 4096, None, big, None) == mxc.MXC_ERR_NULL
    assert lib.mxc_conv2d_bwd_data_prepare_filter(*GOOD, 0, 0, 4096, 8192, 16, None) == mxc.MXC_ERR_WORKSPACE
    assert lib.mxc_conv2d_bwd_data_prepared(*GOOD, 0, 0, 4096, 8192, 16, None, 16384, 32768, big, None) == mxc.MXC_ERR_WORKSPACE
    assert lib.mxc_conv2d_bwd_data_prepared(*GOOD, 0, 0, 4096, None, big, None, 16384, 32768, big, None) == mxc.MXC_ERR_NULL
    # bias gradient: shape, null, workspace
    assert lib.mxc_bias_grad(0, 8, 4, 4, 0, 1, 4096, 8192, 16384, big, None) == mxc.MXC_ERR_SHAPE
    assert lib.mxc_bias_grad(2, 8, 4, 4, 0, 1, None, 8192, 16384, big, None) == mxc.MXC_ERR_NULL
    assert lib.mxc_bias_grad(2, 8, 4, 4, 0, 1, 4096, 8192, 16384, 4, None) == mxc.MXC_ERR_WORKSPACE
    # update: empty, null, momentum without velocity
    assert lib.mxc_sgd_update(0, 4096, 8192, None, None, 0.1, 0.0, 0.0, None) == mxc.MXC_ERR_SHAPE
    assert lib.mxc_sgd_update(16, None, 8192, None, None, 0.1, 0.0, 0.0, None) == mxc.MXC_ERR_NULL
    assert lib.mxc_sgd_update(16, 4096, 8192, None, None, 0.1, 0.9, 0.0, None) == mxc.MXC_ERR_NULL
    assert lib.mxc_sgd_update(16, 4100, 8192, None, None, 0.1, 0.0, 0.0, None) == mxc.MXC_ERR_ALIGN
    # probe
    assert lib.mxc_probe_mfma(0, 10, 4096, 1 << 20, ctypes.byref(ctypes.c_double()), None) == mxc.MXC_ERR_SHAPE
    assert lib.mxc_probe_mfma(4, 10, 4096, 16, ctypes.byref(ctypes.c_double()), None) == mxc.MXC_ERR_WORKSPACE


def test_bias_gradient_limits(mxc):
    """NCHW: planes and the number of planes fit 31 bits, the tensor itself need not.  The last case passes every check, so that
    it is the launch that fails on a machine without a GPU (elsewhere the made-up pointers would reach it)."""
    import torch
    lib = mxc.raw()
    call = lambda N, K, P, Q, dt: lib.mxc_bias_grad(N, K, P, Q, dt, mxc.MXC_NCHW, 4096, 8192, 16384, 1 << 40, None)
    assert call(1, 1, 65536, 32768, mxc.MXC_BF16) == mxc.MXC_ERR_SHAPE
    assert call(65536, 32768, 1, 1, mxc.MXC_BF16) == mxc.MXC_ERR_SHAPE
    if torch.cuda.is_available():
        pytest.skip("no launch with made-up pointers")
    for N, K, P, Q, dt in [(65536, 1, 512, 512, mxc.MXC_BF16), (32768, 1, 1024, 512, mxc.MXC_F32), (2 ** 31 - 1, 1, 16, 16, mxc.MXC_BF16)]:
        assert call(N, K, P, Q, dt) == mxc.MXC_ERR_LAUNCH, (N, K, P, Q)
        dims = (N, 1, P, Q, K, 1, 1, 1, 0)
        assert mxc.mxc_conv2d_workspace_bytes(mxc.MXC_BIAS_GRAD, *dims, dt, mxc.MXC_NHWC) > 0


def test_bias_gradient_of_many_small_planes_is_shared(mxc):
    """NCHW: elements behind a plane's whole 16-byte pieces are loads of their own, and planes of fewer than a piece hold nothing else;
    one workgroup per channel would walk them one after another.  The scratch holds a partial sum per share and channel."""
    size = lambda n, pq, dt: mxc.mxc_conv2d_workspace_bytes(mxc.MXC_BIAS_GRAD, n, 1, pq, 1, 64, 1, 1, 1, 0, dt, mxc.MXC_NCHW)  # noqa: E731
    one = size(1, 1, mxc.MXC_BF16)
    for n, pq, dt in [(32768, 1, mxc.MXC_BF16), (4681, 7, mxc.MXC_BF16), (2730, 12, mxc.MXC_BF16), (16384, 1, mxc.MXC_F32), (5461, 3, mxc.MXC_F32)]:
        assert size(n, pq, dt) >= 3 * one, (n, pq)
    for n, pq, dt in [(4096, 8, mxc.MXC_BF16), (668, 49, mxc.MXC_BF16), (4096, 4, mxc.MXC_F32)]:
        assert size(n, pq, dt) == one, (n, pq)


def test_bias_gradient_shares_of_planes():
    """The two 31-bit counts of the NCHW kernel, over the plan's rule replayed here: whole 16-byte pieces of a workgroup's planes,
    and its planes times the elements behind the last piece."""
    for V in (4, 8):
        for K in (1, 2, 3, 7, 64, 511, 512, 513, 5000, 1 << 20):
            for PQ in (1, 3, 4, 7, 8, 9, 100, 1 << 12, (1 << 18) + 7, 2 ** 31 - 1):
                for N in (1, 2, 3, 511, 512, 65536, 1 << 24, 1 << 30, (2 ** 31 - 1) // K):
                    if N * K > 2 ** 31 - 1 or N * K * PQ >= 2 ** 40:
                        continue
                    parts = max(1, min((512 + K - 1) // K, max(1, N * PQ * (16 // V) // (16 << 10)), N))
                    per = (N + parts - 1) // parts
                    assert per * (PQ // V) < 2 ** 30 and per * (PQ % V) < 2 ** 32, (V, K, PQ, N)


def test_tile_names(mxc):
    """Every kernel shape has a name of its own in one of ten families."""
    families = [mxc.mxc_tile_names(f) for f in range(10)]
    names = [n for f in families for n in f]
    assert all(families) and len(set(names)) == len(names)
    for family, prefix in ((4, "igemm_wave_"), (5, "wgrad_wave_"), (8, "igemm_run_"), (9, "wgrad_run_")):
        assert all(n.startswith(prefix) for n in families[family])
    assert mxc.mxc_tile_name(10, 0) is None and all(mxc.mxc_tile_name(f, -1) is None for f in range(10))
