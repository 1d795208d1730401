"""Softmax of rows that a wave or four hold in registers: every form at its first and last length, the general form beside them, masked
values, infinities and NaN, and in place."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mxc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1512_01274_amd import mxc as m
    return m


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("pieces", [1, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025])
def test_rows(mxc, dtype, pieces):
    N, K = 5, pieces * 16 // dtype.itemsize
    g = torch.Generator(device="cuda").manual_seed(K)
    z = (torch.randn(N, K, generator=g, device="cuda") * 4).to(dtype)
    z[1] += 1000.0
    z[2, 1::2] = -3.0e38
    z[3, : K // 2] = -float("inf")
    z[4, K - 1] = float("nan")
    buf = torch.full((N * K + 64,), 7.0, dtype=dtype, device="cuda")
    mxc.mxc_softmax_fwd(N, K, mxc.dtype_code(dtype), z, buf)
    assert bool((buf[N * K:] == 7.0).all())
    p, want = buf[: N * K].view(N, K), torch.softmax(z.double(), 1)
    assert bool(p[4].isnan().all())
    # a sum of K terms and expf of arguments up to 20 in 32 bits, and one rounding to the stored type
    rel = 2.0 ** -19 + (2.0 ** -8 if dtype == torch.bfloat16 else 0)
    assert bool(((p[:4].double() - want[:4]).abs() <= rel * want[:4] + 1e-37).all())
    mxc.mxc_softmax_fwd(N, K, mxc.dtype_code(dtype), z, z)
    assert torch.equal(z[:4], p[:4])


def test_rows_off_16_bytes(mxc):
    """Rows that begin between 16-byte boundaries take the general form."""
    z = torch.randn(3, 1001, device="cuda").bfloat16()
    p = torch.empty_like(z)
    mxc.mxc_softmax_fwd(3, 1001, mxc.MXC_BF16, z, p)
    want = torch.softmax(z.double(), 1)
    assert bool(((p.double() - want).abs() <= (2.0 ** -8 + 2.0 ** -19) * want).all())
