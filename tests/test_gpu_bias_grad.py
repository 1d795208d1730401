"""Bias gradient on the sizes its plan distinguishes: one share or several, rows of one to eight pixels (K against the
16-byte chunk), left-over pixels, column blocks, planes of unaligned length."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [(1, 1, 1, 1), (2, 8, 3, 3), (1, 7, 1, 1), (3, 7, 5, 9), (5, 30, 33, 31), (64, 20, 33, 7), (70, 96, 13, 13), (9, 1000, 5, 5), (17, 2600, 1, 1),
         (3, 2056, 41, 43), (200, 129, 11, 9), (1, 64, 300, 301), (40, 16, 57, 57), (2, 4096, 1, 1), (130, 6, 12, 20),
         (1, 512, 65, 65), (1, 520, 65, 65), (3, 63, 20, 20), (3, 65, 20, 20),       # 64 chunks a row and one more or less
         # one share in blocks of 4, 2 and 1 chunks: the lines at 1024, 2048 and 4096 rows, and at 20 and 10 chunks a row
         (1, 80, 32, 32), (1, 80, 25, 41), (1, 160, 25, 41), (1, 168, 25, 41), (2, 160, 32, 32), (2, 84, 32, 32), (1, 80, 3, 683), (1, 88, 3, 683), (1, 40, 3, 683),
         (1, 44, 3, 683), (4, 80, 32, 32), (4, 88, 32, 32), (4, 8, 32, 32), (1, 80, 17, 241), (1, 24, 17, 241)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("N,K,P,Q", CASES)
def test_bias_gradient(N, K, P, Q, layout, dtype):
    from paper_1512_01274_amd import mxc
    g = torch.Generator(device="cuda").manual_seed(N * 7919 + K)
    dy = torch.randn(*((N, P, Q, K) if layout == "nhwc" else (N, K, P, Q)), generator=g, device="cuda").to(dtype)
    lay = mxc.MXC_NHWC if layout == "nhwc" else mxc.MXC_NCHW
    dims = (N, 1, P, Q, K, 1, 1, 1, 0)
    ws = mxc.alloc_workspace(mxc.mxc_conv2d_workspace_bytes(mxc.MXC_BIAS_GRAD, *dims, mxc.dtype_code(dtype), lay))
    got = torch.full((2, (K + 67) // 4 * 4), 7.0, device="cuda")      # what follows the K values of each row must stay as it is
    for i in range(2):
        ws.fill_(255)
        mxc.mxc_bias_grad(N, K, P, Q, mxc.dtype_code(dtype), lay, dy, got[i][:K], ws)
    a = dy.double().cpu().numpy().transpose((3, 0, 1, 2) if layout == "nhwc" else (1, 0, 2, 3)).reshape(K, -1)
    assert torch.equal(got[0], got[1]) and bool((got[:, K:] == 7.0).all())
    err = np.abs(got[0][:K].double().cpu().numpy() - a.sum(1))
    assert np.all(err <= 64 * 2.0 ** -24 * np.abs(a).sum(1) + 1e-30)


def test_planes_of_more_than_two_to_the_31_pieces():
    """65536 NCHW images of one 512x512 channel, 34 GB of bf16: small whole numbers, so that every partial sum is exact."""
    from paper_1512_01274_amd import mxc
    N, P, Q = 65536, 512, 512
    value = (torch.arange(N, device="cuda") * 5 % 7 - 2).to(torch.bfloat16)
    dy = torch.empty(N, 1, P, Q, dtype=torch.bfloat16, device="cuda").copy_(value.view(N, 1, 1, 1))
    ws = mxc.alloc_workspace(mxc.mxc_conv2d_workspace_bytes(mxc.MXC_BIAS_GRAD, N, 1, P, Q, 1, 1, 1, 1, 0, mxc.MXC_BF16, mxc.MXC_NCHW))
    db = torch.full((4,), 7.0, device="cuda")
    mxc.mxc_bias_grad(N, 1, P, Q, mxc.MXC_BF16, mxc.MXC_NCHW, dy, db[:1], ws)
    assert db.tolist() == [float(value.double().sum() * (P * Q)), 7.0, 7.0, 7.0]
    del dy
    torch.cuda.empty_cache()
