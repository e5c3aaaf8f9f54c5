"""First layer on uint8 codes for few rows: tiles one off 32 x 32, rows of codes that end with half a unit of 32, more units than waves and fewer, a
pitch, both numbers of waves, thresholds over the whole range, the largest sums; and which calls stay on the bit planes."""
import pytest
import torch

from qnn_testlib import kernels_of
from test_gpu_codes import _case
from test_gpu_threshold_range import _thresholds

pytestmark = pytest.mark.gpu


def _run(q, x, w, T, flip):
    K, N = x.shape[1], w[0].shape[0]
    W = [q.qnn_pack_sign(v.float()) for v in w]
    return lambda: q.qnn_binary_mlp_forward(x, 8, [K, N, 10], W, [T], flip=[flip])


@pytest.mark.parametrize("M,N", [(1, 1), (31, 33), (33, 64), (100, 1000), (300, 1030), (20, 4096)])
@pytest.mark.parametrize("K,ldx", [(16, 16), (784, 784), (784, 800), (1040, 1040), (48, 48), (4112, 4112), (70000, 70000)])
def test_few_rows(seed, M, N, K, ldx):
    import paper_1609_07061_amd as q

    x, w = _case(seed, M, N, K, ldx)
    x[:1] = 255
    x[-1:] = 0
    w[0][:3], w[0][3:5] = 1, -1
    sums = (x.double() @ w[0].double().t().contiguous()).to(torch.int64)
    T = _thresholds(sums)
    for flip in (None, (torch.arange(N, device="cuda") % 5 == 0).to(torch.uint8)):
        bit = (sums >= T[None]) != (0 if flip is None else flip[None] != 0)
        want = ((2.0 * bit - 1.0).double() @ w[1].double().t().contiguous()).to(torch.int32)
        assert torch.equal(_run(q, x, w, T, flip)(), want)
    many = -(-M // 32) * -(-N // 32) > 512
    assert kernels_of(_run(q, x, w, T, None))[0] == f"gemm_codes_small_kernel<{4 if many else 16}>"


@pytest.mark.parametrize("K,ldx,bits", [(784, 790, 8), (780, 784, 8), (784, 784, 7), (12288, 12288, 8)])
def test_others_go_through_planes(seed, K, ldx, bits):
    import paper_1609_07061_amd as q

    x, w = _case(seed, 40, 200, K, ldx)
    x &= (1 << bits) - 1
    sums = (x.double() @ w[0].double().t().contiguous()).to(torch.int64)
    T = _thresholds(sums)
    want = ((2.0 * (sums >= T[None]) - 1.0).double() @ w[1].double().t().contiguous()).to(torch.int32)
    W = [q.qnn_pack_sign(v.float()) for v in w]
    run = lambda: q.qnn_binary_mlp_forward(x, bits, [K, 200, 10], W, [T])
    assert torch.equal(run(), want)
    assert not any(k.startswith("gemm_codes") for k in kernels_of(run))
