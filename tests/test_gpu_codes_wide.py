"""Wide first layers on uint8 codes with few rows, whose weights' image finds no room: the kernel of 32 x 32 tiles up to a number of tiles, the one of large
tiles (which expands the bits per wave) beyond it, or the bit planes; thresholds over the whole range."""
import pytest
import torch

from qnn_testlib import kernels_of
from test_gpu_codes import _case
from test_gpu_codes_small import _run
from test_gpu_threshold_range import _thresholds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,ldx,small", [
    (160, 24576, 1024, 1024, True),    # 3840 tiles
    (160, 24577, 1024, 1024, False),
    (131, 18016, 1040, 1040, True),    # 2815
    (131, 18017, 1040, 1040, False),   # 2820
    (999, 32768, 784, 784, False),
    (160, 32768, 128, 128, True),     # bit planes otherwise: 20480 steps
    (160, 32769, 128, 128, False),
    (100, 20480, 256, 256, True),
    (100, 20481, 256, 256, False),
    (160, 32769, 112, 112, True),
    (160, 32769, 112, 128, False),
    (160, 32769, 128, 144, True),
    (130, 8193, 131056, 131056, True),  # longer than the kernels of large tiles take: VALU otherwise
])
def test_both_sides(seed, M, N, K, ldx, small):
    import paper_1609_07061_amd as q

    x, w = _case(seed, M, N, K, ldx)
    sums = (x.double() @ w[0].double().t().contiguous()).to(torch.int64)
    T = _thresholds(sums)
    flip = (torch.arange(N, device="cuda") % 5 == 0).to(torch.uint8)
    want = ((2.0 * ((sums >= T[None]) != (flip != 0)) - 1.0).double() @ w[1].double().t().contiguous()).to(torch.int32)
    run = _run(q, x, w, T, flip)
    assert torch.equal(run(), want)
    assert kernels_of(run)[0].startswith("gemm_codes_small_kernel") == small
