"""Which convolutions of bit planes the kernel with pixels in LDS takes: on both sides of each line of the rule."""
import pytest
import torch

from qnn_testlib import kernels_of
from test_gpu_image import _operands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,C,N,bits,sign,taken", [
    (35, 32, 32, 32, 2, False, False), (35, 32, 32, 33, 2, False, True), (35, 32, 32, 8, 1, True, True),
    (35, 32, 32, 63, 1, False, False), (35, 32, 64, 64, 1, False, True), (35, 32, 65, 64, 1, False, False),
    (35, 32, 96, 63, 2, False, True), (35, 32, 97, 63, 2, False, False), (35, 32, 97, 64, 2, False, True),
    (35, 32, 128, 64, 1, True, True), (35, 32, 129, 64, 1, True, False), (35, 32, 129, 65, 1, False, True),
    (19, 127, 9, 313, 1, False, True), (20, 127, 9, 313, 1, False, False), (20, 127, 9, 320, 1, False, True), (20, 127, 33, 316, 1, False, True),
])
def test_lines(seed, B, H, C, N, bits, sign, taken):
    import paper_1609_07061_amd as q

    torch.manual_seed(seed)
    planes, w, want = _operands(q, B, H, H, C, N, bits)
    coef = [1 << p for p in range(bits)]
    if sign:
        T = torch.zeros(N, dtype=torch.int32, device="cuda")
        call = lambda: q.qnn_bitplane_conv2d_sign(planes, coef, q.PLANE_BIT, C, w, [1], q.PLANE_SIGN, 1, 1, T)
        assert torch.equal(call().reshape(B * H * H, -1), q.qnn_pack_sign(want.reshape(-1, N).float()))
    else:
        call = lambda: q.qnn_bitplane_conv2d(planes, coef, q.PLANE_BIT, C, w, [1], q.PLANE_SIGN, 1, 1)
        assert torch.equal(call(), want.to(torch.int32))
    assert any(k.startswith("gemm_image_kernel") for k in kernels_of(call)) == taken
