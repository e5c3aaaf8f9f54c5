"""The convolution kernels that hold a tile's pixels in LDS: images of one pixel row or column and of odd sizes, tiles that span several images, the
last tile ragged in pixels and filters, channels of one word to several pieces (ragged ones among them), one to five bit planes with a
factor of either sign; the +-1 maps of a ConvNet with max-pooling of odd sizes along."""
import numpy as np
import pytest
import torch

from qnn_testlib import dev, host, kernels_of
from test_gpu_convnet import _case, _run
from test_gpu_convnet_routes import _bits, _conv

pytestmark = pytest.mark.gpu


def _operands(q, B, H, W, C, N, bits):
    u = torch.randint(0, 1 << bits, (B, H, W, C), dtype=torch.uint8, device="cuda")
    w = torch.randint(0, 2, (N, 3, 3, C), device="cuda") * 2 - 1
    planes = q.qnn_pack_bitplanes(u.reshape(-1, C), bits).reshape(bits, B, H, W, -1)
    packed = q.qnn_pack_sign(w.reshape(-1, C).float()).reshape(N, 3, 3, -1)
    return planes, packed[None], _conv(u, w).to(torch.int64)  # (integers, exact)


@pytest.mark.parametrize("B,H,W,N", [(300, 1, 57, 129), (70, 241, 1, 130), (1000, 5, 3, 200), (130, 11, 13, 65), (9, 45, 47, 132), (1, 129, 130, 128), (17, 32, 32, 100)])
@pytest.mark.parametrize("C,bits", [(1, 2), (32, 1), (33, 3), (64, 2), (100, 5), (128, 4), (160, 1), (129, 2)])
def test_convolutions(seed, B, H, W, N, C, bits):
    import paper_1609_07061_amd as q

    torch.manual_seed(seed)
    planes, w, want = _operands(q, B, H, W, C, N, bits)
    for factor in (1, -3):
        coef = [factor << p for p in range(bits)]
        call = lambda: q.qnn_bitplane_conv2d(planes, coef, q.PLANE_BIT, C, w, [1], q.PLANE_SIGN, 1, 1)
        assert torch.equal(call().to(torch.int64), factor * want), factor
    assert all(k in ("gemm_image_kernel<2, 2, false>", "gemm_image_kernel<4, 2, false>") for k in kernels_of(call)), kernels_of(call)
    T = (want[0, 0, 0] + torch.arange(N, device="cuda") % 3 - 1).to(torch.int32)
    flip = (torch.arange(N, device="cuda") % 5 == 0).to(torch.uint8)
    coef = [1 << p for p in range(bits)]
    got = q.qnn_bitplane_conv2d_sign(planes, coef, q.PLANE_BIT, C, w, [1], q.PLANE_SIGN, 1, 1, T, flip)
    bit = (want >= T) != (flip != 0)
    assert torch.equal(got, q.qnn_pack_sign((bit.reshape(-1, N)).float() * 2 - 1).reshape(got.shape))


@pytest.mark.parametrize("bits,last,taken", [(8, 100, True), (8, 912, False)])
def test_largest_sums(seed, bits, last, taken):
    """Every code and weight at its largest; the kernel leaves sums of 2^21 (thresholds) to others."""
    import paper_1609_07061_amd as q

    B, H, W, C, N = 60, 20, 20, last, 128
    u = torch.full((B, H, W, C), (1 << bits) - 1, dtype=torch.uint8, device="cuda")
    planes = q.qnn_pack_bitplanes(u.reshape(-1, C), bits).reshape(bits, B, H, W, -1)
    signs = torch.where(torch.arange(N, device="cuda") % 2 == 0, 1.0, -1.0)
    w = q.qnn_pack_sign(signs[:, None].expand(N, 9 * C).reshape(-1, C).contiguous()).reshape(1, N, 3, 3, -1)
    ones = torch.nn.functional.conv2d(torch.ones(1, 1, H, W, device="cuda"), torch.ones(1, 1, 3, 3, device="cuda"), padding=1)[0, 0]
    want = (ones[..., None] * signs * (C * ((1 << bits) - 1))).to(torch.int64)
    coef = [1 << p for p in range(bits)]
    call = lambda: q.qnn_bitplane_conv2d(planes, coef, q.PLANE_BIT, C, w, [1], q.PLANE_SIGN, 1, 1)
    assert torch.equal(call().to(torch.int64), want[None].expand(B, H, W, N))
    for T in (-2**31, -2**21 - 1, 0, 9 * C * 255, 9 * C * 255 + 1, 2**31 - 1):
        t = torch.full((N,), T, dtype=torch.int32, device="cuda")
        sign = lambda: q.qnn_bitplane_conv2d_sign(planes, coef, q.PLANE_BIT, C, w, [1], q.PLANE_SIGN, 1, 1, t)
        bit = (want >= T).reshape(-1, N).float() * 2 - 1
        assert torch.equal(sign().reshape(B, H * W, -1), q.qnn_pack_sign(bit)[None].expand(B, -1, -1)), T
    assert any(k.startswith("gemm_image_kernel") for k in kernels_of(sign)) == taken


@pytest.mark.parametrize("B,H,W,couts,pools", [
    (40, 15, 13, [64, 96, 160, 64], [0, 1, 0, 1]),    # odd sizes: a row and a column that no window covers
    (3, 9, 33, [32, 64, 96], [0, 1, 1]),              # one tile and less
    (200, 7, 5, [100, 70, 33, 32], [0, 0, 1, 0]),     # ragged words of channels and filters
    (64, 4, 6, [128, 256, 224, 32], [0, 1, 0, 1]),    # several images a tile
    (1, 2, 2, [64, 64, 32], [0, 0, 1]),
])
@pytest.mark.parametrize("with_flip", [True, False])
def test_maps(seed, B, H, W, couts, pools, with_flip):
    import paper_1609_07061_amd as q

    case = _case(seed, B, H, W, 3, couts, pools, [5], 2700, span=40)
    x, conv_w, _, fc_w, T, flip = case
    h = dev(x)
    for l, pool in enumerate(pools):
        f = dev(flip[l]) if with_flip else torch.zeros(couts[l], dtype=torch.uint8, device="cuda")
        z = _conv(h, dev(conv_w[l]))
        if pool:
            hh, ww = z.shape[1] // 2, z.shape[2] // 2
            z = z[:, :2 * hh, :2 * ww].reshape(B, hh, 2, ww, 2, -1).amax(dim=(2, 4))
        h = _bits(z, dev(T[l]), f)
    want = host((h.reshape(B, -1).double() @ dev(fc_w[0]).double().t().contiguous()).to(torch.int32))
    for engine in (q.ENGINE_AUTO, q.ENGINE_MFMA_FP4):
        assert np.array_equal(_run(q, case, couts, [5], engine=engine, with_flip=with_flip), want)
    kernels = kernels_of(lambda: _run(q, case, couts, [5], engine=q.ENGINE_MFMA_FP4))
    assert sum(k in ("gemm_map_image_kernel<2>", "gemm_map_image_kernel<4>") for k in kernels) == len(couts) - 1 and kernels.count("pool_bits_kernel") == pools[0], kernels
