"""The two ways of a +-1 convolution inside the ConvNet forward give the same logits: on the map's plane "value is -1" (tiled FP4
kernel; the FP4 engine takes it at any size, the library itself from 48 tiles of 128 x 128 on), with the max-pooling done along
where the maps are 8, 16 or 32 pixels wide and of even height, and on the map's 2-bit code on the kernels for any size."""
import numpy as np
import pytest
import torch

import oracle
from qnn_testlib import dev, host
from test_gpu_convnet import _case, _products, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,Wd,couts,pools,fcs", [
    (3, 10, 14, [256, 200, 64], [0, 0, 1], [10]),        # ragged tiles of pixels and filters
    (2, 8, 16, [1024, 40, 32], [0, 0, 1], [6]),          # long patches; pooled along, 16 wide
    (8, 32, 32, [128, 128, 256, 64], [0, 1, 1, 0], [10]),  # 64 tiles (on planes), pooled along 32 and 16 wide
    (7, 20, 32, [128, 128, 256], [0, 1, 1], [10]),       # 35 tiles: on planes by request only; ten rows of 16
    (3, 16, 8, [96, 64, 160], [0, 1, 1], [10]),          # 8 wide, three and two words of channels; then 4 wide (not along)
    (2, 9, 32, [70, 33, 32], [0, 1, 0], [7]),            # odd height: pooling apart; ragged words of channels and filters
    (1, 2, 2, [40, 64], [0, 1], [5]),                    # every pixel in a corner
    (5, 6, 16, [140, 130, 32], [0, 1, 1], [4]),          # a 16-byte piece and a ragged one per tap
])
@pytest.mark.parametrize("with_flip", [True, False])
def test_both_ways_of_a_convolution(seed, B, H, Wd, couts, pools, fcs, with_flip):
    import paper_1609_07061_amd as q

    x, conv_w, pools, fc_w, T, flip = _case(seed, B, H, Wd, 3, couts, pools, fcs, 2200)
    want = oracle.convnet(x, conv_w, pools, fc_w, T, flip if with_flip else None)
    for engine in (q.ENGINE_AUTO, q.ENGINE_MFMA_FP4):
        got = _run(q, (x, conv_w, pools, fc_w, T, flip), couts, fcs, engine=engine, with_flip=with_flip)
        assert np.array_equal(got, want), engine


def _conv(x, w):
    """3 x 3 "same" convolution, channels last, in double precision, on the GPU (the oracle takes minutes for these layers)."""
    B, H, Wd, C = x.shape
    w2 = w.reshape(w.shape[0], -1).double().t().contiguous()
    out = []
    for part in x.split(max(1, (1 << 27) // (H * Wd * 9 * C))):
        p = torch.nn.functional.pad(part.double(), (0, 0, 1, 1, 1, 1))
        patches = torch.stack([p[:, y:y + H, z:z + Wd] for y in range(3) for z in range(3)], dim=3)
        out.append((patches.reshape(-1, 9 * C) @ w2).reshape(-1, H, Wd, w.shape[0]))
    return torch.cat(out)


def _bits(sums, T, flip):
    return torch.where((sums >= T) != (flip != 0), 1.0, -1.0)


@pytest.mark.parametrize("B,H,Wd,cin,N,pool,kernel", [
    (13, 29, 31, 990, 1056, 0, "gemm_map_kernel<2, 4>"),   # 128 x 256, pixels and filters ragged (32 filters in the last tile), 31 words of channels
    (57, 12, 16, 990, 1056, 1, "gemm_map_kernel<2, 4>"),   # ... pooled along
    (26, 29, 31, 990, 800, 0, "gemm_map_kernel<4, 4>"),    # 256 x 128
    (123, 12, 16, 990, 800, 1, "gemm_map_kernel<4, 4>"),
    (37, 21, 30, 990, 96, 0, "gemm_map_kernel<2, 2>"),   # 128 x 128
    (75, 12, 16, 990, 96, 1, "gemm_map_kernel<2, 2>"),
    (37, 21, 30, 100, 96, 0, "gemm_map_image_kernel<2>"),   # pixels in LDS: 128 x 128
    (256, 17, 15, 100, 160, 1, "gemm_map_image_kernel<4>"),  # 256 x 128, odd sizes pooled along
])
@pytest.mark.parametrize("with_flip", [True, False])
def test_tiles_of_wide_layers(seed, B, H, Wd, cin, N, pool, kernel, with_flip):
    import paper_1609_07061_amd as q

    couts, pools, fcs = [cin, N], [0, pool], [5]
    case = _case(seed, B, H, Wd, 3, couts, pools, fcs, 2300, span=40)
    x, conv_w, _, fc_w, T, flip = case
    got = _run(q, case, couts, fcs, with_flip=with_flip)
    flips = [dev(f) if with_flip else torch.zeros(len(f), dtype=torch.uint8, device="cuda") for f in flip]
    h = _bits(_conv(dev(x), dev(conv_w[0])), dev(T[0]), flips[0])
    z = _conv(h, dev(conv_w[1]))
    if pool:
        z = z[:, :H // 2 * 2, :Wd // 2 * 2].reshape(B, H // 2, 2, Wd // 2, 2, N).amax(dim=(2, 4))
    h = _bits(z, dev(T[1]), flips[1]).reshape(B, -1)
    want = h.double() @ dev(fc_w[0]).double().t().contiguous()
    assert np.array_equal(got, host(want.to(torch.int32)))
    kernels = _products(q, case, couts, fcs)
    assert kernels[1] == kernel, kernels
