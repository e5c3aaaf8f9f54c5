"""Convolutions of +-1 maps with few tiles on the sliced kernel: a plane's words one to seven a pixel, odd sizes with and without pooling (rows and
columns that no window covers), filters that end within a word, one pixel tiles and less, both numbers of waves, maps of ragged channels between."""
import numpy as np
import pytest
import torch

from qnn_testlib import dev, host, kernels_of
from test_gpu_convnet import _case, _run
from test_gpu_image import _bits, _conv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,W,couts,pools,sliced", [
    (3, 9, 11, [32, 70, 64, 33, 32], [0, 1, 0, 0, 1], 2),     # one word a pixel, ragged channels (2-bit code), two words
    (2, 15, 13, [96, 96, 160, 64], [0, 1, 0, 1], 3),          # three words, then five: the last piece of a tap brings one word
    (1, 6, 7, [224, 128, 100], [1, 1, 0], 2),                 # maps of 3 x 3 and 1 x 1 pixels
    (5, 8, 8, [256, 512, 512], [0, 1, 1], 2),
    (13, 8, 16, [128, 384, 32], [0, 0, 1], 2),                # four waves a tile
    (1, 2, 2, [128, 96, 96], [0, 0, 1], 2),                   # less than a tile, the image's edge at every pixel
])
@pytest.mark.parametrize("with_flip", [True, False])
def test_maps(seed, B, H, W, couts, pools, sliced, with_flip):
    import paper_1609_07061_amd as q

    if couts[-1] % 32 and (H >> sum(pools), W >> sum(pools)) != (1, 1):
        couts = couts[:-1] + [32]
    case = _case(seed, B, H, W, 3, couts, pools, [5], 2900, span=40)
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
    for engine in (q.ENGINE_AUTO, q.ENGINE_MFMA_FP4, q.ENGINE_VALU):
        assert np.array_equal(_run(q, case, couts, [5], engine=engine, with_flip=with_flip), want)
    kernels = kernels_of(lambda: _run(q, case, couts, [5], with_flip=with_flip))
    assert sum(k.startswith("gemm_slice_kernel<3, 0") for k in kernels) == sliced, kernels
