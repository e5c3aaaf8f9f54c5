"""The two ways of a +-1 convolution inside the ConvNet forward give the same logits: on the map's plane "value is -1" (tiled FP4
kernel; the FP4 engine takes it at any size, the library itself from 48 tiles of 128 x 128 on), with the max-pooling done along
where the maps are 8, 16 or 32 pixels wide and of even height, and on the map's 2-bit code on the kernels for any size."""
import numpy as np
import pytest

import oracle
from test_gpu_convnet import _case, _run

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
