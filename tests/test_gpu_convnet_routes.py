"""The two ways of a +-1 convolution inside the ConvNet forward give the same logits: the panel-fed kernel on the map's sign plane
(the FP4 engine takes it at any size; the library itself from 32 tiles of 256 x 128 on) and the map's 2-bit code on the kernels
for products of any size."""
import numpy as np
import pytest

import oracle
from test_gpu_convnet import _case, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,Wd,couts,pools,fcs", [
    (3, 10, 14, [256, 200, 64], [0, 0, 1], [10]),        # ragged tiles of pixels and filters
    (2, 8, 16, [1024, 40, 32], [0, 0, 1], [6]),          # every step of the last group multiplied
    (8, 32, 32, [128, 128, 256], [0, 1, 1], [10]),       # 32 tiles (panel-fed), then 16 (not)
    (7, 32, 32, [128, 128, 256], [0, 1, 1], [10]),       # 28 tiles: nowhere by choice
])
def test_both_ways_of_a_convolution(seed, B, H, Wd, couts, pools, fcs):
    import paper_1609_07061_amd as q

    case = _case(seed, B, H, Wd, 3, couts, pools, fcs, 2200)
    want = oracle.convnet(*case)
    for engine in (q.ENGINE_AUTO, q.ENGINE_MFMA_FP4):
        assert np.array_equal(_run(q, case, couts, fcs, engine=engine), want), engine
