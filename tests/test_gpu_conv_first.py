"""First convolution from the uint8 image: maps smaller and larger than a tile of 32 pixels, so that tiles at the ends of the image array (read
byte by byte) and inside it meet every border of an image; one to three channels; filters that end inside a word and inside four words.
Then the "inside the image" planes of maps behind a pooling, which fills them."""
import numpy as np
import pytest

import oracle
from qnn_testlib import kernels_of
from test_gpu_convnet import _case, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C0", [1, 2, 3])
@pytest.mark.parametrize("B,H,Wd", [(1, 1, 1), (70, 3, 1), (70, 1, 3), (3, 2, 31), (5, 9, 7), (2, 17, 32), (1, 3, 100), (9, 16, 16)])
@pytest.mark.parametrize("N", [5, 32, 100, 160])
def test_first_convolution(seed, C0, B, H, Wd, N):
    import paper_1609_07061_amd as q

    couts, pools, fcs = [N, 32], [0, 0], [7]
    case = _case(seed, B, H, Wd, C0, couts, pools, fcs, 2600 + C0)
    for with_flip in (True, False):
        want = oracle.convnet(*case[:5], case[5] if with_flip else None)
        assert np.array_equal(_run(q, case, couts, fcs, with_flip=with_flip), want), (B, H, Wd, C0, N)
    assert q.qnn_last_engines()[0] == 2


def test_most_filters(seed):
    import paper_1609_07061_amd as q

    couts, pools, fcs = [1024], [1], [4]
    case = _case(seed, 3, 10, 14, 3, couts, pools, fcs, 2610)
    assert np.array_equal(_run(q, case, couts, fcs), oracle.convnet(*case))


@pytest.mark.parametrize("couts,pools,ones", [
    ([32, 200, 64], [1, 0, 0], 0),          # seven words a pixel behind one
    ([200, 40, 96, 64], [1, 0, 1, 0], 0),   # two behind seven, then (pooled) none
    ([40, 70, 100, 32], [1, 0, 0, 0], 1),   # the second unpooled map has no pooling before it
    ([40, 70, 32], [0, 0, 0], 1),
])
@pytest.mark.parametrize("B,H,Wd", [(2, 9, 14), (1, 2, 2)])
def test_plane_of_the_next_map_filled_by_the_pooling(seed, couts, pools, ones, B, H, Wd):
    import paper_1609_07061_amd as q

    if (H >> sum(pools)) == 0:
        pytest.skip("the maps would be empty")
    case = _case(seed, B, H, Wd, 3, couts, pools, [6], 2620)
    want = oracle.convnet(*case)
    for _ in range(2):
        assert np.array_equal(_run(q, case, couts, [6]), want)
    kernels = kernels_of(lambda: _run(q, case, couts, [6]))
    assert kernels.count("ones_plane_kernel") == ones and kernels.count("pool_bits_kernel") == sum(pools), kernels
