"""A convolution's weights or thresholds at odd addresses are refused before anything is launched, whichever kernel the layer's size selects (CPU)."""
import ctypes as C

import pytest

FAKE = 0x100000  # never dereferenced


@pytest.mark.parametrize("B,H,W,couts", [
    (4, 8, 8, [128, 512, 64]),       # few tiles, whole words: one plane on the sliced kernel
    (4, 8, 8, [100, 70, 64]),        # ragged channels: the map's 2-bit code
    (4, 8, 8, [32, 64, 64]),         # few channels: pixels in LDS
    (256, 16, 16, [128, 256, 64]),   # many tiles: pixels in LDS
    (64, 28, 28, [1024, 1024, 64]),  # pixels beyond it
])
@pytest.mark.parametrize("which", ["W", "T"])
@pytest.mark.parametrize("layer", [1, 2])
def test_refused(B, H, W, couts, which, layer):
    import paper_1609_07061_amd as q

    lib, n = q._lib, len(couts)
    i64, i32, ptr = C.c_int64, C.c_int32, C.c_void_p
    co, pool, fc = (i64 * n)(*couts), (i32 * n)(*([0] * n)), (i64 * 1)(10)
    addresses = {"W": [FAKE] * (n + 1), "T": [FAKE] * n + [None]}
    addresses[which][layer] = FAKE + 2
    need = lib.qnn_binary_convnet_workspace_bytes(i64(B), i64(H), i64(W), i64(3), 8, n, co, pool, 1, fc)
    assert need > 0
    status = lib.qnn_binary_convnet_forward(ptr(FAKE), i64(B), i64(H), i64(W), i64(3), 8, n, co, pool, 1, fc, (ptr * (n + 1))(*addresses["W"]),
                                            (ptr * (n + 1))(*addresses["T"]), None, ptr(FAKE), i64(10), ptr(FAKE), C.c_size_t(need), 0, None)
    assert status == 3
