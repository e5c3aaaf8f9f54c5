"""Host time of a ConvNet call: choosing the layers' kernels costs less than the rest of the call's preparation (CPU: the first launch is refused, so a
call is its planning)."""
import ctypes as C
import time

import pytest
import torch

FAKE = 0x100000  # never dereferenced


@pytest.mark.parametrize("B,size,width", [(1, 32, 128), (4, 32, 128), (16, 32, 128), (256, 32, 128), (1, 16, 32)])
def test_planning_time(B, size, width):
    if torch.cuda.is_available():
        pytest.skip("the call would be launched")
    import paper_1609_07061_amd as q

    lib, i64, ptr = q._lib, C.c_int64, C.c_void_p
    co, pool, fc = (i64 * 6)(width, width, 2 * width, 2 * width, 4 * width, 4 * width), (C.c_int32 * 6)(0, 1, 0, 1, 0, 1), (i64 * 3)(1024, 1024, 10)
    W, T, flip = (ptr * 9)(*[FAKE] * 9), (ptr * 8)(*[FAKE] * 8), (ptr * 8)(*[FAKE] * 8)
    need = lib.qnn_binary_convnet_workspace_bytes(i64(B), i64(size), i64(size), i64(3), 8, 6, co, pool, 3, fc)

    def best(engine):
        args = (ptr(FAKE), i64(B), i64(size), i64(size), i64(3), 8, 6, co, pool, 3, fc, W, T, flip, ptr(FAKE), i64(10), ptr(FAKE), C.c_size_t(need), engine, None)
        times = []
        for _ in range(40):
            start = time.perf_counter()
            for _ in range(50):
                assert lib.qnn_binary_convnet_forward(*args) == 7
            times.append(time.perf_counter() - start)
        return min(times)

    assert best(q.ENGINE_AUTO) < 2.5 * best(q.ENGINE_VALU)
