"""The backward step from bytes: sizes one off the tiles of its operand kernels (128 rows x 256 columns, four rows x 32 columns),
of its products (256 x 256, halves in the last round) and of their groups of 128; planes that stand for every kind of value."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import qnn_inputs as qi
from qnn_testlib import dev, host, kernels_of, np_pack_bits, np_pack_pm1

pytestmark = pytest.mark.gpu

VALUES = [1, 2, 4, 8, 16, 32, 64, -128]


@pytest.mark.parametrize("M,N,K", [(2560, 2600, 2050), (2817, 2433, 2049), (2400, 2304, 2273)])
@pytest.mark.parametrize("coef,mode", [(VALUES, 0), ([-3 * c for c in VALUES], 0), ([-3 * c for c in VALUES[:7]], 0),
                                       ([64, 1, 2, -4, 16, 8, 32], 0), ([1, -2, 4, 8, 16, -32], 1)])
def test_large_backward_step(seed, M, N, K, coef, mode):
    import paper_1609_07061_amd as q

    planes = qi.bernoulli_bits(seed, 1300, (len(coef), M, N)).astype(np.int64)
    g = sum(c * (planes[p] if mode == 0 else 2 * planes[p] - 1) for p, c in enumerate(coef))
    w, a = qi.pm1(seed, 1301, (N, K)), qi.pm1(seed, 1302, (M, K))
    Nw = (N + 31) // 32
    G = dev(np_pack_bits(planes.astype(np.uint8), Nw + 1))[:, :, :Nw]  # rows and planes with a gap
    W, A = dev(np_pack_pm1(w)), dev(np_pack_pm1(a))
    ga, gw = q.qnn_binary_backward(G, coef, mode, N, W, A, K)
    fits = coef[-1] != 384  # (the values / -3 run to 128: no bytes)
    assert ("merge_transpose_kernel" in kernels_of(lambda: q.qnn_binary_backward(G, coef, mode, N, W, A, K))) == fits
    want_ga = torch.from_numpy(g).double().cuda() @ torch.from_numpy(w.astype(np.float64)).cuda()
    want_gw = torch.from_numpy(np.ascontiguousarray(g.T)).double().cuda() @ torch.from_numpy(a.astype(np.float64)).cuda()
    assert torch.equal(ga, want_ga.to(torch.int32)), (M, N, K, coef)
    assert torch.equal(gw, want_gw.to(torch.int32)), (M, N, K, coef)
    rows = np.array([0, M - 1])
    assert np.array_equal(host(ga)[rows], oracle.gemm_int(g[rows].astype(np.int32), np.ascontiguousarray(w.T).astype(np.int32)))


class _PoolProps(ctypes.Structure):
    _fields_ = [("alloc_type", ctypes.c_int), ("handle_types", ctypes.c_int), ("location_type", ctypes.c_int),
                ("location_id", ctypes.c_int), ("security", ctypes.c_void_p), ("max_size", ctypes.c_size_t),
                ("reserved", ctypes.c_ubyte * 56)]


@pytest.fixture
def small_pool():
    """A device memory pool of 16 MiB as the current one, for calls that take temporary memory from their stream's pool."""
    hip = ctypes.CDLL("libamdhip64.so")
    torch.cuda.synchronize()
    before, pool = ctypes.c_void_p(), ctypes.c_void_p()
    device = torch.cuda.current_device()
    assert hip.hipDeviceGetMemPool(ctypes.byref(before), device) == 0
    props = _PoolProps(alloc_type=1, location_type=1, location_id=device, max_size=16 << 20)
    assert hip.hipMemPoolCreate(ctypes.byref(pool), ctypes.byref(props)) == 0
    assert hip.hipDeviceSetMemPool(device, pool) == 0
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

    def supplies(size):
        p = ctypes.c_void_p()
        rc = hip.hipMallocAsync(ctypes.byref(p), ctypes.c_size_t(size), stream)
        if rc == 0:
            assert hip.hipFreeAsync(p, stream) == 0
        else:
            hip.hipGetLastError()
        torch.cuda.synchronize()
        return rc == 0

    yield supplies
    torch.cuda.synchronize()
    assert hip.hipDeviceSetMemPool(device, before) == 0
    assert hip.hipMemPoolDestroy(pool) == 0


def test_pool_that_holds_the_operands_of_one_product_only(seed, small_pool):
    """Six +-1 planes, 2560 x 2600 x 2050: 19 MB of operands for both products together, 12.4 MB for the larger one."""
    import paper_1609_07061_amd as q

    M, N, K, coef = 2560, 2600, 2050, [1, -2, 4, 8, 16, -32]
    if small_pool(18 << 20):
        pytest.skip("the runtime does not keep a pool to its size")
    planes = qi.bernoulli_bits(seed, 1310, (len(coef), M, N)).astype(np.int64)
    g = sum(c * (2 * planes[p] - 1) for p, c in enumerate(coef))
    w, a = qi.pm1(seed, 1311, (N, K)), qi.pm1(seed, 1312, (M, K))
    ga, gw = q.qnn_binary_backward(dev(np_pack_bits(planes.astype(np.uint8))), coef, 1, N, dev(np_pack_pm1(w)), dev(np_pack_pm1(a)), K)
    want_ga = torch.from_numpy(g).double().cuda() @ torch.from_numpy(w.astype(np.float64)).cuda()
    want_gw = torch.from_numpy(np.ascontiguousarray(g.T)).double().cuda() @ torch.from_numpy(a.astype(np.float64)).cuda()
    assert torch.equal(ga, want_ga.to(torch.int32)) and torch.equal(gw, want_gw.to(torch.int32))


@pytest.mark.parametrize("planes,M,N,K,from_bytes", [(8, 1024, 1024, 1024, False), (4, 3000, 2048, 2048, False), (6, 3000, 2048, 2048, True),
                                                     (8, 1000, 4096, 4096, True), (8, 64, 4096, 4096, False)])
def test_way_by_the_expected_times(planes, M, N, K, from_bytes):
    import paper_1609_07061_amd as q

    G = torch.zeros((planes, M, N // 32), dtype=torch.int32, device="cuda")
    W, A = torch.zeros((N, K // 32), dtype=torch.int32, device="cuda"), torch.zeros((M, K // 32), dtype=torch.int32, device="cuda")
    coef = [1 << p for p in range(planes - 1)] + [-(1 << (planes - 1))]
    kernels = kernels_of(lambda: q.qnn_binary_backward(G, coef, 0, N, W, A, K))
    assert ("merge_transpose_kernel" in kernels) == from_bytes, kernels
