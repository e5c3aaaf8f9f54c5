"""The backward step on FP6 or int8 gradients: sizes one off its tiles (128 x 128, 128 x 256) and its groups of 256 and 128; gradients whose
values are all E3M2 numbers (three leading bits), and the same with a single one that is not, which turns both images to int8."""
import ctypes

import pytest
import torch

from qnn_testlib import kernels_of

pytestmark = pytest.mark.gpu

EXACT = sorted({s * m << e for s in (1, -1) for m in (0, 4, 5, 6, 7) for e in range(5) if m << e <= 112} | {1, 2, 3, -1, -2, -3, -128})
COEF = [1, 2, 4, 8, 16, 32, 64, -128]


def _step(q, v, coef, K, planes=None, mode=0, mixed=True):
    M, N = v.shape
    w, a = (torch.randint(0, 2, (r, K), device="cuda") * 2 - 1 for r in (N, M))
    G = q.qnn_pack_bitplanes((v & 255).to(torch.uint8), 8) if planes is None else planes
    W, A = q.qnn_pack_sign(w.float()), q.qnn_pack_sign(a.float())

    def call():
        return q.qnn_binary_backward(G, coef, mode, N, W, A, K)

    ga, gw = call()
    kernels = kernels_of(call)
    assert (kernels[:2] == ["transpose_to_image_kernel", "merge_transpose_kernel"]) == mixed, kernels
    assert sum(k.startswith("gemm_mixed_kernel") for k in kernels) == (2 if mixed else 0), kernels
    assert torch.equal(ga, (v.double() @ w.double()).to(torch.int32))
    assert torch.equal(gw, (v.t().contiguous().double() @ a.double()).to(torch.int32))


@pytest.mark.parametrize("M,N,K", [(1281, 2050, 2049), (2305, 1151, 1100), (4100, 2817, 385), (1000, 4096, 4100), (8192, 2304, 257),
                                   (128, 6000, 4096), (8000, 128, 4096), (100, 4000, 4096)])  # half groups of k: one alone, one with less
@pytest.mark.parametrize("kind", ["exact", "one other", "any"])
def test_formats(seed, M, N, K, kind):
    import paper_1609_07061_amd as q

    torch.manual_seed(seed)
    v = torch.tensor(EXACT, device="cuda")[torch.randint(0, len(EXACT), (M, N), device="cuda")]
    if kind == "one other":
        v[M - 1, N - 1] = -127
    elif kind == "any":
        v = torch.randint(-128, 128, (M, N), device="cuda")
    _step(q, v, COEF, K)


@pytest.mark.parametrize("value", [1, 7, -7, 9, -9, 17, 33, 65, 127, -127, 112, -128, 120])
def test_one_value_decides(seed, value):
    """A gradient of zeros but for one row of `value`: eight bits, and six +-1 planes of which all sums are odd."""
    import paper_1609_07061_amd as q

    torch.manual_seed(seed)
    M, N, K = 1009, 1280, 2784
    v = torch.zeros((M, N), dtype=torch.int64, device="cuda")
    v[500] = value
    _step(q, v, COEF, K)
    if value % 2 and abs(value) < 64:
        v = torch.ones((M, N), dtype=torch.int64, device="cuda")
        v[500] = value
        u = (v + 63) // 2  # v = sum of +-2^p over six planes
        _step(q, v, [1, 2, 4, 8, 16, 32], K, planes=q.qnn_pack_bitplanes(u.to(torch.uint8), 6), mode=1)


@pytest.mark.parametrize("kind", ["exact", "one other"])
def test_sums_up_to_the_bound(seed, kind):
    """131 071 rows of -128 but for the last ones, small odd values: sums close to the bound of 2^24 whose lowest bits count, added to
    accumulators that are close to it already."""
    import paper_1609_07061_amd as q

    torch.manual_seed(seed)
    M, N, K = 131071, 2048, 1024
    v = torch.full((M, N), -128, dtype=torch.int64, device="cuda")
    v[M - 255:] = torch.tensor([-7, -5, -3, -1, 1, 3, 5, 7], device="cuda")[torch.randint(0, 8, (255, N), device="cuda")]
    if kind == "one other":
        v[5, 7] = 127  # (both images are int8 then)
    w, a = torch.ones((N, K), device="cuda"), torch.randint(0, 2, (M, K), device="cuda").float() * 2 - 1
    w[::3, ::2] = -1
    a[:, :400], a[:, 400:800] = 1, -1
    G, W, A = q.qnn_pack_bitplanes((v & 255).to(torch.uint8), 8), q.qnn_pack_sign(w), q.qnn_pack_sign(a)
    ws = torch.empty(q.qnn_binary_backward_workspace_bytes(M, N, K, 8), dtype=torch.uint8, device="cuda")
    ga, gw = q.qnn_binary_backward(G, COEF, 0, N, W, A, K, workspace=ws)
    kernels = kernels_of(lambda: q.qnn_binary_backward(G, COEF, 0, N, W, A, K, workspace=ws))
    assert sum(k.startswith("gemm_mixed_kernel") for k in kernels) == 2, kernels
    want = (v.t().contiguous().double() @ a.double()).to(torch.int32)
    assert int(want.abs().max()) > 2 ** 24 - 2 ** 16 and bool((want[:, :400] % 2 != 0).any())
    assert torch.equal(gw, want)
    assert torch.equal(ga, (v.double() @ w.double()).to(torch.int32))


def test_largest_sums():
    """60 000 rows of -128 against weights of +1 in their larger half: sums up to 7.6e6 with steps of 128, and odd ones beside them."""
    import paper_1609_07061_amd as q

    M, N, K = 60000, 2048, 1024
    for odd in (64, 127):
        v = torch.full((M, N), -128, dtype=torch.int64, device="cuda")
        v[:, ::3] = 1
        v[::7, ::5] = odd
        w, a = torch.ones((N, K), device="cuda"), torch.ones((M, K), device="cuda")
        w[:, ::2] *= -1
        a[::3, 1::2] *= -1
        G, W, A = q.qnn_pack_bitplanes((v & 255).to(torch.uint8), 8), q.qnn_pack_sign(w), q.qnn_pack_sign(a)
        ga, gw = q.qnn_binary_backward(G, COEF, 0, N, W, A, K)
        assert torch.equal(ga, (v.double() @ w.double()).to(torch.int32))
        assert torch.equal(gw, (v.t().contiguous().double() @ a.double()).to(torch.int32))
        kernels = kernels_of(lambda: q.qnn_binary_backward(G, COEF, 0, N, W, A, K))
        assert sum(k.startswith("gemm_mixed_kernel") for k in kernels) == 2, kernels


@pytest.mark.parametrize("M,N,K,mixed", [
    (10000, 300, 300, False), (20000, 100, 1000, False), (7735, 325, 473, False), (393, 3517, 960, False),  # few tiles, long rows
    (1718, 452, 1895, True), (1451, 3329, 367, True), (300, 300, 20000, True),
])
def test_where_thin_steps_stay_on_the_planes(seed, M, N, K, mixed):
    import paper_1609_07061_amd as q

    torch.manual_seed(seed)
    _step(q, torch.randint(-128, 128, (M, N), device="cuda"), COEF, K, mixed=mixed)


def _hip():
    """The HIP runtime that this process has loaded."""
    with open("/proc/self/maps") as f:
        return ctypes.CDLL(next(w for line in f for w in line.split() if "libamdhip64.so" in w))


_USED_HIGH = 8  # hipMemPoolAttrUsedMemHigh


def _roundup(v, to):
    return (v + to - 1) // to * to


@pytest.mark.parametrize("M,N,K,P", [(7572, 2368, 444, 8), (20000, 4000, 300, 8), (2561, 2305, 1025, 8), (1281, 2050, 2049, 8), (3031, 2083, 906, 6),
                                     (17596, 1675, 760, 5), (1451, 3329, 367, 8)])
def test_memory_from_the_pool(seed, M, N, K, P):
    """No more than the header states: nothing for a transposed gradient of eight planes, which lies in the workspace."""
    import paper_1609_07061_amd as q

    torch.manual_seed(seed)
    v = torch.randint(-(1 << (P - 1)), 1 << (P - 1), (M, N), device="cuda")
    w, a = (torch.randint(0, 2, (r, K), device="cuda") * 2 - 1 for r in (N, M))
    G = q.qnn_pack_bitplanes((v & ((1 << P) - 1)).to(torch.uint8), P)
    W, A, coef = q.qnn_pack_sign(w.float()), q.qnn_pack_sign(a.float()), [1 << p for p in range(P - 1)] + [-(1 << (P - 1))]
    hip, pool, used = _hip(), ctypes.c_void_p(), ctypes.c_uint64(0)
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), torch.cuda.current_device()) == 0
    torch.cuda.synchronize()
    assert hip.hipMemPoolSetAttribute(pool, _USED_HIGH, ctypes.byref(used)) == 0
    ga, gw = q.qnn_binary_backward(G, coef, 0, N, W, A, K)
    torch.cuda.synchronize()
    assert hip.hipMemPoolGetAttribute(pool, _USED_HIGH, ctypes.byref(used)) == 0
    pitch_n, pitch_m = _roundup(N, 128), _roundup(M, 128)
    stated = M * pitch_n + (0 if P == 8 else N * pitch_m) + K * max(pitch_n, pitch_m) + _roundup(4 * (M + N), 256)
    assert 0 < used.value <= _roundup(stated, 4096), (used.value, stated)
    assert torch.equal(ga, (v.double() @ w.double()).to(torch.int32))
    assert torch.equal(gw, (v.t().contiguous().double() @ a.double()).to(torch.int32))


@pytest.mark.parametrize("M,N,K", [(1009, 1280, 2784), (1451, 3329, 367)])
def test_captured_step(seed, M, N, K):
    """In a graph, with its memory from the pool: new gradients, FP6 ones and others, and eager work between the replays."""
    import paper_1609_07061_amd as q

    torch.manual_seed(seed)
    w, a = (torch.randint(0, 2, (r, K), device="cuda") * 2 - 1 for r in (N, M))
    W, A = q.qnn_pack_sign(w.float()), q.qnn_pack_sign(a.float())
    values = [torch.tensor(EXACT, device="cuda")[torch.randint(0, len(EXACT), (M, N), device="cuda")], torch.randint(-128, 128, (M, N), device="cuda")]
    G = q.qnn_pack_bitplanes((values[0] & 255).to(torch.uint8), 8)
    ws = torch.empty(q.qnn_binary_backward_workspace_bytes(M, N, K, 8), dtype=torch.uint8, device="cuda")
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        q.qnn_binary_backward(G, COEF, 0, N, W, A, K, workspace=ws)
    torch.cuda.current_stream().wait_stream(stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ga, gw = q.qnn_binary_backward(G, COEF, 0, N, W, A, K, workspace=ws)
    for i in (0, 1, 0, 0, 1):
        q.qnn_pack_bitplanes((values[i] & 255).to(torch.uint8), 8, out=G)
        ga.zero_(), gw.zero_()
        graph.replay()
        assert torch.equal(ga, (values[i].double() @ w.double()).to(torch.int32)), i
        assert torch.equal(gw, (values[i].t().contiguous().double() @ a.double()).to(torch.int32)), i
        eager = q.qnn_binary_backward(G, COEF, 0, N, W, A, K)
        assert torch.equal(eager[0], ga) and torch.equal(eager[1], gw)
