"""The panel-fed FP4 kernels: sizes one off 128 x 128 tiles, rows of one, three and more groups of 512, and rows of any length: one word, a
piece or a step more or less than a group, at any pitch; then sizes that the cost rule gives to the other tiles (128 x 256, 256 x 128, 256 x
256), cut by the last row, the last column or both."""
import numpy as np
import pytest
import torch

import oracle
from qnn_testlib import host, host_u32, kernels_of

pytestmark = pytest.mark.gpu


def _operands(seed, M, N, K):
    torch.manual_seed(seed)
    a, w = (torch.randint(0, 2, (rows, K), device="cuda") * 2 - 1 for rows in (M, N))
    return a, w, (a.double() @ w.double().t().contiguous()).to(torch.int32)


@pytest.mark.parametrize("M,N", [(129, 33), (127, 257), (1025, 2047), (385, 1281), (8200, 130), (2100, 4100)])
@pytest.mark.parametrize("K", [512, 1536, 4608, 481, 513, 768, 800, 1153, 2500])
def test_edges(seed, M, N, K):
    import paper_1609_07061_amd as q

    a, w, want = _operands(seed, M, N, K)
    A, W = q.qnn_pack_sign(a.float()), q.qnn_pack_sign(w.float())
    if K % 128:  # rows with a gap that holds anything
        A, W = (torch.cat([x, torch.full((x.shape[0], 3), -1, dtype=torch.int32, device="cuda")], 1)[:, :-3] for x in (A, W))
    T = want[0] + torch.arange(N, device="cuda", dtype=torch.int32) % 3 - 1
    flip = (torch.arange(N, device="cuda") % 5 == 0).to(torch.uint8)
    wide = torch.full((M, N + 3), 7, dtype=torch.int32, device="cuda")
    for C in (torch.empty((M, N), dtype=torch.int32, device="cuda"), wide[:, 1:1 + N]):
        q.qnn_binary_gemm(A, W, K, out=C, engine=q.ENGINE_MFMA_FP4)
        assert torch.equal(C, want), (M, N, K)
    assert bool((wide[:, 0] == 7).all()) and bool((wide[:, 1 + N:] == 7).all())
    rows = int(K % 512 != 0)  # whole groups or any
    assert kernels_of(lambda: q.qnn_binary_gemm(A, W, K, out=C, engine=q.ENGINE_MFMA_FP4)) == [f"gemm_panel_kernel<false, 2, 2, {rows}>"]
    got = q.qnn_binary_gemm_sign(A, W, K, T, flip, engine=q.ENGINE_MFMA_FP4)
    bit = host(((want >= T[None]) != (flip[None] != 0)).to(torch.int8))
    assert np.array_equal(host_u32(got), oracle.pack_bits((2 * bit - 1).astype(np.int8))), (M, N, K)
    assert kernels_of(lambda: q.qnn_binary_gemm_sign(A, W, K, T, engine=q.ENGINE_MFMA_FP4)) == [f"gemm_panel_kernel<true, 2, 2, {rows}>"]


@pytest.mark.parametrize("K", [512, 2560, 513, 2500])
@pytest.mark.parametrize("M,N,tile", [
    (2565, 5931, "2, 4"), (2688, 5900, "2, 4"), (2571, 6016, "2, 4"),  # 128 x 256; with all rows, with all columns
    (8209, 1803, "4, 4"), (8448, 1810, "4, 4"), (8213, 1920, "4, 4"),  # 256 x 128
])
def test_larger_tiles(seed, M, N, K, tile):
    import paper_1609_07061_amd as q

    a, w, want = _operands(seed, M, N, K)
    A, W = q.qnn_pack_sign(a.float()), q.qnn_pack_sign(w.float())
    if K % 512:  # rows with a gap that holds anything
        A, W = (torch.cat([x, torch.full((x.shape[0], 3), -1, dtype=torch.int32, device="cuda")], 1)[:, :-3] for x in (A, W))
    # C dense, on 16-byte boundaries, and word by word
    wide, pitch = torch.full((M, N + 3), 7, dtype=torch.int32, device="cuda"), (N + 3) // 4 * 4 + 4
    aligned = torch.full((M, pitch), 7, dtype=torch.int32, device="cuda")
    for C in (torch.empty((M, N), dtype=torch.int32, device="cuda"), aligned[:, :N], wide[:, 1:1 + N]):
        q.qnn_binary_gemm(A, W, K, out=C, engine=q.ENGINE_MFMA_FP4)
        assert torch.equal(C, want), (M, N, K, C.stride())
        rows = int(K % 512 != 0)
        assert kernels_of(lambda: q.qnn_binary_gemm(A, W, K, out=C, engine=q.ENGINE_MFMA_FP4)) == [f"gemm_panel_kernel<false, {tile}, {rows}>"]
    assert bool((wide[:, 0] == 7).all()) and bool((wide[:, 1 + N:] == 7).all()) and bool((aligned[:, N:] == 7).all())
    T = want[0] + torch.arange(N, device="cuda", dtype=torch.int32) % 3 - 1
    flip = (torch.arange(N, device="cuda") % 5 == 0).to(torch.uint8)
    bits = torch.full((M, (N + 31) // 32 + 2), 7, dtype=torch.int32, device="cuda")
    for f in (None, flip):
        q.qnn_binary_gemm_sign(A, W, K, T, f, out=bits[:, 1:-1], engine=q.ENGINE_MFMA_FP4)
        bit = host(((want >= T[None]) != (flip[None] != 0 if f is not None else False)).to(torch.int8))
        assert np.array_equal(host_u32(bits)[:, 1:-1], oracle.pack_bits((2 * bit - 1).astype(np.int8))), (M, N, K)
    assert bool((bits[:, 0] == 7).all()) and bool((bits[:, -1] == 7).all())
    kernel = kernels_of(lambda: q.qnn_binary_gemm_sign(A, W, K, T, flip, engine=q.ENGINE_MFMA_FP4))
    assert kernel == [f"gemm_panel_kernel<true, {tile}, {rows}>"], kernel


@pytest.mark.parametrize("M,N", [(4090, 4091), (4090, 4096), (4096, 4096)])
def test_wide_tiles(seed, M, N):
    import paper_1609_07061_amd as q

    K = 10240
    a, w, want = _operands(seed, M, N, K)
    A, W = q.qnn_pack_sign(a.float()), q.qnn_pack_sign(w.float())
    assert torch.equal(q.qnn_binary_gemm(A, W, K), want)  # (rows below the last whole tile: C on 16-byte boundaries and not)
    assert kernels_of(lambda: q.qnn_binary_gemm(A, W, K)) == ["gemm_panel_wide_kernel"]


@pytest.mark.parametrize("M,N,K,panel", [  # (GPU of 256 compute units)
    (4187, 1024, 3860, False), (1999, 3000, 600, True),     # C in 16-byte pieces: 1056 and 1504 tiles of 64 x 64
    (1270, 2303, 513, False), (1503, 2557, 1199, True), (2502, 1573, 3584, False),  # C word by word: 720, 960 and 1000
    (1999, 3001, 2500, True), (3053, 2174, 513, True),      # ... 384 and 408 tiles of 128 x 128
    (2376, 3953, 640, False), (2376, 3953, 1500, True),     # 589
    (2428, 7085, 2552, False), (2428, 7088, 2552, True), (3296, 6079, 5301, True),  # 1064, in 16-byte pieces, 1248
    (4861, 5809, 1090, False), (3535, 6269, 3378, True),    # 1748, 1372
])
def test_where_rows_of_other_lengths_leave_the_tiled_kernels(seed, M, N, K, panel):
    import paper_1609_07061_amd as q

    a, w, want = _operands(seed, M, N, K)
    A, W = q.qnn_pack_sign(a.float()), q.qnn_pack_sign(w.float())
    assert torch.equal(q.qnn_binary_gemm(A, W, K), want)
    assert kernels_of(lambda: q.qnn_binary_gemm(A, W, K))[0].startswith("gemm_panel_kernel") == panel
