"""Products of operands merged to bytes at every tile height (256, 192, 128 rows, halves in the last round), with rows and columns
that end inside a tile, rows of C at any alignment, and planes at every position of a byte or none."""
import numpy as np
import pytest
import torch

import oracle
import qnn_inputs as qi
from qnn_testlib import dev, host, kernels_of, np_pack_bits

pytestmark = pytest.mark.gpu

# tiles of 256 rows on 256 compute units: half a round (taken as 128 rows), 0.56 and 0.75 rounds (192), 1.25 rounds (halves), one; the
# kernel's arguments for that: halves in the last round, rows / 64
SHAPES = [(1793, 4081, 600, "false, 2"), (2230, 4096, 513, "false, 3"), (3071, 4090, 640, "false, 3"), (5000, 4100, 513, "true, 4"),
          (4096, 4096, 512, "false, 4")]
PLANES = [([1, 2, 4, -8], 0, [1, 2, 4, -8], 0), ([1, 4, 16, -64], 0, [2, 1, -4], 1), ([3, 5, -7], 0, [1, 3], 1)]


@pytest.mark.parametrize("M,N,K,tile", SHAPES)
@pytest.mark.parametrize("ca,ma,cw,mw", PLANES)
def test_merged_products(seed, M, N, K, tile, ca, ma, cw, mw):
    import paper_1609_07061_amd as q

    def operand(stream, coef, mode, rows):
        planes = qi.bernoulli_bits(seed, stream, (len(coef), rows, K)).astype(np.uint8)
        values = sum(c * (planes[p].astype(np.int32) if mode == 0 else 2 * planes[p].astype(np.int32) - 1) for p, c in enumerate(coef))
        return dev(np_pack_bits(planes, (K + 31) // 32)), values

    A, va = operand(1400, ca, ma, M)
    W, vw = operand(1401, cw, mw, N)
    wide = torch.full((M, N + 3), 7, dtype=torch.int32, device="cuda")
    for C in (torch.empty((M, N), dtype=torch.int32, device="cuda"), wide[:, 1:1 + N]):
        q.qnn_bitplane_gemm(A, ca, ma, W, cw, mw, K, out=C, engine=q.ENGINE_MFMA_LDS)
        # (sums below 2^24: exact in float64)
        want = torch.from_numpy(va).cuda().double() @ torch.from_numpy(vw).cuda().double().t().contiguous()
        assert torch.equal(C, want.to(torch.int32)), (M, N, K, ca)
    assert bool((wide[:, 0] == 7).all()) and bool((wide[:, 1 + N:] == 7).all())
    kernels = kernels_of(lambda: q.qnn_bitplane_gemm(A, ca, ma, W, cw, mw, K, out=C, engine=q.ENGINE_MFMA_LDS))
    assert kernels[-1] == f"gemm_bytes_panel_kernel<{tile}>", kernels
    rows = np.array([0, M - 1])
    assert np.array_equal(host(C)[rows], oracle.gemm_int(va[rows].astype(np.int32), vw.astype(np.int32)))


@pytest.mark.parametrize("rows", [1, 31, 33, 127, 200])
def test_rows_below_the_last_one_are_not_written(seed, rows):
    """Tiles cut by the last row of C alone, with 16-byte stores: 256 x 128 tiles of single planes, 256- and 128-row tiles of bytes."""
    import paper_1609_07061_amd as q

    M, N, K = 768 + rows, 1024, 3072  # (products of fewer than 2^31 elements are not merged to bytes)
    a, w = qi.bernoulli_bits(seed, 1410, (2, M, K)), qi.bernoulli_bits(seed, 1411, (N, K))
    A, W = dev(np_pack_bits(a)), dev(np_pack_bits(w[None]))
    vw = 2 * w.astype(np.int32) - 1
    for planes, coef, mode, engine in ((A[:1], [1], 1, q.ENGINE_MFMA_FP4), (A, [1, 2], 0, q.ENGINE_MFMA_LDS)):
        out = torch.full((M + 40, N), -7, dtype=torch.int32, device="cuda")
        q.qnn_bitplane_gemm(planes, coef, mode, W, [1], 1, K, out=out[:M], engine=engine)
        va = 2 * a[0].astype(np.int32) - 1 if mode == 1 else a[0].astype(np.int32) + 2 * a[1]
        got = host(out)
        assert np.array_equal(got[:M], oracle.gemm_int(va, vw)) and (got[M:] == -7).all(), (rows, engine)
