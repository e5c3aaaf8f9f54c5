"""The FP4 kernels for products of any size and layout (32 x 32 and 64 x 64 tiles with k shared between waves, 128 x 128 tiles),
at the sizes where they can go wrong: one word more or less than a 16-byte piece, a 256-element chunk, a 1024-element group;
one row or column more or less than a tile; rows that start at any word; every pairing of planes into digits.  All results are
whole numbers: equality with the oracle."""
import numpy as np
import pytest
import torch

import oracle
import qnn_inputs as qi
from qnn_testlib import dev, host, host_u32, kernels_of, np_pack_bits, np_pack_pm1

pytestmark = pytest.mark.gpu

# 32 x 32 tiles on up to sixteen waves and, where there are many, on four; 64 x 64 (two shapes); 128 x 128; ragged on both edges
SHAPES = [(1, 1), (31, 33), (65, 32), (16500, 20), (640, 1025), (1601, 2049), (1601, 3300)]
KS = [97, 128, 129, 255, 257, 1024, 1056, 2049]


@pytest.mark.parametrize("M,N", SHAPES)
@pytest.mark.parametrize("K", KS)
def test_any_row_length_and_pitch(seed, M, N, K):
    import paper_1609_07061_amd as q

    a, w = qi.pm1(seed, 1200, (M, K)), qi.pm1(seed, 1201, (N, K))
    Kw = (K + 31) // 32
    A, W = dev(np_pack_pm1(a, Kw + 1))[:, :Kw], dev(np_pack_pm1(w, Kw + 3))[:, :Kw]
    want = oracle.gemm_pm1(a, w)
    for pad in (0, 3):
        out = torch.full((M, N + pad), -7, dtype=torch.int32, device="cuda")
        q.qnn_binary_gemm(A, W, K, out=out[:, :N])
        got = host(out)
        assert np.array_equal(got[:, :N], want) and (got[:, N:] == -7).all(), (M, N, K, pad)
    T, flip = qi.uniform_int(seed, 1202, (N,), -9, 9), qi.bernoulli_bits(seed, 1203, (N,))
    Nw = (N + 31) // 32
    bits = torch.full((M, Nw + 1), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    q.qnn_binary_gemm_sign(A, W, K, dev(T), dev(flip), out=bits[:, :Nw])
    got = host_u32(bits)
    assert np.array_equal(got[:, :Nw], oracle.pack_bits(oracle.threshold(want, T, flip))), (M, N, K)
    assert (got[:, Nw:] == 0x5A5A5A5A).all(), (M, N, K)


# pairs of consecutive powers of two with every combination of signs, gaps between powers, common factors, both modes
PLANES = [([1, 2], 0, [1], 1), ([1, -2], 0, [-1, 2], 0), ([-1, -2, 4], 0, [3], 0), ([1, 2, 4, -8], 0, [1, 2, 4, -8], 0),
          ([4, 1], 0, [2, -16], 0), ([-3, 6, 12], 1, [5, 10], 0), ([1, -4], 1, [-2, 1], 1), ([-5], 0, [1], 1), ([1], 1, [-2, 4], 0),
          ([3], 0, [1, -2], 0), ([1], 0, [-4], 0), ([1 << p for p in range(8)], 0, [1], 1)]


@pytest.mark.parametrize("M,N,K", [(33, 65, 300), (700, 1100, 1100), (1700, 2000, 131)])
@pytest.mark.parametrize("ca,ma,cw,mw", PLANES)
def test_digits_of_every_plane_pairing(seed, M, N, K, ca, ma, cw, mw):
    import paper_1609_07061_amd as q

    pa, pw = qi.bernoulli_bits(seed, 1210, (len(ca), M, K)), qi.bernoulli_bits(seed, 1211, (len(cw), N, K))
    want = oracle.gemm_planes(pa, ca, ma, pw, cw, mw)
    got = q.qnn_bitplane_gemm(dev(np_pack_bits(pa)), ca, ma, dev(np_pack_bits(pw)), cw, mw, K)
    assert np.array_equal(host(got), want), (M, N, K)


# (images, height = width, channels, filters, kernel, pad, stride): channels of one, two, three words and of one word more or less
# than a piece; maps whose windows reach outside on every side; enough tiles for the 128 x 128 kernel in the last two
CONVS = [(1, 6, 20, 33, 3, 1, 1), (2, 7, 64, 40, 3, 1, 2), (3, 9, 96, 64, 5, 2, 1), (2, 8, 128, 65, 3, 1, 1), (2, 9, 150, 70, 3, 0, 1),
         (3, 11, 230, 130, 1, 0, 1), (100, 23, 96, 100, 3, 1, 1), (64, 28, 160, 129, 3, 2, 1)]


@pytest.mark.parametrize("B,S,cin,cout,k,pad,stride", CONVS)
@pytest.mark.parametrize("coef", [[1], [1, 2], [1, 2, -4]])
def test_convolutions_of_any_channel_count(seed, B, S, cin, cout, k, pad, stride, coef):
    import paper_1609_07061_amd as q

    planes = qi.bernoulli_bits(seed, 1220, (len(coef), B, S, S, cin))
    u = sum(int(c) * planes[p].astype(np.int32) for p, c in enumerate(coef))
    w = qi.pm1(seed, 1221, (cout, k, k, cin))
    want = oracle.conv2d(u, w.astype(np.int32), pad, stride)
    A, W = dev(np_pack_bits(planes)), dev(np_pack_pm1(w)[None])
    got = q.qnn_bitplane_conv2d(A, coef, q.PLANE_BIT, cin, W, [1], q.PLANE_SIGN, pad, stride)
    assert np.array_equal(host(got), want)
    T, flip = qi.uniform_int(seed, 1222, (cout,), -9, 9), qi.bernoulli_bits(seed, 1223, (cout,))
    got = q.qnn_bitplane_conv2d_sign(A, coef, q.PLANE_BIT, cin, W, [1], q.PLANE_SIGN, pad, stride, dev(T), dev(flip))
    want_bits = oracle.pack_bits(oracle.threshold(want.reshape(-1, cout), T, flip))
    assert np.array_equal(host_u32(got).reshape(want_bits.shape), want_bits)


@pytest.mark.parametrize("cin", [20, 64, 130])
def test_convolution_of_sign_maps_without_padding(seed, cin):
    """+-1 activations: where a piece holds fewer words than four, or a chunk fewer taps than it has room for, the surplus counts
    (-1)(-1) and is taken off."""
    import paper_1609_07061_amd as q

    a, w = qi.pm1(seed, 1230, (2, 9, 9, cin)), qi.pm1(seed, 1231, (37, 3, 3, cin))
    got = q.qnn_bitplane_conv2d(dev(np_pack_pm1(a)[None]), [1], q.PLANE_SIGN, cin, dev(np_pack_pm1(w)[None]), [1], q.PLANE_SIGN, 0, 1)
    assert np.array_equal(host(got), oracle.conv2d(a.astype(np.int32), w.astype(np.int32), 0, 1))


def test_kernel_by_the_number_of_tiles():
    """Which of the kernels the library takes (GPU of 256 compute units)."""
    import paper_1609_07061_amd as q

    def product(planes, M, N, K):
        A = torch.zeros((planes, M, (K + 31) // 32), dtype=torch.int32, device="cuda")
        W = torch.zeros((1, N, (K + 31) // 32), dtype=torch.int32, device="cuda")
        mode = q.PLANE_SIGN if planes == 1 else q.PLANE_BIT
        return kernels_of(lambda: q.qnn_bitplane_gemm(A, [1 << p for p in range(planes)], mode, W, [1], q.PLANE_SIGN, K))

    small, many, large = "gemm_slice_kernel<0, 0, 0, 1, 1, 16>", "gemm_slice_kernel<0, 0, 0, 1, 1, 4>", "gemm_slice_kernel<0, 0, 0, 2, 2, 4>"
    assert product(1, 20, 1000, 2000) == [small]
    assert product(1, 20, 1000, 1000) == [many]          # four chunks of k, four waves
    assert product(1, 20000, 10, 2000) == [many]         # 625 tiles
    assert product(1, 20000, 10, 16000) == [small]       # ... of long rows
    assert product(1, 1000, 1000, 300) == [large]
    assert product(1, 40000, 96, 300) == [large]         # 1250 tiles
    assert product(1, 1999, 3001, 300) == ["gemm_tile_kernel<2, 2, 0>"]
    assert product(2, 1800, 1800, 300) == ["gemm_tile_kernel<1, 2, 0>"]


def test_panels_or_tiles_for_single_planes_of_whole_groups():
    """Rows of whole 128-byte groups, which the panel-fed kernel takes too: by the number of tiles, the row length and the output."""
    import paper_1609_07061_amd as q

    def kernel(M, N, K, sign):
        A = torch.zeros((M, K // 32), dtype=torch.int32, device="cuda")
        W, T = torch.zeros((N, K // 32), dtype=torch.int32, device="cuda"), torch.zeros(N, dtype=torch.int32, device="cuda")
        found = kernels_of(lambda: q.qnn_binary_gemm_sign(A, W, K, T) if sign else q.qnn_binary_gemm(A, W, K))
        assert len(found) == 1
        return found[0].split("<")[0]

    panel, small, tile = "gemm_panel_kernel", "gemm_slice_kernel", "gemm_tile_kernel"
    assert [kernel(10000, 256, K, False) for K in (1024, 8192)] == [small, small]        # 628 tiles of 64 x 64
    assert [kernel(10000, 256, K, True) for K in (1024, 8192)] == [small, small]
    assert [kernel(1500, 2048, K, True) for K in (1024, 8192)] == [panel, panel]         # 768
    assert [kernel(3000, 2048, K, False) for K in (1024, 2048, 4096)] == [tile, tile, panel]  # 1504; 192 tiles of 256 x 128
    assert [kernel(3000, 2048, K, True) for K in (1024, 4096)] == [panel, panel]
    assert [kernel(3000, 4096, K, sign) for K in (1024, 4096) for sign in (False, True)] == [panel] * 4


def test_tiles_or_merged_planes_by_the_pairs_of_digits():
    """Large products of several planes: each pair of digits is a product of its own on the tiles, one for all pairs on merged planes."""
    import paper_1609_07061_amd as q

    def merged(pa, pw, M, N, K, sign=False):
        A = torch.zeros((pa, M, (K + 31) // 32), dtype=torch.int32, device="cuda")
        W = torch.zeros((pw, N, (K + 31) // 32), dtype=torch.int32, device="cuda")
        T = torch.zeros(N, dtype=torch.int32, device="cuda")
        ca, cw = [1 << p for p in range(pa)], [1 << p for p in range(pw)]
        if sign:
            found = kernels_of(lambda: q.qnn_bitplane_gemm_sign(A, ca, 0, W, cw, 0 if pw > 1 else 1, K, T))
        else:
            found = kernels_of(lambda: q.qnn_bitplane_gemm(A, ca, 0, W, cw, 0 if pw > 1 else 1, K))
        return found[-1].startswith(("gemm_bytes_panel", "gemm_stage"))

    assert [merged(p, 1, 4096, 4096, 4096) for p in (2, 4, 5, 7)] == [False, False, True, True]
    assert [merged(p, p, 2240, 4096, 2048) for p in (2, 4)] == [False, True]
    assert [merged(p, 1, 2240, 4096, 2048) for p in (2, 4, 7)] == [False, False, True]
    assert not merged(4, 4, 1000, 1000, 16384)  # 64 tiles
    # eight unsigned planes do not fit a signed byte: merged per workgroup, in rounds of 256 x 256 tiles
    assert [merged(8, 1, M, N, K) for M, N, K in ((8192, 8192, 8192), (8192, 8192, 1024), (5000, 4096, 4096))] == [True, False, False]
    assert [merged(8, 1, M, N, K, True) for M, N, K in ((8192, 8192, 8192), (5000, 4096, 4096))] == [True, False]
