"""Thresholds over the whole range of int32 in the epilogues that clamp them, next to the sums and at the clamping bounds; single planes whose
sums are formed in single precision (coefficients +-1, both kinds of plane) and those that are not."""
import pytest
import torch

pytestmark = pytest.mark.gpu

_INT = (-2**31, -2**31 + 1, -2**30 - 1, -2**30, -2**26, -2**24 - 1, -2**24, -2**22, -3 * 2**20 - 1, -3 * 2**20, -1, 0, 1, 3 * 2**20, 3 * 2**20 + 1, 2**22,
        2**24, 2**24 + 1, 2**26, 2**30, 2**30 + 1, 2**31 - 2, 2**31 - 1)


def _thresholds(sums):
    """One per column: the values above in every second column, elsewhere a sum of that column, one less or one more."""
    N = sums.shape[1]
    n = torch.arange(N, device="cuda")
    near = sums[n % sums.shape[0], n] + n % 3 - 1
    far = torch.tensor(_INT, dtype=torch.int64, device="cuda")[n // 2 % len(_INT)]
    return torch.where(n % 2 == 0, far, near).clamp(-2**31, 2**31 - 1).to(torch.int32)


def _packed(q, bit):
    return q.qnn_pack_sign(bit.float() * 2 - 1)


@pytest.mark.parametrize("M,N,K", [(130, 300, 512), (257, 129, 1300), (3000, 4100, 2048)])
@pytest.mark.parametrize("cA,modeA,cW,modeW", [(1, 1, 1, 1), (-1, 1, 1, 0), (1, 0, -1, 1), (1, 0, 1, 0), (3, 1, -2, 1), (-4, 0, 4, 1)])
def test_single_planes(seed, M, N, K, cA, modeA, cW, modeW):
    import paper_1609_07061_amd as q

    torch.manual_seed(seed)
    a, w = torch.randint(0, 2, (M, K), device="cuda"), torch.randint(0, 2, (N, K), device="cuda")
    value = lambda b, c, mode: (c * (2 * b - 1 if mode else b)).double()
    want = (value(a, cA, modeA) @ value(w, cW, modeW).t().contiguous()).to(torch.int64)  # (integers, exact)
    A, W, T = _packed(q, a), _packed(q, w), _thresholds(want)
    flip = (torch.arange(N, device="cuda") % 5 == 0).to(torch.uint8)
    C = q.qnn_bitplane_gemm(A[None], [cA], modeA, W[None], [cW], modeW, K, engine=q.ENGINE_MFMA_FP4)
    assert torch.equal(C.to(torch.int64), want)
    got = q.qnn_bitplane_gemm_sign(A[None], [cA], modeA, W[None], [cW], modeW, K, T, flip, engine=q.ENGINE_MFMA_FP4)
    assert torch.equal(got, _packed(q, (want >= T[None]) != (flip[None] != 0)))


@pytest.mark.parametrize("N", [300, 4100])
def test_codes(seed, N):
    import paper_1609_07061_amd as q

    torch.manual_seed(seed)
    M, K = 2100, 784
    x = torch.randint(0, 256, (M, K), dtype=torch.uint8, device="cuda")
    x[:3], x[3:6] = 0, 255
    w = [torch.randint(0, 2, s, device="cuda") * 2 - 1 for s in ((N, K), (10, N))]
    w[0][:40] = torch.where(torch.arange(40, device="cuda")[:, None] % 2 == 0, 1, -1)
    sums = (x.double() @ w[0].double().t().contiguous()).to(torch.int64)
    T = _thresholds(sums)
    flip = (torch.arange(N, device="cuda") % 5 == 0).to(torch.uint8)
    bit = (sums >= T[None]) != (flip[None] != 0)
    want = ((2.0 * bit - 1.0).double() @ w[1].double().t().contiguous()).to(torch.int32)
    W = [q.qnn_pack_sign(v.float()) for v in w]
    assert torch.equal(q.qnn_binary_mlp_forward(x, 8, [K, N, 10], W, [T], flip=[flip], engine=q.ENGINE_MFMA), want)
