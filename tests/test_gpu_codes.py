"""First layer on uint8 codes with the weights kept as bits: rows and columns one off the tiles (128 x 128, 128 x 256), rows of codes that end
with a step, a half or a group of 128 elements or one piece of 16 behind it, a pitch; and the longest rows."""
import pytest
import torch

from qnn_testlib import kernels_of

pytestmark = pytest.mark.gpu


def _case(seed, M, N, K, ldx):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.randint(0, 256, (M, ldx), dtype=torch.uint8, device="cuda", generator=g)[:, :K]
    w = [torch.randint(0, 2, s, device="cuda", generator=g) * 2 - 1 for s in ((N, K), (10, N))]
    return x, w


def _check(q, x, w, kernel):
    (M, K), N = x.shape, w[0].shape[0]
    # (integers below 2^53, exact in float64)
    sums = torch.cat([r.double() @ w[0].double().t().contiguous() for r in x.split(256)]).to(torch.int64)
    T = (sums[0] + torch.arange(N, device="cuda") % 3 - 1).to(torch.int32)
    flip = (torch.arange(N, device="cuda") % 5 == 0).to(torch.uint8)
    W = [q.qnn_pack_sign(v.float()) for v in w]
    dims = [K, N, 10]
    for f in (None, flip):
        bit = (sums >= T[None]) != (0 if f is None else f[None] != 0)
        want = ((2.0 * bit - 1.0).double() @ w[1].double().t().contiguous()).to(torch.int32)
        run = lambda: q.qnn_binary_mlp_forward(x, 8, dims, W, [T], flip=[f], engine=q.ENGINE_MFMA)
        assert torch.equal(run(), want), (M, N, K, f is None)
    assert any(k.startswith(kernel) for k in kernels_of(run)), kernels_of(run)


@pytest.mark.parametrize("M,N", [(127, 129), (129, 255), (1025, 257), (2100, 2047), (4097, 4096), (4097, 4001), (4000, 4097), (9000, 130)])
@pytest.mark.parametrize("K,ldx", [(784, 784), (1024, 1040), (1040, 1040), (832, 848), (848, 848), (800, 800)])
def test_edges(seed, M, N, K, ldx):
    import paper_1609_07061_amd as q

    _check(q, *_case(seed, M, N, K, ldx), f"gemm_codes_kernel<{4 if N > 4000 else 2}>")


@pytest.mark.parametrize("K", [16, 32, 48, 64, 80, 112, 128, 144])
def test_short_rows(seed, K):
    import paper_1609_07061_amd as q

    _check(q, *_case(seed, 3001, 1030, K, K), "gemm_codes_kernel")


def test_longest_rows(seed):
    """Codes and weights that give the largest sums, near the row length at which matrix-core products end."""
    import paper_1609_07061_amd as q

    x, w = _case(seed, 600, 300, 130000, 130000)
    x[:2] = 255
    x[2:4] = 0
    w[0][:5] = 1
    w[0][5:9] = -1
    _check(q, x, w, "gemm_codes_kernel")
