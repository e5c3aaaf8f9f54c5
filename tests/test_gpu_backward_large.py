"""The backward step on bit planes on both sides of the line above which a large gradient's transposition is a tiled launch of its own: coefficients that
are no powers of two keep the step on planes."""
import pytest
import torch

from qnn_testlib import kernels_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,tiled", [
    (12416, 12416, 3),   # 1.23e9 bits; weights and inputs have whole groups of words too
    (12288, 12160, 0),   # 1.195e9
    (12416, 12420, 0),   # rows of 389 words
])
def test_large_gradients(seed, M, N, tiled):
    import paper_1609_07061_amd as q

    torch.manual_seed(seed)
    K, coef = 256, [5, 1, 7, -3, 2, 11, -13, 4]
    w, a = torch.randint(0, 2, (N, K), device="cuda").float() * 2 - 1, torch.randint(0, 2, (M, K), device="cuda").float() * 2 - 1
    want_a, want_w = torch.zeros(M, K, device="cuda"), torch.zeros(N, K, device="cuda")
    planes = []
    for c in coef:  # (whole numbers below 2^24: exact in single precision)
        bits = torch.randint(0, 2, (M, N), device="cuda", dtype=torch.int8).float()
        want_a += c * (bits @ w)
        want_w += c * (bits.t().contiguous() @ a)
        planes.append(q.qnn_pack_sign(bits * 2 - 1))
    G, W, A = torch.stack(planes), q.qnn_pack_sign(w), q.qnn_pack_sign(a)
    run = lambda: q.qnn_binary_backward(G, coef, q.PLANE_BIT, N, W, A, K)
    ga, gw = run()
    assert torch.equal(ga.float(), want_a) and torch.equal(gw.float(), want_w)
    kernels = kernels_of(run)
    assert kernels.count("transpose_bits_tile_kernel") == tiled and kernels.count("transpose_jobs_kernel") == (tiled == 0), kernels
