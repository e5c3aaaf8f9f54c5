"""The backward step on bit planes, whose three transpositions share a launch: sizes one off the blocks of 256 rows and 32 words, rows with a gap
that holds anything, one to eight planes of either mode."""
import pytest
import torch

from qnn_testlib import kernels_of

pytestmark = pytest.mark.gpu


def _gap(x, extra):
    return torch.cat([x, torch.full((*x.shape[:-1], extra), -1, dtype=torch.int32, device="cuda")], -1)[..., :x.shape[-1]]


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (31, 33, 32), (255, 257, 1023), (257, 64, 1025), (64, 300, 1056), (513, 129, 95), (300, 1025, 33)])
@pytest.mark.parametrize("coef,mode", [([1, 2, 4, 8, 16, 32, 64, -128], 0), ([1, -2], 0), ([3], 1), ([1, 2, 4], 1), ([5, 1, 7, -3, 2], 0)])
@pytest.mark.parametrize("extra", [0, 3])
def test_small_steps(seed, M, N, K, coef, mode, extra):
    import paper_1609_07061_amd as q

    torch.manual_seed(seed)
    bits = torch.randint(0, 2, (len(coef), M, N), device="cuda")
    w, a = torch.randint(0, 2, (N, K), device="cuda") * 2 - 1, torch.randint(0, 2, (M, K), device="cuda") * 2 - 1
    value = sum(c * (2 * b - 1 if mode else b) for c, b in zip(coef, bits)).double()
    pack = lambda x: q.qnn_pack_sign((x.reshape(-1, x.shape[-1])).float()).reshape(*x.shape[:-1], -1)
    G, W, A = _gap(pack(2 * bits - 1), extra), _gap(pack(w), extra), _gap(pack(a), extra)
    run = lambda: q.qnn_binary_backward(G, coef, mode, N, W, A, K)
    ga, gw = run()
    assert torch.equal(ga.double(), value @ w.double()) and torch.equal(gw.double(), value.t().contiguous() @ a.double())
    assert kernels_of(run).count("transpose_jobs_kernel") == 1
