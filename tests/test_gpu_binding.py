"""The calls whose arguments are marshalled natively give what the general path gives, and leave to it what they do not handle: views at
any pitch, tuples, other streams; errors of both kinds."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _general(q, monkeypatch):
    for name in ("pack_sign", "linear_quant_planes", "binary_gemm", "binary_gemm_sign", "bitplane_gemm", "bitplane_conv2d"):
        monkeypatch.setattr(q._native, name, lambda *a: -1)


def _calls(q):
    torch.manual_seed(3)
    x = torch.randn(40, 300, device="cuda")[::2, :257]
    A = q.qnn_pack_sign(x)
    W = q.qnn_pack_sign(torch.randn(70, 257, device="cuda"))
    u = q.qnn_pack_bitplanes(torch.randint(0, 4, (2 * 9 * 9, 64), dtype=torch.uint8, device="cuda"), 2).reshape(2, 2, 9, 9, 2)
    f = q.qnn_pack_sign(torch.randn(24 * 9, 64, device="cuda")).reshape(1, 24, 3, 3, 2)
    T, flip = torch.arange(70, dtype=torch.int32, device="cuda") - 35, (torch.arange(70, device="cuda") % 2).to(torch.uint8)

    def new(*shape):
        return torch.full(shape, -1, dtype=torch.int32, device="cuda")

    planes = q.qnn_linear_quant_planes(x, 0.25, -8, 7, 4, out=new(4, 20, 12)[:, :, :9])
    wp = q.qnn_linear_quant_planes(torch.randn(70, 257, device="cuda"), 0.5, -2, 1, 2, out=new(2, 70, 9))
    return [q.qnn_pack_sign(x, out=new(20, 15)[:, :9]), planes, wp, q.qnn_binary_gemm(A, W, 257, out=new(20, 75)[:, 2:72]),
            q.qnn_binary_gemm_sign(A, W, 257, T, out=new(20, 3)), q.qnn_binary_gemm_sign(A, W, 257, T, flip, out=new(20, 3)),
            q.qnn_bitplane_gemm(planes, [1, 2, 4, -8], q.PLANE_BIT, wp, (1, -2), q.PLANE_BIT, 257, out=new(20, 70)),
            q.qnn_bitplane_conv2d(u, [1, 2], q.PLANE_BIT, 64, f, (1,), q.PLANE_SIGN, 1, 2, out=new(2, 5, 5, 24))]


def test_same_results(monkeypatch):
    import paper_1609_07061_amd as q

    used = []
    for name in ("pack_sign", "linear_quant_planes", "binary_gemm", "binary_gemm_sign", "bitplane_gemm", "bitplane_conv2d"):
        native = getattr(q._native, name)
        monkeypatch.setattr(q._native, name, lambda *a, native=native: used.append(native(*a)) or used[-1])
    got = _calls(q)
    assert used == [0] * 8
    _general(q, monkeypatch)
    assert all(torch.equal(a, b) for a, b in zip(got, _calls(q)))


def test_current_stream():
    import paper_1609_07061_amd as q

    x, out = torch.randn(64, 4096, device="cuda"), torch.empty(64, 128, dtype=torch.int32, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        x.neg_()
        q.qnn_pack_sign(x, out=out)
    s.synchronize()
    assert torch.equal(out, q.qnn_pack_sign(x))


def test_errors():
    import paper_1609_07061_amd as q

    x, out = torch.randn(8, 64, device="cuda"), torch.empty(8, 2, dtype=torch.int32, device="cuda")
    with pytest.raises(ValueError, match="must be a GPU tensor"):
        q.qnn_pack_sign(x.cpu(), out=out)
    with pytest.raises(ValueError, match="must have dtype"):
        q.qnn_pack_sign(x.double(), out=out)
    with pytest.raises(ValueError, match="2-D with contiguous rows"):
        q.qnn_pack_sign(x.t(), out=out)
    with pytest.raises(q.QnnError, match="leading dimension"):
        q.qnn_pack_sign(x, out=out[:, :1].contiguous())
    with pytest.raises(ValueError, match="one coefficient per plane"):
        q.qnn_bitplane_gemm(out[None], [1, 2], 0, out[None], [1], 0, 64, out=torch.empty(8, 8, dtype=torch.int32, device="cuda"))
    with pytest.raises(q.QnnError, match="fit int32"):
        q.qnn_bitplane_gemm(out[None], [1 << 30], 0, out[None], [1], 0, 64, out=torch.empty(8, 8, dtype=torch.int32, device="cuda"))
