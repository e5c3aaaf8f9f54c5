"""LogQuant over all exponents, mantissas around sqrt(2), infinities, NaN and denormals, at magnitudes where the short form of the rule begins and
ends; both sizes of a wave's share, rows that end within one, and the gate's edge values."""
import numpy as np
import pytest
import torch

import oracle
from qnn_testlib import dev, host_u32, np_unpack_bits

pytestmark = pytest.mark.gpu


def _floats(K, rows):
    man = np.array([0, 1, 0x1A827A, 0x3504F2, 0x3504F3, 0x3504F4, 0x3504F5, 0x7FFFFF], dtype=np.uint32)
    b = (np.arange(256, dtype=np.uint32)[:, None] << 23 | man[None]).reshape(-1)
    b = np.concatenate([b, b | np.uint32(1 << 31)])
    return np.resize(b, rows * K).view(np.float32).reshape(rows, K)


@pytest.mark.parametrize("emin,emax,as_value", [(-6, 0, 1), (-125, -119, 1), (-126, -120, 1), (-130, -124, 1), (122, 128, 1), (123, 129, 1), (-20, 40, 0), (0, 126, 0), (3, 3, 1)])
@pytest.mark.parametrize("rows,K", [(9, 1024), (8, 1028), (5, 2052), (4500, 2052)])
def test_log_quant(emin, emax, as_value, rows, K):
    import paper_1609_07061_amd as q

    x = _floats(K, rows)
    planes = q.qnn_log_quant_planes(dev(x), emin, emax, 8, as_value=bool(as_value))
    few = min(rows, 9)
    codes = oracle.log_quant(x[:few], emin, emax)
    want = np.sign(codes).astype(np.int64) * (1 << np.maximum(np.abs(codes.astype(np.int64)) - 1, 0)) if as_value else codes.astype(np.int64)
    got = host_u32(planes)
    for part, first in ((got[:, :few], 0), (got[:, rows - few:], rows - few)):
        bits = np_unpack_bits(part, K).astype(np.int64)
        value = sum(bits[p] * (1 << p if p < 7 else -128) for p in range(8))
        ref = want if first == 0 else None
        if ref is None:
            c = oracle.log_quant(x[first:first + few], emin, emax).astype(np.int64)
            ref = np.sign(c) * (1 << np.maximum(np.abs(c) - 1, 0)) if as_value else c
        assert np.array_equal(value, ref), (emin, emax, as_value, rows, K)


@pytest.mark.parametrize("rows,K", [(20, 2048), (3, 1540), (9000, 1032)])
def test_gate_and_linear_quant(rows, K):
    import paper_1609_07061_amd as q

    x = torch.from_numpy(_floats(K, rows).copy()).cuda()
    gate = torch.tensor([1.0, -1.0, 0.0, -0.0, 1.0000001, -1.0000001, float("nan"), float("inf"), 1e-42, 0.5], device="cuda").repeat(rows * K // 10 + 1)[:rows * K].reshape(rows, K)
    open_, gated = (q.qnn_log_quant_planes(x, -6, 0, 8, as_value=True, gate=g) for g in (None, gate))
    keep = q.qnn_pack_sign(torch.where(gate.abs() <= 1, 1.0, -1.0))
    assert torch.equal(gated, open_ & keep[None])
    for step in (0.25, 0.3):
        r = torch.round(x / step)  # (ties to even)
        want = torch.where(torch.isnan(r), torch.zeros_like(r), r).clamp(-8, 7).to(torch.int32)
        planes = q.qnn_linear_quant_planes(x, step, -8, 7, 4)
        for p in range(4):
            assert torch.equal(planes[p], q.qnn_pack_sign(((want >> p) & 1).float() * 2 - 1)), (step, p)
