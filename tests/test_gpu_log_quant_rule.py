"""LogQuant of short rows: which of its two forms a call takes, on both sides of the line, over all exponents, zeros and denormals."""
import numpy as np
import pytest

import oracle
from qnn_testlib import dev, host_u32, kernels_of, np_unpack_bits
from test_gpu_quant_range import _floats

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,K,short", [(2048, 128, True), (2049, 128, False), (2049, 129, True), (5000, 33, False)])
def test_both_forms(rows, K, short):
    import paper_1609_07061_amd as q

    x = _floats(K, rows)
    x[::7, ::3] = 0.0
    run = lambda: q.qnn_log_quant_planes(dev(x), -6, 0, 8, as_value=False)
    bits = np_unpack_bits(host_u32(run()), K).astype(np.int64)
    assert np.array_equal(sum(bits[p] * (1 << p if p < 7 else -128) for p in range(8)), oracle.log_quant(x, -6, 0).astype(np.int64))
    assert kernels_of(run)[0].endswith("LogQNormal>" if short else "LogQ>")
