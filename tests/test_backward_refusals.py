"""The backward step refuses a bad argument before anything is launched that would read its operands (CPU; without a device a launch reports 7)."""
import ctypes as C

import pytest

FAKE = 0x100000  # never dereferenced
SHAPE, ALIGN, OVERFLOW = 2, 3, 4


@pytest.mark.parametrize("M,N,K", [(20, 96, 64), (300, 500, 700), (1000, 1024, 1024)])
@pytest.mark.parametrize("change,status", [
    (dict(stride=-1), SHAPE),
    (dict(mode=2), SHAPE),
    (dict(mode=-1), SHAPE),
    (dict(G=FAKE + 2), ALIGN),
    (dict(W=FAKE + 1), ALIGN),
    (dict(A=FAKE + 2), ALIGN),
    (dict(gA=FAKE + 2), ALIGN),
    (dict(gW=FAKE + 3), ALIGN),
    (dict(coef=[1 << 30, 1 << 30]), OVERFLOW),
])
@pytest.mark.parametrize("sign", [0, 1])
def test_refused(M, N, K, change, status, sign):
    import paper_1609_07061_amd as q

    lib, words = q._lib, lambda n: (n + 31) // 32
    i64, ptr = C.c_int64, C.c_void_p
    a = dict(G=FAKE, W=FAKE, A=FAKE, gA=FAKE, gW=FAKE, stride=M * words(N), mode=sign, coef=[1, 2])
    a.update(change)
    need = lib.qnn_binary_backward_workspace_bytes(i64(M), i64(N), i64(K), 2)
    got = lib.qnn_binary_backward(ptr(a["G"]), 2, (C.c_int32 * 2)(*a["coef"]), a["mode"], i64(words(N)), i64(a["stride"]), ptr(a["W"]), i64(words(K)), ptr(a["A"]),
                                  i64(words(K)), ptr(a["gA"]), i64(K), ptr(a["gW"]), i64(K), i64(M), i64(N), i64(K), ptr(FAKE), C.c_size_t(need), None)
    assert got == status
