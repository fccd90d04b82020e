"""sage_decide rejects bad arguments before it touches a device (CPU only)."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2603_07917_amd", "libsage.so")
SAGE_OK, SAGE_EINVAL, SAGE_EWORKSPACE = 0, -1, -2
A = 0x10000


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2603_07917_amd import build
        build.build()
    lib = ctypes.CDLL(LIB)
    P, I, F, Z = ctypes.c_void_p, ctypes.c_int, ctypes.c_float, ctypes.c_size_t
    lib.sage_decide.argtypes = [P, I, I, P, I, P, I, I, I, F, P, P, P, I, P, P, P, P, P, P, P, Z, P]
    lib.sage_decide_workspace_bytes.argtypes = [I] * 6
    lib.sage_decide_workspace_bytes.restype = Z
    lib.sage_predict_workspace_bytes.argtypes = [I] * 5
    lib.sage_predict_workspace_bytes.restype = Z
    return lib


def test_decide_validation(lib):
    need = lib.sage_decide_workspace_bytes(2, 4, 100, 64, 8, 16)
    assert need >= lib.sage_predict_workspace_bytes(4, 100, 64, 8, 16) + 4 * 64 * 2
    assert lib.sage_decide_workspace_bytes(3, 4, 100, 64, 8, 16) == 0
    assert lib.sage_decide_workspace_bytes(2, 0, 100, 64, 8, 16) == 0

    def call(kind=2, Q=4, layout=1, N=100, d=64, k=8, tau=0.8, B=16, ws=1 << 30, null=None, odd=None):
        p = [A + 0x1000 * i for i in range(12)]
        if null is not None:
            p[null] = None
        if odd is not None:
            p[odd] += 4
        return lib.sage_decide(p[0], kind, Q, p[1], layout, p[2], N, d, k, tau, p[3], p[4], p[5], B, *p[6:11], A + 0x800,
                               p[11], ws, None)

    for bad in (dict(kind=3), dict(kind=-1), dict(layout=2), dict(Q=-1), dict(N=0), dict(d=48), dict(k=0), dict(k=257),
                dict(tau=0.0), dict(tau=1.5), dict(B=0), dict(B=4097), dict(Q=1 << 29)):
        assert call(**bad) == SAGE_EINVAL, bad
    for i in range(12):
        assert call(null=i) == SAGE_EINVAL, i
        assert call(odd=i) == SAGE_EINVAL, i
    assert call(ws=need - 1) == SAGE_EWORKSPACE
    assert call(Q=0) == SAGE_OK
