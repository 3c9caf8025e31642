"""Host-only checks of the product dispatch: which kernel and form a call takes."""
import ctypes

import pytest

from paper_2606_07116_amd import _lib

I64, I32 = ctypes.c_int64, ctypes.c_int32
KERNELS = ("plain", "plain_gemv", "gemv", "ksplit", "i8", "fp6")


class _Route(ctypes.Structure):
    _fields_ = [("kernel", I32), ("form", I32)]


_fn = ctypes.CDLL(_lib.LIB_PATH)["_ZN4offq10gemm_routeEllli"]
_fn.restype, _fn.argtypes = _Route, [I64, I64, I64, I32]


def route(M, N, K, g):
    """(kernel, form) as csrc/internal.h names them; the i8 kernel's form with its
    stages of 128 k per group (8: eight or more)."""
    r = _fn(M, N, K, g.bit_length() - 1)
    k = KERNELS[r.kernel]
    return (k, r.form, min(g // 128, 8)) if k == "i8" else (k, r.form)


@pytest.mark.parametrize("size,expect", [
    ((1, 4096, 4096, 64), ("plain_gemv", 0)), ((64, 4096, 4096, 64), ("plain", 0)),
    ((16, 8192, 28672, 512), ("gemv", 0)), ((64, 6144, 4096, 128), ("ksplit", 40208)),
    ((1777, 10240, 8192, 128), ("fp6", 2)), ((4096, 28672, 4096, 128), ("fp6", 1)),
    ((4096, 28672, 4096, 4096), ("fp6", 0)), ((2048, 4096, 4096, 4096), ("i8", 0, 8)),
    ((4096, 4096, 14336, 512), ("i8", 1, 4)), ((4096, 8192, 28672, 512), ("i8", 2, 4)),
])
def test_routes(size, expect):
    assert route(*size) == expect
