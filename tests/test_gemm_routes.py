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


@pytest.mark.parametrize("M,N,K,g,kernel", [
    # one round of large tiles against 896 ... 2048 tiles of 64 x 64: the K-split kernel
    # took 1.1 to 1.5 times as long
    (1024, 4096, 4096, 4096, "i8"), (1024, 4096, 1024, 1024, "i8"), (512, 8192, 512, 512, "i8"),
    (2048, 2048, 2048, 2048, "i8"), (4096, 1024, 4096, 512, "i8"), (850, 4096, 4096, 512, "i8"),
    (128, 28672, 512, 512, "i8"),
    # and where it stays ahead
    (333, 4096, 14336, 512, "ksplit"), (512, 4096, 4096, 4096, "ksplit"),
    (768, 4096, 14336, 512, "ksplit"), (1024, 4096, 14336, 256, "ksplit"),
    (1024, 4096, 28672, 512, "ksplit"), (640, 4096, 8192, 8192, "ksplit"),
    (512, 4096, 4096, 128, "ksplit"), (333, 6144, 4096, 128, "fp6"),
])
def test_ksplit_ends_where_large_tiles_are_faster(M, N, K, g, kernel):
    assert route(M, N, K, g)[0] == kernel
