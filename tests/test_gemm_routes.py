"""Host-only checks of the product dispatch: which kernel and form a call takes, and
that the GPU tests run every form that some call takes."""
import pytest

from paper_2606_07116_amd import _lib
from tests import test_gpu_gemm as G

def route(M, N, K, g):
    """The dispatch's (kernel, form); the i8 kernel's form with its stages of 128 k per
    group (8: eight or more)."""
    k, form = _lib.gemm_route(M, N, K, g)
    return (k, form, min(g // 128, 8)) if k == "i8" else (k, form)


@pytest.mark.parametrize("size,expect", [
    ((1, 4096, 4096, 64), ("plain_gemv", 0)), ((64, 4096, 4096, 64), ("plain", 0)),
    ((16, 8192, 28672, 512), ("gemv", 0)), ((64, 6144, 4096, 128), ("ksplit", 40208)),
    ((1777, 10240, 8192, 128), ("fp6", 2)), ((4096, 28672, 4096, 128), ("fp6", 1)),
    ((4096, 28672, 4096, 4096), ("fp6", 0)), ((2500, 8192, 256, 256), ("i8", 0, 2)), ((2048, 4096, 4096, 4096), ("i8", 0, 8)),
    ((4096, 4096, 14336, 512), ("i8", 1, 4)), ((4096, 8192, 28672, 512), ("i8", 2, 4)),
])
def test_routes(size, expect):
    assert route(*size) == expect


@pytest.mark.parametrize("M,N,K,g,kernel", [
    # one round of large tiles against 896 ... 2048 tiles of 64 x 64: the K-split kernel
    # took 1.1 to 1.5 times as long
    (1024, 4096, 4096, 4096, "i8"), (1024, 4096, 1024, 1024, "i8"), (512, 8192, 512, 512, "i8"),
    (2048, 2048, 2048, 2048, "i8"), (4096, 1024, 4096, 512, "i8"), (1024, 4096, 4096, 512, "i8"),
    (128, 28672, 512, 512, "i8"),
    # and where it stays ahead
    (333, 4096, 14336, 512, "ksplit"), (512, 4096, 4096, 4096, "ksplit"),
    (768, 4096, 14336, 512, "ksplit"), (1024, 4096, 14336, 256, "ksplit"),
    (1024, 4096, 28672, 512, "ksplit"), (700, 4096, 8192, 8192, "ksplit"),
    (700, 4096, 1024, 256, "ksplit"), (1000, 4096, 8192, 512, "ksplit"), (640, 4096, 2048, 512, "ksplit"),
    (512, 4096, 4096, 128, "ksplit"), (333, 6144, 4096, 128, "fp6"),
])
def test_ksplit_ends_where_large_tiles_are_faster(M, N, K, g, kernel):
    assert route(M, N, K, g)[0] == kernel


@pytest.mark.parametrize("M,N,K,g,form", [
    # short K: the sums of eight or sixteen waves took longer than their one step
    (1280, 1024, 512, 512, 40404), (1280, 1024, 1024, 1024, 40404), (96, 10240, 512, 512, 40404),
    (17, 14336, 256, 256, 20404), (1280, 1024, 2048, 2048, 40408),
    # the same for decode calls, 1.1 to 1.45 times as long
    (1, 14336, 128, 128, 10101), (8, 10240, 256, 128, 10101), (16, 10240, 512, 512, 10104),
    (5, 57344, 768, 256, 10102), (16, 10240, 1024, 128, 10108),
    # wide outputs, too few waves or too wide tiles, 1.05 to 1.25 times as long
    (1, 16384, 8192, 8192, 10108), (5, 20480, 8192, 2048, 10208), (16, 18432, 14336, 2048, 10208),
    (16, 16384, 16384, 2048, 10208), (8, 16368, 16384, 2048, 10108),
    (16, 16384, 12288, 512, 10216), (16, 28672, 12288, 512, 10408), (16, 14336, 8192, 128, 10208), (16, 10240, 8192, 128, 10108), (8, 6144, 8192, 128, 10216),
    # as they were
    (16, 28672, 8192, 8192, 10408), (16, 28672, 4096, 128, 10204), (1, 28672, 4096, 128, 10104),
    (16, 4096, 14336, 128, 10116), (1, 4096, 4096, 128, 10108), (16, 14336, 4096, 512, 10216),
])
def test_ksplit_forms(M, N, K, g, form):
    assert route(M, N, K, g) == ("ksplit", form)


@pytest.mark.parametrize("M,N,K,g,kernel", [
    (16, 8192, 28672, 512, "gemv"), (16, 6144, 20480, 128, "gemv"), (1, 8192, 24576, 4096, "gemv"),
    (16, 14336, 28672, 512, "gemv"), (16, 10240, 28672, 128, "ksplit"), (8, 10240, 28672, 512, "ksplit"),
    # measured slower there by 1.05 to 1.4 times
    (16, 8192, 16384, 512, "ksplit"), (1, 8192, 32768, 512, "ksplit"), (16, 8192, 32768, 8192, "ksplit"),
    (1, 10240, 28672, 512, "ksplit"), (16, 14336, 16384, 128, "ksplit"), (16, 6000, 28672, 512, "ksplit"),
])
def test_gemv_window(M, N, K, g, kernel):
    assert route(M, N, K, g)[0] == kernel


def _tested():
    shapes = [(5, 200, 1024, 64)]  # (of test_gemv_shapes)
    for t in (G.test_gemm_shapes, G.test_large_gemm_shapes, G.test_gemv_parts_of_k,
              G.test_few_token_rows, G.test_large_tile_forms, G.test_decode_shapes):
        shapes += next(m for m in t.pytestmark if m.name == "parametrize").args[1]
    return shapes


def _reachable():
    """Every route over a grid of sizes."""
    out = {}
    for K in (128, 256, 384, 640, 1024, 1536, 2048, 4096, 6144, 8192, 11008, 14336, 16384, 20480,
              28672, 32768):
        for g in (64, 128, 256, 512, 1024, 2048, 4096, 8192):
            if K % g:
                continue
            for N in (64, 1000, 4096, 5120, 8192, 10240, 14336, 16384, 28672, 57344):
                for M in (1, 4, 5, 16, 17, 33, 64, 100, 333, 600, 1000, 2048, 4096, 16384):
                    out.setdefault(route(M, N, K, g), (M, N, K, g))
    return out


def test_gpu_tests_run_every_form_that_a_call_takes():
    """Each form is run at least once, and once at sizes that leave remainders in both
    the rows and the columns."""
    tested = {route(*s) for s in _tested()}
    ragged = {route(*s) for s in _tested() if s[0] % 16 and s[1] % 16}
    reach = _reachable()
    assert len(reach) > 20
    missing = {r: s for r, s in reach.items() if r not in tested}
    assert not missing, missing
    assert not {r: s for r, s in reach.items() if r not in ragged}


def test_large_tile_list_has_every_form():
    """The shapes that the output-stride and extreme-value tests run."""
    assert [route(*s) for s in G.LARGE_TILES] == [("fp6", 2), ("fp6", 1), ("fp6", 0), ("i8", 0, 4),
                                                  ("i8", 1, 4), ("i8", 2, 2)]
