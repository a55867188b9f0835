"""The host rules of the tile GEMMs (CPU): which products they take, and which kernel
the choice gives.  The two functions are the library's own, by their C++ names."""
import ctypes

import pytest

lib_mod = pytest.importorskip("paper_2410_15352_amd._lib")


def _fn(name, restype, args):
    lib = ctypes.CDLL(lib_mod.LIB_PATH)
    fn = getattr(lib, name)
    fn.restype, fn.argtypes = restype, args
    return fn


def eligible(M, K, lda, ldb, rows_b, ldc0, ldc1=0):
    return _fn("_ZN7compact18gemm_tile_eligibleElllllll", ctypes.c_bool, [ctypes.c_int64] * 7)(M, K, lda, ldb, rows_b,
                                                                                               ldc0, ldc1)


def test_output_leading_dimensions_fit_an_int():
    """They reach the kernel as int: from 2^31 elements on, rows would go elsewhere."""
    big = 1 << 31
    assert eligible(4, 64, 64, 64, 256, big - 8) and eligible(4, 64, 64, 64, 256, 64, big - 8)
    assert not eligible(4, 64, 64, 64, 256, big) and not eligible(4, 64, 64, 64, 256, 64, big)
    assert not eligible(4, 64, 64, 64, 256, big + 64) and not eligible(4, 64, 64, 64, 256, 64, 3 * big)


def test_operands_fit_32_bit_offsets():
    assert eligible(1, 8, 8, 8, 1, 8)
    assert not eligible(1, 9, 8, 16, 1, 16) and not eligible(1, 8, 12, 8, 1, 8)
    assert not eligible(300, 64, 1 << 22, 64, 256, 64) and not eligible(300, 64, 64, 1 << 22, 256, 64)
    assert not eligible(1 << 31, 64, 64, 64, 256, 64) and not eligible(0, 64, 64, 64, 256, 64)


def choose(M, n0, n1, K, persistent, copies, cus=256):
    return _fn("_ZN7compact16gemm_tile_chooseEllllbbi", ctypes.c_int,
               [ctypes.c_int64] * 4 + [ctypes.c_bool] * 2 + [ctypes.c_int])(M, n0, n1, K, persistent, copies, cus)


def test_kernels_of_the_gpu_cases():
    """The GPU cases compare one kernel with another, and reach all four tiles, each with
    a whole last chunk of K and without."""
    gpu = pytest.importorskip("test_gpu_tile")
    seen = set()
    for (T, n, m, r), fwd, dx, long_f, long_d in gpu.CASES:
        f = lambda M: choose(M, m, r, n, n >= 320, False)
        d = lambda M: choose(M, n, 0, m, m >= 320, True)
        assert (f(T), d(T)) == (fwd, dx), (T, n, m, r)
        assert not long_f or f(long_f) == gpu.PERS, (T, n, m, r)
        assert not long_d or d(long_d) == gpu.PERS, (T, n, m, r)
        seen |= {(fwd, n % 8 != 0), (dx, m % 8 != 0)}
    assert seen >= {(k, mask) for k in range(4) for mask in (False, True)}


@pytest.mark.parametrize("M,n0,n1,K,persistent,copies,kind", [
    (65536, 1024, 128, 1024, True, False, 4), (65536, 2736, 0, 1024, True, True, 4),   # tiles fill the CUs
    (24040, 317, 0, 1384, True, True, 4), (26310, 1254, 0, 1816, True, True, 4),       # just past whole rounds
    (65536, 3072, 64, 256, False, False, 4), (12000, 700, 150, 300, False, False, 4),  # K < 320, many rows
    (8192, 1024, 0, 3072, True, True, 0), (1000, 512, 0, 2752, True, True, 3)])        # few tiles
def test_choice(M, n0, n1, K, persistent, copies, kind):
    """Where a tile kernel was measured slower than what ran before it, it is not taken."""
    assert choose(M, n0, n1, K, persistent, copies) == kind
