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
