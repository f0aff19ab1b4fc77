"""The transform length of a plan that forces a workgroup shape but no length (n_f = 0), by the size of
its workspace: the chunk table and the spectra of a length whose windows are nearly all halo are far
beyond those of the length the plan takes by itself."""

import ctypes

import numpy as np
import pytest


@pytest.fixture(scope="module")
def lib():
    import paper_0906_1775_amd
    return paper_0906_1775_amd.load()


@pytest.mark.parametrize("n_c", [33, 1000, 1023, 2047, 4095])   # 2 n_c just below a power of two among them
@pytest.mark.parametrize("shape", range(1, 11))
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_forced_shape_keeps_the_length(lib, precision, shape, n_c):
    from paper_0906_1775_amd import _lib
    n_t = 1 << 24
    iv, flt, lags = np.array([0, n_t], dtype=np.int64), np.zeros(1, np.int32), np.ones(n_c)
    d = _lib.MMDesc()
    d.n_stokes, d.n_pix, d.n_samples, d.n_intervals = 1, 1024, n_t, 1
    d.iv_start = iv.ctypes.data_as(ctypes.POINTER(ctypes.c_int64))
    d.iv_filter = flt.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))
    d.n_filters = 1
    d.filter_lags = lags.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
    d.n_c, d.n_rhs = n_c, 1
    d.precision = _lib.MM_FP64 if precision == "fp64" else _lib.MM_MIXED
    n = [ctypes.c_size_t(0), ctypes.c_size_t(0)]
    for i, s in enumerate((0, shape)):
        d.fft_shape = s
        assert lib.mm_plan_workspace_size(ctypes.byref(d), ctypes.byref(n[i])) == _lib.MM_OK, lib.mm_last_error()
    # (tables of the shapes themselves: at most 2^16 complex values of either precision)
    assert abs(n[1].value - n[0].value) <= 24 << 16
