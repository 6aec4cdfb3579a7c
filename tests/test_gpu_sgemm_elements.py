"""Every element of C at the edges of the SGEMM's tiles and k-tiles, on the GPU.

An element sums n products in binary32, each added by a fused multiply-add that
is off by at most 2^-24 of the running value, so with u = 2^-24 it is within
n u / (1 - n u) of the sum of the products' magnitudes of the exact one."""

import ctypes

import numpy as np
import pytest

from paper_1511_07658_amd import gvm as G
from paper_1511_07658_amd import workloads as wl
from test_gpu_sgemm_launch import SIZES
from test_zz_no_alloc import D2H, H2D, hip


def wrong_elements(C, A, B):
    """(row, column) of the elements of C outside the bound."""
    A, B = A.astype(np.float64), B.astype(np.float64)
    nu = len(A) * 2.0 ** -24
    return np.argwhere(~(np.abs(C - A @ B) <= nu / (1 - nu) * (np.abs(A) @ np.abs(B))))


def test_one_wrong_element_is_seen():
    A, B = wl.sgemm_inputs(82, 0, 1025)
    C = (A.astype(np.float64) @ B.astype(np.float64)).astype(np.float32)
    assert wrong_elements(C, A, B).size == 0
    C[1024, 1024] = 0.0                     # the 1 x 1 corner tile not stored
    C[1024, 3] -= A[1024, 1024] * B[1024, 3]   # the remainder of k left out
    assert wrong_elements(C, A, B).tolist() == [[1024, 3], [1024, 1024]]


@pytest.mark.gpu
@pytest.mark.parametrize("n", SIZES)
def test_every_element_at_the_edges(n):
    h = hip()
    A, B = wl.sgemm_inputs(82, 0, n)
    x = np.concatenate([A.ravel(), B.ravel()])
    C = np.full((n, n), np.nan, np.float32)
    d_in, d_out = ctypes.c_void_p(), ctypes.c_void_p()
    assert h.hipMalloc(ctypes.byref(d_in), x.nbytes) == 0
    assert h.hipMalloc(ctypes.byref(d_out), C.nbytes) == 0
    try:
        assert h.hipMemcpy(d_in, x.ctypes.data, x.nbytes, H2D) == 0
        assert h.hipMemcpy(d_out, C.ctypes.data, C.nbytes, H2D) == 0
        rc = G.gvm_plain_run_noalloc(G.GVM_K_SGEMM, d_in.value, d_out.value, n)
        assert rc == 0, G.gvm_last_error()
        assert h.hipDeviceSynchronize() == 0
        assert h.hipMemcpy(C.ctypes.data, d_out, C.nbytes, D2H) == 0
    finally:
        h.hipFree(d_in)
        h.hipFree(d_out)
    bad = wrong_elements(C, A, B)
    assert bad.size == 0, (len(bad), bad[:5].tolist())
