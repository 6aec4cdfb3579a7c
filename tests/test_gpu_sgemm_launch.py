"""SGEMM on the GPU where a launch can go wrong: one request of sizes at the
edges of its tiles and k-tiles, and operands that start at any float.

Against the product in binary64: C sums n products in binary32, each with a
relative rounding error of at most 2^-24 of the running value, so the
Frobenius error is below n 2^-24 sqrt(n) (sqrt(n): |a||b| sums against the
norm of C for N(0, 1) entries), and far below it at these sizes."""

import ctypes

import numpy as np
import pytest

from paper_1511_07658_amd import gvm as G
from paper_1511_07658_amd import workloads as wl
from test_zz_no_alloc import D2H, H2D, hip

pytestmark = pytest.mark.gpu

SIZES = [1, 15, 17, 31, 33, 47, 63, 65, 95, 97, 127, 129, 200, 258, 385, 517, 1023, 1025]


@pytest.mark.parametrize("offset", [0, 1, 2])
@pytest.mark.parametrize("n", SIZES)
def test_one_request_at_the_edges(n, offset):
    h = hip()
    A, B = wl.sgemm_inputs(81, offset, n)
    x = np.concatenate([np.full(offset, np.nan, np.float32), A.ravel(), B.ravel()])
    out = np.full(n * n + 2 * offset, np.nan, np.float32)
    d_in, d_out = ctypes.c_void_p(), ctypes.c_void_p()
    assert h.hipMalloc(ctypes.byref(d_in), x.nbytes) == 0
    assert h.hipMalloc(ctypes.byref(d_out), out.nbytes) == 0
    try:
        assert h.hipMemcpy(d_in, x.ctypes.data, x.nbytes, H2D) == 0
        assert h.hipMemcpy(d_out, out.ctypes.data, out.nbytes, H2D) == 0
        rc = G.gvm_plain_run_noalloc(G.GVM_K_SGEMM, d_in.value + 4 * offset, d_out.value + 4 * offset, n)
        assert rc == 0, G.gvm_last_error()
        assert h.hipDeviceSynchronize() == 0
        assert h.hipMemcpy(out.ctypes.data, d_out, out.nbytes, D2H) == 0
    finally:
        h.hipFree(d_in)
        h.hipFree(d_out)
    C = out[offset:offset + n * n].reshape(n, n)
    want = A.astype(np.float64) @ B.astype(np.float64)
    assert np.linalg.norm(C - want) <= n * 2.0 ** -24 * np.sqrt(n) * np.linalg.norm(want) + 1e-30
    # nothing outside C is written
    assert np.isnan(out[:offset]).all() and np.isnan(out[offset + n * n:]).all()
