"""Error of a tallied pair on the GPU: requests of one pair under many keys,
each returning its Gaussian pair, against 64-bit-mantissa arithmetic.

In units of 2^-53 of a value.  A rounding is uniform within half a unit in the
last place, which for a mantissa m spread over 1 .. 2 by its logarithm is a mean
square of (3 / 8 / ln 2) / 3 = 0.18; under a root it counts a quarter.  X =
x sqrt(-2 ln t / t) by a rounded logarithm, divide, root and product has the root
mean square sqrt(0.18 (1 + 1 + 1/4 + 1/4)) = 0.671, which is the limit here.
The largest: 1 of the product, 1 of the factor, 1/2 of the product under the root,
1/4 of the reduced argument next to t = 1, and 1/4 for the rest."""

import ctypes

import numpy as np
import pytest

from oracle import ep as oe
from paper_1511_07658_amd import gvm as G
from paper_1511_07658_amd import workloads as wl
from test_zz_no_alloc import D2H, H2D, hip

pytestmark = pytest.mark.gpu


def test_error_of_single_pairs():
    h = hip()
    keys = [wl.ep_key(95, r, 0) for r in range(10000)]
    kin = np.array(keys, np.uint64)
    out = np.zeros((len(keys), 12), np.float64)
    d_in, d_out = ctypes.c_void_p(), ctypes.c_void_p()
    assert h.hipMalloc(ctypes.byref(d_in), kin.nbytes) == 0
    assert h.hipMalloc(ctypes.byref(d_out), out.nbytes) == 0
    try:
        assert h.hipMemcpy(d_in, kin.ctypes.data, kin.nbytes, H2D) == 0
        for i in range(len(keys)):
            rc = G.gvm_plain_run_noalloc(G.GVM_K_EP, d_in.value + 16 * i, d_out.value + 96 * i, 1)
            assert rc == 0, G.gvm_last_error()
        assert h.hipDeviceSynchronize() == 0
        assert h.hipMemcpy(out.ctypes.data, d_out, out.nbytes, D2H) == 0
    finally:
        h.hipFree(d_in)
        h.hipFree(d_out)
    xy = np.array([oe.ep_uniform_pairs(k, 1) for k in keys])[:, :, 0]
    t = xy[:, 0] * xy[:, 0] + xy[:, 1] * xy[:, 1]
    ok = (t > 0) & (t <= 1)
    assert (out[~ok, :2] == 0).all() and ok.sum() > 7000
    tl = t[ok].astype(np.longdouble)
    want = xy[ok].astype(np.longdouble) * np.sqrt(-2 * np.log(tl) / tl)[:, None]
    err = ((out[ok, :2] - want) / want * np.longdouble(2) ** 53).astype(np.float64)
    rms, worst = np.sqrt(np.mean(err ** 2)), np.abs(err).max()
    print(f"error of X and Y, 2^-53: rms {rms:.4f} max {worst:.3f}")
    assert rms <= 0.671 and worst <= 3.0, (rms, worst)
