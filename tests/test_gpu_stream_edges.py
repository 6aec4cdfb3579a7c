"""Streaming kernels on the GPU where a launch can go wrong: lengths around
the float4 and the work unit, operands that start at any float, and options
whose operands the fast quotient does not serve."""

import ctypes

import numpy as np
import pytest

from oracle import kernels as ok
from paper_1511_07658_amd import gvm as G
from paper_1511_07658_amd import workloads as wl
from test_zz_no_alloc import D2H, H2D, hip

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 4, 5, 7, 1023, 2047, 2048, 2049, 2051, 4097, 65537]


def run(kernel, n, x, offset=0, rate=0.02, vol=0.3):
    """One request whose packed input and output start `offset` floats into
    their buffers; also checks that nothing around the output is written."""
    h = hip()
    nout = G.out_elems(kernel, n)
    xin = np.concatenate([np.full(offset, np.nan, np.float32), x])
    out = np.full(nout + offset + 4, np.nan, np.float32)
    d_in, d_out = ctypes.c_void_p(), ctypes.c_void_p()
    assert h.hipMalloc(ctypes.byref(d_in), xin.nbytes) == 0
    assert h.hipMalloc(ctypes.byref(d_out), out.nbytes) == 0
    try:
        assert h.hipMemcpy(d_in, xin.ctypes.data, xin.nbytes, H2D) == 0
        assert h.hipMemcpy(d_out, out.ctypes.data, out.nbytes, H2D) == 0
        rc = G.gvm_plain_run_noalloc(kernel, d_in.value + 4 * offset, d_out.value + 4 * offset, n, rate, vol)
        assert rc == 0, G.gvm_last_error()
        assert h.hipDeviceSynchronize() == 0
        assert h.hipMemcpy(out.ctypes.data, d_out, out.nbytes, D2H) == 0
    finally:
        h.hipFree(d_in)
        h.hipFree(d_out)
    assert np.isnan(out[:offset]).all() and np.isnan(out[offset + nout:]).all()
    return out[offset:offset + nout]


@pytest.mark.parametrize("offset", [0, 1, 3])
@pytest.mark.parametrize("n", SIZES)
def test_vectors_exact_at_any_start(n, offset):
    a, b = wl.vecadd_inputs(83, offset, n)
    x = wl.pack_request(1, a, b)
    assert np.array_equal(run(G.GVM_K_VECADD, n, x, offset), a + b)
    assert np.array_equal(run(G.GVM_K_VECMUL, n, x, offset), a * b)


@pytest.mark.parametrize("n", SIZES)
def test_options_have_the_same_bits_in_any_place(n):
    # options priced as part of a long request and as requests of their own,
    # every lane of a unit and the remainders included
    S, K, T = wl.bs_inputs(83, 0, 4096 + 65537)
    whole = run(G.GVM_K_BLACKSCHOLES, S.size, wl.pack_request(2, S, K, T))
    at = 1001
    part = run(G.GVM_K_BLACKSCHOLES, n, wl.pack_request(2, S[at:at + n], K[at:at + n], T[at:at + n]), offset=n % 4)
    call, put = whole[:S.size], whole[S.size:]
    assert np.array_equal(part[:n].view(np.uint32), call[at:at + n].view(np.uint32))
    assert np.array_equal(part[n:].view(np.uint32), put[at:at + n].view(np.uint32))


def test_extreme_options():
    # strikes and spots far outside the usual range beside ordinary ones, all
    # against the binary64 formula: within 1e-5 of the larger of S and K, the
    # scale of the two terms whose difference a price is
    vals = [0.0, 1e-42, 1e-38, 1e-31, 1e-3, 1.0, 30.0, 1e5, 1e29, 3e30, 1e38]
    S, K = (np.array(v, np.float32) for v in zip(*[(s, k) for s in vals for k in vals if s or k]))
    T = np.full(S.size, 2.0, np.float32)
    with np.errstate(all="ignore"):
        call, put = ok.black_scholes_f64(S, K, T, float(np.float32(0.02)), float(np.float32(0.3)))
    got = run(G.GVM_K_BLACKSCHOLES, S.size, wl.pack_request(2, S, K, T))
    scale = np.maximum(S, K).astype(np.float64)
    for g, want in ((got[:S.size], call), (got[S.size:], put)):
        fine = np.isfinite(want)
        assert (np.abs(g[fine] - want[fine]) <= 1e-5 * scale[fine] + 2e-38).all()
    # NaN stays NaN, an infinite strike gives no call, and the neighbours of
    # either keep their prices
    S, K, T = wl.bs_inputs(84, 0, 64)
    base = run(G.GVM_K_BLACKSCHOLES, 64, wl.pack_request(2, S, K, T))
    K2, S2 = K.copy(), S.copy()
    K2[5], S2[9] = np.inf, np.nan
    odd = run(G.GVM_K_BLACKSCHOLES, 64, wl.pack_request(2, S2, K2, T))
    keep = np.array([i not in (5, 9) for i in range(64)])
    for half in (slice(0, 64), slice(64, 128)):
        assert np.array_equal(odd[half][keep], base[half][keep])
        assert np.isnan(odd[half][9])
    assert not odd[5] > 0.0


def test_zero_volatility_is_the_discounted_payoff():
    S = np.array([5.0, 30.0, 20.0], np.float32)
    K = np.array([30.0, 5.0, 10.0], np.float32)
    T = np.array([1.0, 2.0, 0.5], np.float32)
    got = run(G.GVM_K_BLACKSCHOLES, 3, wl.pack_request(2, S, K, T), vol=0.0)
    kd = K * np.exp(-np.float32(0.02) * T)
    assert np.allclose(got[:3], np.maximum(S - kd, 0), rtol=1e-5, atol=1e-5)
    assert np.allclose(got[3:], np.maximum(kd - S, 0), rtol=1e-5, atol=1e-5)
