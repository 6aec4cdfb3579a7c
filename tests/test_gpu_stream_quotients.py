"""Options at the edges of the fast quotients on the GPU: S / K on both sides of
the float range with S and K far inside it, and expiries whose reciprocal root,
divided by the volatility, leaves it.

Against the binary64 formula, within 1e-5 of the larger of S and K (the scale
of the two terms whose difference a price is): each term carries the 7.5e-8 of
the distribution's polynomial and some ten roundings of 6e-8."""

import numpy as np
import pytest

from oracle import kernels as ok
from paper_1511_07658_amd import gvm as G
from paper_1511_07658_amd import workloads as wl
from test_gpu_stream_edges import run

pytestmark = pytest.mark.gpu


def check(S, K, T, vol):
    S, K, T = (np.asarray(x, np.float32) for x in (S, K, T))
    with np.errstate(all="ignore"):
        want = ok.black_scholes_f64(S, K, T, float(np.float32(0.02)), float(np.float32(vol)))
    got = run(G.GVM_K_BLACKSCHOLES, S.size, wl.pack_request(2, S, K, T), vol=vol)
    scale = np.maximum(S, K).astype(np.float64)
    for g, w in zip((got[:S.size], got[S.size:]), want):
        bad = ~(np.abs(g - w) <= 1e-5 * scale + 2e-38)
        assert not bad.any(), [(S[i], K[i], T[i], g[i], w[i]) for i in np.flatnonzero(bad)[:5]]


@pytest.mark.parametrize("n", [1, 4, 7])   # remainder, float4, both
def test_quotients_around_the_float_range(n):
    exps = [-120, -100, -64, -61, -60, -59, -28, 0, 28, 59, 60, 61, 64, 67, 100, 120]
    pairs = [(2.0 ** s, 2.0 ** k) for s in exps for k in exps] + [(1e20, 1e-20), (1e29, 1e-10), (1e-20, 1e20)]
    for at in range(0, len(pairs), 64):
        S, K = zip(*pairs[at:at + 64])
        for i in range(0, len(S), 16 * n):
            check(S[i:i + n], K[i:i + n], np.full(len(S[i:i + n]), 2.0), 0.3)
        check(S, K, np.full(len(S), 2.0), 0.3)


@pytest.mark.parametrize("vol", [0.3, 2.0 ** -59, 2.0 ** 59])
def test_expiries_down_to_the_smallest(vol):
    # an expiry this short leaves the payoff: out of the money, where the root
    # may be infinite (below the normal range), and in it
    small = [2.0 ** e for e in (-149, -140, -127)]
    normal = [2.0 ** e for e in (-126, -100, -61, -60, -59, -30)]
    if vol < 1.0:
        check([20.0] * 9, [30.0] * 9, small + normal, vol)
        check([30.0] * 6, [20.0] * 6, normal, vol)
    else:  # vol sqrt(T) is large again: the call is the spot, or near it
        check([20.0] * 2, [30.0] * 2, [2.0 ** -100, 2.0 ** -60], vol)
