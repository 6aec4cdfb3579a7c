"""Streaming kernels on both sides of the lines where their loads change: all
inputs cached up to 96 MiB of them, the last operand alone up to 96 MiB of it,
none beyond.  Vectors exact; options have the bits of a short request."""

import numpy as np
import pytest

from paper_1511_07658_amd import gvm as G
from paper_1511_07658_amd import workloads as wl
from test_gpu_stream_edges import run

pytestmark = pytest.mark.gpu
MIB96 = (96 << 20) // 4   # floats


@pytest.mark.parametrize("n", [MIB96 // 2, MIB96 // 2 + 1, MIB96, MIB96 + 1])
def test_vectors(n):
    a, b = wl.vecadd_inputs(93, 0, n)
    assert np.array_equal(run(G.GVM_K_VECADD, n, wl.pack_request(1, a, b), offset=n % 4), a + b)


@pytest.mark.parametrize("n", [MIB96 // 3, MIB96 // 3 + 1, MIB96, MIB96 + 1])
def test_options(n):
    m = 5003
    S, K, T = wl.bs_inputs(93, 1, m)
    short = run(G.GVM_K_BLACKSCHOLES, m, wl.pack_request(2, S, K, T))
    x = [np.resize(v, n) for v in (S, K, T)]
    out = run(G.GVM_K_BLACKSCHOLES, n, wl.pack_request(2, *x))
    assert np.array_equal(out[:n], np.resize(short[:m], n)) and np.array_equal(out[n:], np.resize(short[m:], n))
