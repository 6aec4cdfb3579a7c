"""EP-like tally on the GPU where the cut into units can go wrong: sizes
around one unit, one record and whole multiples of the units, against the
oracle (counts equal; sums within the rounding of their terms: the kernel adds
at most 64 terms per thread and 14 levels of partial sums, and each term
carries a few roundings, so 128 eps of the sum of magnitudes is ample)."""

import numpy as np
import pytest

from oracle import ep as oe
from paper_1511_07658_amd import gvm as G
from paper_1511_07658_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 1023, 1024, 1025, 2049, 32769, 89 * 1024, 89 * 1024 + 1, 1 << 20, 3000001])
def test_units_of_one_request(n):
    key = wl.ep_key(82, 0, n)
    out = np.empty(24, np.float32)
    rc, _ = G.gvm_plain_run(G.GVM_K_EP, wl.ep_request(key), out, n)
    assert rc == 0, G.gvm_last_error()
    got, ref = wl.ep_result(out), oe.ep_reference(key, n)
    assert np.array_equal(got["q"], ref["q"])
    for s, a in (("sx", "abs_x"), ("sy", "abs_y")):
        assert abs(got[s] - ref[s]) <= 128 * np.finfo(np.float64).eps * ref[a]
