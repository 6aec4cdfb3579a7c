"""The sum of a tally's records at its dispatch edges: 64 records (one wave) and
65 (eight waves) against the oracle, and a request of few records summed beside
one of many in the same launch: the same bits as alone.  Sums within 128 eps of
the sum of magnitudes (at most 64 terms per thread and 14 levels above them)."""

import threading

import numpy as np
import pytest

from oracle import ep as oe
from paper_1511_07658_amd import gvm as G
from paper_1511_07658_amd import workloads as wl

pytestmark = pytest.mark.gpu


def plain(key, n):
    out = np.empty(24, np.float32)
    rc, _ = G.gvm_plain_run(G.GVM_K_EP, wl.ep_request(key), out, n)
    assert rc == 0, G.gvm_last_error()
    return out


@pytest.mark.parametrize("records", [2, 63, 64, 65, 88])
def test_records_around_a_wave(records):
    n = records * 1024 - 3
    key = wl.ep_key(91, 0, n)
    got, ref = wl.ep_result(plain(key, n)), oe.ep_reference(key, n)
    assert np.array_equal(got["q"], ref["q"])
    for s, a in (("sx", "abs_x"), ("sy", "abs_y")):
        assert abs(got[s] - ref[s]) <= 128 * np.finfo(np.float64).eps * ref[a]


def test_few_records_beside_many(ns_name):
    sizes = [1, 5000, 64 * 1024, 3000001]
    cfg = G.gvm_config_default(nranks=len(sizes), shm_bytes_per_rank=1 << 20, hbm_budget_bytes=64 << 20,
                               policy=G.GVM_POLICY_GROUPED, batch_window_us=10_000_000, name=ns_name)
    G.check(G.gvm_init(cfg), "gvm_init")
    outs, errors = [np.zeros(24, np.float32) for _ in sizes], []

    def rank(r):
        try:
            G.check(G.gvm_attach_ns(ns_name, r), "attach")
            t = G.check(G.gvm_submit(r, G.GVM_K_EP, wl.ep_request(wl.ep_key(92, r, 0)), outs[r], sizes[r]), "submit")
            G.check(G.gvm_wait(r, t, 60_000_000_000), "wait")
            G.check(G.gvm_detach(r), "detach")
        except Exception as e:
            errors.append((r, repr(e)))

    ths = [threading.Thread(target=rank, args=(r,)) for r in range(len(sizes))]
    [t.start() for t in ths]
    [t.join() for t in ths]
    G.gvm_shutdown()
    assert not errors, errors
    for r, n in enumerate(sizes):
        assert outs[r].tobytes() == plain(wl.ep_key(92, r, 0), n).tobytes(), n
