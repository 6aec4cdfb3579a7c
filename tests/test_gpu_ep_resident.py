"""EP-like requests through the manager, whose input comes with the launch and
whose result the kernel writes to the staging: fresh results every step, and a
request on the resident input after one with a copy, in every policy."""

import threading

import numpy as np
import pytest

from oracle import ep as oe
from paper_1511_07658_amd import gvm as G
from paper_1511_07658_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [G.GVM_MODE_BATCH, G.GVM_MODE_SERVING])
@pytest.mark.parametrize("policy", [G.GVM_POLICY_PS1, G.GVM_POLICY_PS2, G.GVM_POLICY_GROUPED])
def test_fresh_keys_and_resident_input(ns_name, mode, policy):
    nr, steps = 3, 6
    sizes = [1, 1025, 70001]   # one unit, two, many
    cfg = G.gvm_config_default(nranks=nr, shm_bytes_per_rank=1 << 20, hbm_budget_bytes=64 << 20, mode=mode,
                               policy=policy, batch_window_us=10_000_000, name=ns_name)
    G.check(G.gvm_init(cfg), "gvm_init")
    errors = []
    bar = threading.Barrier(nr)

    def same(r, step, what, out, key):
        got, ref = wl.ep_result(out), oe.ep_reference(key, sizes[r])
        eps = np.finfo(np.float64).eps
        if not np.array_equal(got["q"], ref["q"]) or any(
                abs(got[s] - ref[s]) > 256 * eps * ref[a] for s, a in (("sx", "abs_x"), ("sy", "abs_y"))):
            errors.append((r, step, what))

    def rank(r):
        try:
            G.check(G.gvm_attach_ns(ns_name, r), "attach")
            bar.wait()
            out = np.zeros(24, np.float32)
            for step in range(steps):
                key = wl.ep_key(85, r, step)
                t = G.check(G.gvm_submit(r, G.GVM_K_EP, wl.ep_request(key), out, sizes[r]), "submit")
                G.check(G.gvm_wait(r, t, 60_000_000_000), "wait")
                same(r, step, "copied", out, key)
                out[:] = 0
                t = G.check(G.gvm_submit_ex(r, G.GVM_K_EP, None, out, sizes[r], G.GVM_F_IN_RESIDENT), "resident")
                G.check(G.gvm_wait(r, t, 60_000_000_000), "wait")
                same(r, step, "resident", out, key)
                out[:] = 0
            G.check(G.gvm_detach(r), "detach")
        except Exception as e:
            errors.append((r, repr(e)))
            bar.abort()

    ths = [threading.Thread(target=rank, args=(r,)) for r in range(nr)]
    [t.start() for t in ths]
    [t.join() for t in ths]
    G.gvm_shutdown()
    assert not errors, errors
