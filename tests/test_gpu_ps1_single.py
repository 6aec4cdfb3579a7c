"""One request under PS-1 on the GPU: its copy-in, kernel and copy-out run as the
policy's phases, on the copy FIFOs and the rank's stream, and not as PS-2's chain
on one stream.  Seen from outside by the device phase: it spans the dependencies
between three queues (about 10 us each on this machine), where a small request's
chain has none."""

import statistics

import pytest

from paper_1511_07658_amd import gvm as G
from paper_1511_07658_amd import spmd

pytestmark = pytest.mark.gpu
WARM, REPS = 4, 24


def waits(ns, policy, kernel, n):
    """Median device phase of a request less its copies and kernel, us."""
    cfg = G.gvm_config_default(nranks=1, shm_bytes_per_rank=4 << 20, hbm_budget_bytes=64 << 20, policy=policy,
                               batch_timing=1, name=ns)
    G.check(G.gvm_init(cfg), "gvm_init")
    try:
        G.check(G.gvm_attach_ns(ns, 0), "attach")
        ni, no = G.in_elems(kernel, n), G.out_elems(kernel, n)
        view = G.gvm_rank_buffer(0, (ni + no) * 4)
        view[:ni] = spmd.make_input(kernel, 71, 0, n)
        for _ in range(WARM + REPS):
            t = G.check(G.gvm_submit(0, kernel, view[:ni], view[ni:ni + no], n), "submit")
            G.check(G.gvm_wait(0, t, 60_000_000_000), "wait")
        G.check(G.gvm_detach(0), "detach")
        tm = G.gvm_stats_json()["timing"]
    finally:
        G.gvm_shutdown()
    parts = [tm[k][WARM:] for k in ("batch_device_us", "h2d_us", "launch_us", "d2h_us")]
    assert all(len(p) == REPS for p in parts), tm
    span, *work = (statistics.median(p) for p in parts)
    return span - sum(work)


@pytest.mark.parametrize("kernel,n", [(G.GVM_K_VECADD, 4096), (G.GVM_K_EP, 1 << 15)])
def test_one_request_runs_as_phases(ns_name, kernel, n):
    ps1 = waits(ns_name + ".1", G.GVM_POLICY_PS1, kernel, n)
    ps2 = waits(ns_name + ".2", G.GVM_POLICY_PS2, kernel, n)
    print(f"waits in the device phase: PS-1 {ps1:.1f} us, PS-2 {ps2:.1f} us")
    assert ps1 > ps2 + 8.0, (ps1, ps2)
