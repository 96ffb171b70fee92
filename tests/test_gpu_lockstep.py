"""Batches in lockstep (a launch per stage over all plans): the proofs equal the
plain launches' and the persistent kernel's, for plans that have not begun next
to plans that an earlier run with a limit began or finished, for layers on
either side of the wide rounds' limit, and when captured in a HIP graph.
"""
import pytest

import gkr_synth as gs
from test_gpu_batch import MIX, _Job, _mix, gkr  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def _specs():
    mk = lambda d, n, sig, seed: gs.CircuitSpec(depth=d, log_copies=n, log_sub_width=sig, mu=(1, 2), seed=seed)
    # 2^13 and 2^14 pairs in the first rounds, from copies, sub-circuits and both
    return [mk(2, 0, (14, 14, 15), 21), mk(2, 14, (0, 1, 0), 22), mk(2, 7, (7, 8, 7), 23)]


def _plain(gkr, j):
    import torch
    keep = j.proof.clone(), j.out.clone()
    j.proof.zero_()
    j.out.zero_()
    gkr.prove_circuit(j.c, j.d_in, j.spec.seed, j.out, j.proof, j.ws)
    torch.cuda.synchronize()
    same = torch.equal(j.proof, keep[0]) and torch.equal(j.out, keep[1])
    return same


@pytest.mark.parametrize("begun", [0, 1, 40, 100000], ids=["none", "one-step", "forty-steps", "finished"])
def test_fresh_and_begun_plans_in_one_run(gkr, begun):  # noqa: F811
    import torch
    jobs = _mix(gkr)
    plans = [gkr.Plan(j.job) for j in jobs]
    ctl = torch.zeros(4, dtype=torch.int32, device="cuda")
    left = len(plans)
    if begun:
        gkr.run_batch(plans[::2], ctl, step_budget=begun)
        torch.cuda.synchronize()
        left -= int(ctl[0])
    gkr.run_batch(plans, ctl)
    torch.cuda.synchronize()
    assert int(ctl[0]) == left
    assert all(d == t for d, t in (p.progress() for p in plans))
    gkr.run_batch(plans, ctl)  # nothing is left
    torch.cuda.synchronize()
    assert int(ctl[0]) == 0
    for j in jobs:
        assert j.proof_bytes() == j.oracle_bytes(), j.spec


def test_lockstep_persistent_and_plain_agree_around_the_wide_limit(gkr):  # noqa: F811
    import torch
    jobs = [_Job(gkr, s) for s in _specs()]
    plans = [gkr.Plan(j.job) for j in jobs]
    ctl = torch.zeros(4, dtype=torch.int32, device="cuda")
    for wg in (-1, 192):
        for j, p in zip(jobs, plans):
            j.proof.zero_()
            p.reset()
        gkr.run_batch(plans, ctl, workgroups=wg)
        torch.cuda.synchronize()
        assert int(ctl[0]) == len(jobs)
        for j in jobs:
            assert _plain(gkr, j), (wg, j.spec)


def test_captured_lockstep_run_replays(gkr):  # noqa: F811
    import torch
    jobs = _mix(gkr)[:4]
    plans = [gkr.Plan(j.job) for j in jobs]
    want = [j.oracle_bytes() for j in jobs]
    ctl = torch.zeros(4, dtype=torch.int32, device="cuda")
    stream = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(g, stream=stream):
            for p in plans:
                p.reset(stream=stream)
            gkr.run_batch(plans, ctl, stream=stream)
    torch.cuda.synchronize()
    for rep in range(3):
        for j in jobs:
            j.proof.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert int(ctl[0]) == len(jobs)
        assert [j.proof_bytes() for j in jobs] == want, rep
        assert _plain(gkr, jobs[0])
