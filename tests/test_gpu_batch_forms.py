"""Which form a run to the end on the whole device takes (a launch per stage, or one
persistent launch), read off the launch counts, and the lockstep form over small
and odd plans: beside a plan whose steps are large enough to choose it, the mix of
test_gpu_batch gives the oracle's proofs, with plans begun before, and in a graph."""
import ctypes

import pytest

import gkr_synth as gs
from test_gpu_batch import _Job, _mix, gkr  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


class _Entry(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char * 32), ("launches", ctypes.c_uint64), ("ms", ctypes.c_double),
                ("bytes", ctypes.c_double), ("mulmods", ctypes.c_double)]


def _batch_launches(gkr, call):
    """Launches of the batch kernels during call()."""
    import torch
    lib, arr, n = gkr.lib(), (_Entry * 32)(), ctypes.c_uint32(0)
    torch.cuda.synchronize()
    assert lib.gkr_profile_enable(1) == 0
    try:
        call()
        torch.cuda.synchronize()
        assert lib.gkr_profile_read(arr, 32, ctypes.byref(n)) == 0
    finally:
        lib.gkr_profile_enable(0)
    return {e.name: e.launches for e in arr[:n.value]}.get(b"batch", 0)


def _spec(depth, copies, width, seed):
    return gs.CircuitSpec(depth=depth, log_copies=copies, log_sub_width=(width,) * (depth + 1), mu=(1, 2), seed=seed)


LARGE = _spec(3, 4, 16, 41)
FORMS = {
    "few small uneven plans": ([_spec(9, 2, 8, 1), _spec(4, 5, 6, 2), _spec(12, 0, 11, 3), _spec(7, 4, 9, 4)], False),
    "one plan": ([_spec(3, 2, 8, 5)], True),
    "plans of one shape": ([_spec(3, 2, 8, s) for s in (6, 7, 8)], True),
    "small plans beside a large one": ([_spec(9, 2, 8, 9), _spec(4, 5, 6, 10), LARGE], True),
    "large uneven plans": ([_spec(3, 4, 14, 11), _spec(5, 7, 10, 12)], True),
}


@pytest.mark.parametrize("name", list(FORMS))
def test_form_of_a_run_follows_the_plans(gkr, name):  # noqa: F811
    import torch
    specs, lockstep = FORMS[name]
    jobs = [_Job(gkr, s) for s in specs]
    plans = [gkr.Plan(j.job) for j in jobs]
    ctl = torch.zeros(4, dtype=torch.int32, device="cuda")
    print("batch form: %s" % name, flush=True)
    for wg in (-1, 0):
        for p in plans:
            p.reset()
        launches = _batch_launches(gkr, lambda: gkr.run_batch(plans, ctl, workgroups=wg))
        assert int(ctl[0]) == len(plans)
        assert launches > 50 if lockstep else launches == 1, (wg, launches)
    for j in jobs:
        got = j.proof_bytes()
        j.proof.zero_()
        gkr.prove_circuit(j.c, j.d_in, j.spec.seed, j.out, j.proof, j.ws)
        torch.cuda.synchronize()
        assert j.proof_bytes() == got, j.spec


@pytest.mark.parametrize("begun", [0, 40], ids=["none-begun", "some-begun"])
def test_small_and_odd_plans_in_lockstep(gkr, begun):  # noqa: F811
    import torch
    jobs = _mix(gkr) + [_Job(gkr, LARGE)]
    plans = [gkr.Plan(j.job) for j in jobs]
    ctl = torch.zeros(4, dtype=torch.int32, device="cuda")
    left = len(plans)
    if begun:
        gkr.run_batch(plans[:8:2], ctl, step_budget=begun)
        torch.cuda.synchronize()
        left -= int(ctl[0])
    print("batch: the mix in lockstep beside a large plan", flush=True)
    assert _batch_launches(gkr, lambda: gkr.run_batch(plans, ctl)) > 50
    assert int(ctl[0]) == left
    assert all(d == t for d, t in (p.progress() for p in plans))
    for j in jobs[:-1]:
        assert j.proof_bytes() == j.oracle_bytes(), j.spec


def test_captured_lockstep_run_of_the_mix_replays(gkr):  # noqa: F811
    import torch
    jobs = _mix(gkr)[:4] + [_Job(gkr, LARGE)]
    plans = [gkr.Plan(j.job) for j in jobs]
    want = [j.oracle_bytes() for j in jobs[:-1]]
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
        assert [j.proof_bytes() for j in jobs[:-1]] == want, rep
        gkr.prove_circuit(jobs[0].c, jobs[0].d_in, jobs[0].spec.seed, jobs[0].out, jobs[0].proof, jobs[0].ws)
        torch.cuda.synchronize()
        assert jobs[0].proof_bytes() == want[0], rep


@pytest.mark.parametrize("specs", [[LARGE], [LARGE, _spec(5, 7, 10, 12)]], ids=["one", "two"])
def test_begun_and_finished_plans_take_one_launch(gkr, specs):  # noqa: F811
    """Plans taken by a run since their last reset: only those that have not begun are worth
    the launches of a lockstep run."""
    import torch
    jobs = [_Job(gkr, s) for s in specs]
    plans = [gkr.Plan(j.job) for j in jobs]
    ctl = torch.zeros(4, dtype=torch.int32, device="cuda")
    for j in jobs:
        gkr.prove_circuit(j.c, j.d_in, j.spec.seed, j.out, j.proof, j.ws)
    torch.cuda.synchronize()
    want = [j.proof_bytes() for j in jobs]
    for begun in (plans, plans[:1]):
        for j, p in zip(jobs, plans):
            j.proof.zero_()
            p.reset()
        gkr.run_batch(begun, ctl, step_budget=5)
        launches = _batch_launches(gkr, lambda: gkr.run_batch(plans, ctl))
        assert launches == 1 if len(begun) == len(plans) else launches > 50, launches
        assert int(ctl[0]) == len(plans)
        assert [j.proof_bytes() for j in jobs] == want
        assert _batch_launches(gkr, lambda: gkr.run_batch(plans, ctl)) == 1
        assert int(ctl[0]) == 0
    plans[-1].reset()
    assert _batch_launches(gkr, lambda: gkr.run_batch(plans, ctl)) > 50
    assert int(ctl[0]) == 1 and [j.proof_bytes() for j in jobs] == want
