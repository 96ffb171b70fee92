"""The persistent batch kernel at size. A run to the end on the whole device may go in
lockstep launches, so these runs name a count of workgroups, for which the
persistent kernel always runs alone (one launch, counted): the 64 uneven jobs
against the oracle's digests, the largest serving jobs (hundreds of tiles per step
on every XCD, whose partial sums, counters and tables cross them) against the plain
launches and the verifier, and the small mix against the oracle. Both batch
forms run the large jobs."""
import hashlib
import json
import os

import numpy as np
import pytest

import gkr_synth as gs
from test_gpu_batch import HERE, _Job, _mix, gkr  # noqa: F401 (fixture)
from test_gpu_batch_forms import _batch_launches

pytestmark = pytest.mark.gpu


def _cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def _run(gkr, jobs, plans, workgroups):
    """One run from the start; the launches it took."""
    import torch
    ctl = torch.zeros(4, dtype=torch.int32, device="cuda")
    for j, p in zip(jobs, plans):
        j.proof.zero_()
        j.out.zero_()
        p.reset()
    print("batch: %d jobs, workgroups %d" % (len(jobs), workgroups), flush=True)
    launches = _batch_launches(gkr, lambda: gkr.run_batch(plans, ctl, workgroups=workgroups))
    assert int(ctl[0]) == len(jobs) and int(ctl[2]) == sum(p.progress()[1] for p in plans)
    return launches


@pytest.mark.parametrize("share", [1, 2], ids=["per-cu", "per-two-cus"])
def test_uneven_batch_of_64_matches_the_oracle(gkr, share):  # noqa: F811
    with open(os.path.join(HERE, "golden", "c4_batch.json")) as f:
        gold = json.load(f)["jobs"]
    jobs = [_Job(gkr, s) for s in gs.batch_jobs_c4()]
    plans = [gkr.Plan(j.job) for j in jobs]
    assert _run(gkr, jobs, plans, _cus() // share) == 1
    for k, j in enumerate(jobs):
        outs = np.ascontiguousarray(gkr.host_elements(j.out))
        assert hashlib.sha256(outs.tobytes()).hexdigest() == gold[k]["outputs_sha256"], k
        assert hashlib.sha256(j.proof_bytes()).hexdigest() == gold[k]["proof_sha256"], k


def test_large_jobs_match_plain_and_verify_in_both_forms(gkr):  # noqa: F811
    import torch
    specs = gs.serving_jobs_c5(96)
    big = sorted(range(len(specs)), key=lambda k: (-specs[k].gate_layers, k))[:16]
    jobs = [_Job(gkr, specs[k]) for k in big]
    plans = [gkr.Plan(j.job) for j in jobs]
    want = []
    for j in jobs:
        gkr.prove_circuit(j.c, j.d_in, j.spec.seed, j.out, j.proof, j.ws)
        torch.cuda.synchronize()
        want.append((j.proof_bytes(), np.ascontiguousarray(gkr.host_elements(j.out)).copy()))
    for workgroups in (_cus(), 0):
        launches = _run(gkr, jobs, plans, workgroups)
        assert launches == 1 if workgroups else launches > 50
        for k, j, (proof, outs) in zip(big, jobs, want):
            assert j.proof_bytes() == proof, (workgroups, k, j.spec)
            assert np.array_equal(gkr.host_elements(j.out), outs), (workgroups, k, j.spec)
    for j, (proof, outs) in list(zip(jobs, want))[:4]:
        assert gkr.verify(j.c, j.inputs, outs, j.spec.seed, proof) == 1, j.spec


@pytest.mark.parametrize("workgroups", [1, 7, 512])
def test_mix_matches_the_oracle(gkr, workgroups):  # noqa: F811
    jobs = _mix(gkr)
    plans = [gkr.Plan(j.job) for j in jobs]
    assert _run(gkr, jobs, plans, workgroups) == 1
    for j in jobs:
        assert j.proof_bytes() == j.oracle_bytes(), j.spec
