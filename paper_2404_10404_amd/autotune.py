"""Autotuner of the round schedule and the batch launch shape.

Tunables (none of them changes proof bytes):
  tail_log          a phase finishes in one workgroup once its tables have at
                    most 2^tail_log entries (below that, a grid-wide round costs
                    more in launch and Fiat-Shamir latency than it saves). Plain
                    BN254 proofs stop at 2^7 and lockstep batches at 2^2, so it is
                    the persistent batch kernel that it is tuned on (Goldilocks
                    proofs take three more, up to 2^12)
  max_round_blocks  cap on the workgroups of a grid-wide round (more tiles:
                    more parallel partial sums for the last tile to add)
  pairs_per_thread  a grid-wide round gets ceil(pairs / (256 x this)) workgroups
                    (fewer, longer-lived workgroups for mid-size rounds)
  batch_workgroups  resident workgroups of the persistent batch kernel

The tuner times whole proofs of the given workloads for every setting of the
rounds on a grid, scores a setting by the sum over workloads of its time divided
by that workload's best time on the grid and keeps the setting with the least
score, or the one in use if that is within half a percent; with c4 among the workloads it then times the persistent kernel on the 64
uneven jobs for every tail and count of workgroups. It writes the grids and the
choice to a JSON cache (default: tuning.json next to this file).
`load()` applies a cached choice; the binding calls it on first use when the
cache exists.

    python -m paper_2404_10404_amd.autotune [--workloads c2,c3,c4] [--reps 3]
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
CACHE = os.path.join(HERE, "tuning.json")


def load(path: str = CACHE) -> dict | None:
    """Apply the cached tuning (if any); returns the cache record."""
    if not os.path.exists(path):
        return None
    with open(path) as f:
        rec = json.load(f)
    from . import gkr
    best = rec.get("best", {})
    if "tail_log" in best and "max_round_blocks" in best:
        gkr.set_tuning(int(best["tail_log"]), int(best["max_round_blocks"]), int(best.get("pairs_per_thread", 1)))
    return rec


def _plain_workload(gkr, spec):
    import gkr_synth as gs
    c = gkr.Circuit.from_synth(spec, gs.make_wiring(spec))
    prover = gkr.Prover(c)
    d_in = gkr.device_elements(gs.make_inputs(spec))
    return lambda: prover.prove(d_in, spec.seed)


def _time(fn, reps):
    import torch
    fn()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        fn()
    torch.cuda.synchronize()
    return (time.perf_counter() - t0) / reps


def _choose(grid, key, in_use):
    """The least entry, or the least one in use if it is within half a percent."""
    best = min(grid, key=lambda g: g[key])
    near = [g for g in grid if in_use(g) and g[key] <= 1.005 * best[key]]
    return min(near, key=lambda g: g[key]) if near else best


def tune(workloads=("c2",), tail_logs=(7, 8, 9, 10, 11), blocks=(512, 1024, 2048, 4096), ppts=(1, 2, 4),
         reps=3, path: str = CACHE) -> dict:
    import torch

    import gkr_synth as gs
    from . import gkr
    specs = {"c1": gs.plain_c1, "c2": gs.data_parallel_c2, "c3": gs.worker_share_c3}
    fns = {w: _plain_workload(gkr, specs[w]()) for w in workloads if w in specs}
    tail_log, now_mb, now_ppt = gkr.get_tuning()
    grid = []
    for mb in blocks:
        for ppt in ppts:
            gkr.set_tuning(tail_log, mb, ppt)
            times = {w: _time(fn, reps) for w, fn in fns.items()}
            grid.append({"max_round_blocks": mb, "pairs_per_thread": ppt, "seconds": times})
            print("max_round_blocks %4d  pairs_per_thread %d  %s"
                  % (mb, ppt, {k: round(v * 1e3, 3) for k, v in times.items()}), flush=True)
    best_t = {w: min(g["seconds"][w] for g in grid) for w in fns}
    for g in grid:
        g["score"] = sum(g["seconds"][w] / best_t[w] for w in fns)
    best = _choose(grid, "score", lambda g: (g["max_round_blocks"], g["pairs_per_thread"]) == (now_mb, now_ppt))
    rec = {"device": torch.cuda.get_device_name(0), "workloads": list(fns), "reps": reps, "grid": grid,
           "best": {"tail_log": tail_log, "max_round_blocks": best["max_round_blocks"],
                    "pairs_per_thread": best["pairs_per_thread"]}}
    if "c4" in workloads:
        rec["batch"] = tune_batch(gkr, reps, tail_logs, best["max_round_blocks"], best["pairs_per_thread"])
        rec["best"]["tail_log"] = rec["batch"]["best"]["tail_log"]
        rec["best"]["batch_workgroups"] = rec["batch"]["best"]["workgroups"]
    gkr.set_tuning(rec["best"]["tail_log"], best["max_round_blocks"], best["pairs_per_thread"])
    with open(path, "w") as f:
        json.dump(rec, f, indent=1)
    return rec


def tune_batch(gkr, reps, tail_logs, blocks, ppt) -> dict:
    """Tail and resident workgroups of the persistent kernel for the uneven 64-job batch."""
    import torch

    import gkr_synth as gs
    jobs, keep = [], []
    for spec in gs.batch_jobs_c4():
        c = gkr.Circuit.from_synth(spec, gs.make_wiring(spec))
        d_in = gkr.device_elements(gs.make_inputs(spec))
        out = torch.zeros((1 << c.s(0), 8), dtype=torch.int32, device="cuda")
        proof = gkr.alloc_bytes(c.proof_bytes)
        ws = gkr.alloc_bytes(c.workspace_bytes)
        keep.append((c, d_in, out, proof, ws))
        jobs.append(gkr.make_job(c, d_in, spec.seed, out, proof, ws))
    ctl = torch.zeros(4, dtype=torch.int32, device="cuda")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    now_tail = gkr.get_tuning()[0]
    res = []
    for tl in tail_logs:
        gkr.set_tuning(tl, blocks, ppt)
        plans = [gkr.Plan(job) for job in jobs]  # a plan keeps the tuning it was made under
        for wg in (cus // 4, cus // 2, (3 * cus) // 4, cus, (3 * cus) // 2, 2 * cus):
            def run():
                for p in plans:
                    p.reset()
                gkr.run_batch(plans, ctl, workgroups=wg)
            res.append({"tail_log": tl, "workgroups": wg, "seconds": _time(run, reps)})
            print("batch tail_log %2d  workgroups %4d  %.3f ms" % (tl, wg, res[-1]["seconds"] * 1e3), flush=True)
        for p in plans:
            p.close()
    best = _choose(res, "seconds", lambda r: r["tail_log"] == now_tail)
    return {"grid": res, "best": {"tail_log": best["tail_log"], "workgroups": best["workgroups"]}}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--workloads", default="c2,c3,c4")
    ap.add_argument("--reps", type=int, default=3)
    ap.add_argument("--out", default=CACHE)
    a = ap.parse_args()
    sys.path.insert(0, os.path.dirname(HERE))
    rec = tune(tuple(a.workloads.split(",")), reps=a.reps, path=a.out)
    print(json.dumps(rec["best"]))


if __name__ == "__main__":
    main()
