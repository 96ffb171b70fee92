// Batched proving: plans (a proof's step programs recorded in device memory) and
// their runs, in lockstep launches or by the persistent kernel.
//
// A plan is built once per job (allocating, synchronous). Running plans is
// asynchronous, allocates nothing and copies nothing between host and device:
// counters are cleared by a fill kernel and the job table travels in the
// kernel arguments, so a run can be captured in a HIP graph. A run that stops
// early (step budget, or stop-on-finish) leaves every plan at a step boundary
// or inside a partly claimed step; the next run continues from there.
#include <string.h>

#include <algorithm>
#include <atomic>
#include <memory>
#include <new>
#include <string>
#include <vector>

#include "gkr_kernels.hpp"
#include "gkr_program.hpp"
#include "gkr_tuning.hpp"

struct gkr_plan {
  gkr_job job;
  uint32_t nsteps = 0;
  void* dev = nullptr;  // steps, lockstep steps, then counters
  gkr::Step* steps = nullptr;
  uint32_t* ctr = nullptr;  // [0] current step, claimed and done tiles per step, then the lockstep flag
  size_t ctr_words = 0;
  // The lockstep program: its steps in device memory, and per stage (steps that
  // run together) the first step; per step the workgroups.
  gkr::Step* lock_steps = nullptr;
  std::vector<uint32_t> stage_first, lock_tiles;
  uint64_t gates = 0;  // gates of all layers and inputs
  uint64_t form = 0;   // hash of the lockstep program's step types
  // Queued in a run since the last reset. Only a hint for which launches to queue: the
  // device's counters say what is left to do (a reset may be replayed from a graph).
  std::atomic<bool> queued{false};
  uint32_t* flag() const { return ctr + ctr_words - 1; }
};

namespace gkr {
static bool aligned16b(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
}  // namespace gkr

using namespace gkr;

static BatchJobDev job_dev(const gkr_plan& p) {
  BatchJobDev j;
  memset(&j, 0, sizeof(j));
  j.steps = p.steps;
  j.ctr = p.ctr;
  j.nsteps = p.nsteps;
  return j;
}

// Whether a run to the end goes in lockstep: the smaller of two estimates, in ns.
// Lockstep: launches of the longest plan, waiting for the next longest one (each
// stage takes as long as its longest step, and uneven plans are at different
// points), a little per further plan's stage, and the gates of all. Persistent: the
// chain of the longest plan, a publication and a scan of the counters per step, and
// the gates, which pass through tiles. Fitted to 54 runs of 1..64 plans (2^10..2^20
// gates per layer, depth 2..32), 7 % off on average; the choice was never above the
// better form by more than 4 %. Lockstep / persistent, ms, with the persistent
// kernel that released its L2 for every tile in brackets:
//   16 plans of 2^10..2^13 gates, depth 2..12     9.1 /  6.6  [6.8]
//   uneven ones (2^10..2^18, depth 8..32):  4    17.1 / 14.6 [16.2]
//     8                                          24.0 / 19.8 [21.3]
//    16                                          28.8 / 25.5 [36.9]
//    32                                          36.1 / 34.2 [55.4]
//    48                                          46.0 / 56.0 [113.7]
//    64                                          58.9 / 82.1 [153.9]
//   6 of 2^12..2^20, depth 8..16                 21.5 / 33.1 [45.3]
// Plans with the same steps do not wait: one of 28 x 2^12 11.1 / 12.4 [13.3], one of
// 16 x 2^20 15.2 / 25.2 [30.3], two of 4 x 2^10 1.72 / 1.92 [2.59].
static bool lockstep_pays(gkr_plan* const* plans, uint32_t n) {
  double gates = 0, stages = 0, first = 0, second = 0, chain = 0;
  bool alike = true;
  for (uint32_t i = 0; i < n; ++i) {
    const double k = (double)(plans[i]->stage_first.size() - 1), g = (double)plans[i]->gates;
    gates += g;
    stages += k;
    second = std::max(second, std::min(first, k));
    first = std::max(first, k);
    chain = std::max(chain, 14000 * k + 0.30 * g);
    alike = alike && plans[i]->form == plans[0]->form;
  }
  const double lockstep = 12400 * first + 5500 * second + 400 * (stages - first) + 0.34 * gates;
  return alike || lockstep < chain + 0.78 * gates;
}

// The lockstep run of those of the n plans that have not begun: a launch decides
// which they are, then one launch per stage, then one that marks them finished.
static void run_lockstep(gkr_plan* const* plans, uint32_t n, uint32_t* d_ctl, hipStream_t s) {
  uint32_t* flags[kMaxBatchJobs];
  size_t stages = 0;
  BatchArgs a;
  memset(&a, 0, sizeof(a));
  a.njobs = n;
  a.ctl = d_ctl;
  for (uint32_t i = 0; i < n; ++i) {
    a.jobs[i] = job_dev(*plans[i]);
    flags[i] = plans[i]->flag();
    stages = std::max(stages, plans[i]->stage_first.size() - 1);
  }
  launch_lock_begin(a, flags, s);
  LockArgs la;
  for (size_t k = 0; k < stages; ++k) {
    la.n = 0;
    uint32_t tiles = 0;
    for (uint32_t i = 0; i < n; ++i) {
      const gkr_plan& p = *plans[i];
      if (k + 1 >= p.stage_first.size()) continue;
      for (uint32_t t = p.stage_first[k]; t < p.stage_first[k + 1]; ++t) {
        tiles += p.lock_tiles[t];
        la.end[la.n] = tiles;
        la.step[la.n] = p.lock_steps + t;
        la.flag[la.n++] = flags[i];
      }
    }
    launch_lock_stage(la, tiles, s);
  }
  launch_lock_end(a, flags, s);
}

extern "C" {

int32_t gkr_plan_create(const gkr_job* job, gkr_plan** out) {
  if (!job || !out || !job->circuit) {
    set_error("null argument");
    return GKR_EINVAL;
  }
  *out = nullptr;
  const gkr_circuit* c = job->circuit;
  if (c->general || c->field != GKR_FIELD_BN254) {
    set_error("batch plans take layered BN254 circuits only");
    return GKR_EUNSUPPORTED;
  }
  if (!job->d_inputs || !job->d_outputs || !job->d_proof || !aligned16b(job->d_inputs) ||
      !aligned16b(job->d_outputs) || !aligned16b(job->d_proof)) {
    set_error("null or misaligned job buffer");
    return GKR_EINVAL;
  }
  if (job->proof_cap < gkr_proof_bytes(c)) {
    set_error("proof buffer too small");
    return GKR_EBUFSZ;
  }
  int32_t rc = check_ws(c, job->d_ws, job->ws_bytes);
  if (rc) return rc;
  try {
    Workspace w = bind_workspace(*c, job->d_ws);
    // the persistent program, then the lockstep program, then the counters (zero), in one
    // vector and one upload: a plan holds one statement, so a program makes many
    Program pg;
    pg.steps.reserve(96ull * c->depth + 64);
    pg.mode = Program::kPersistent;
    emit_prove_circuit(pg, *c, w, job->d_inputs, job->seed, job->d_outputs, job->d_proof, current_tuning());
    std::unique_ptr<gkr_plan> p(new gkr_plan());
    p->job = *job;
    p->nsteps = (uint32_t)pg.steps.size();
    p->ctr_words = 2 + 2ull * p->nsteps;
    pg.mode = Program::kLockstep;
    emit_prove_circuit(pg, *c, w, job->d_inputs, job->seed, job->d_outputs, job->d_proof, current_tuning());
    const size_t lock_steps = pg.steps.size() - p->nsteps;
    p->stage_first.reserve(lock_steps + 1);
    p->lock_tiles.reserve(lock_steps);
    for (size_t k = 0; k < lock_steps; ++k) {
      const Step& st = pg.steps[p->nsteps + k];
      if (!st.join) p->stage_first.push_back((uint32_t)k);
      p->lock_tiles.push_back(st.ntiles);
      p->form = (p->form ^ (2 * st.type + st.join + 1)) * 0x9e3779b97f4a7c15ull;
      p->form ^= p->form >> 29;
    }
    p->stage_first.push_back((uint32_t)lock_steps);
    for (uint32_t i = 0; i <= c->depth; ++i) p->gates += 1ull << c->s(i);
    const size_t step_bytes = sizeof(Step) * pg.steps.size();
    pg.steps.resize(pg.steps.size() + (4 * p->ctr_words + sizeof(Step) - 1) / sizeof(Step));
    const size_t total = sizeof(Step) * pg.steps.size();
    if (hipMalloc(&p->dev, total) != hipSuccess) {
      (void)hipGetLastError();
      set_error("device allocation of the plan failed");
      return GKR_ENOMEM;
    }
    p->steps = static_cast<Step*>(p->dev);
    p->lock_steps = p->steps + p->nsteps;
    p->ctr = reinterpret_cast<uint32_t*>(static_cast<char*>(p->dev) + step_bytes);
    if (hipMemcpy(p->dev, pg.steps.data(), total, hipMemcpyHostToDevice) != hipSuccess) {
      (void)hipGetLastError();
      hipFree(p->dev);
      set_error("upload of the plan failed");
      return GKR_EDEVICE;
    }
    *out = p.release();
    return GKR_OK;
  } catch (const std::bad_alloc&) {
    set_error("host allocation failed");
    return GKR_ENOMEM;
  }
}

void gkr_plan_destroy(gkr_plan* p) {
  if (!p) return;
  if (p->dev) hipFree(p->dev);
  delete p;
}

int32_t gkr_plan_reset(gkr_plan* p, void* stream) {
  if (!p) {
    set_error("null plan");
    return GKR_EINVAL;
  }
  launch_fill_u32(p->ctr, p->ctr_words, 0u, static_cast<hipStream_t>(stream));
  p->queued.store(false, std::memory_order_relaxed);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error(std::string("kernel launch failed: ") + hipGetErrorString(e));
    return GKR_EDEVICE;
  }
  return GKR_OK;
}

int32_t gkr_run_batch(gkr_plan* const* plans, uint32_t n, uint32_t* d_ctl, uint32_t workgroups,
                      uint32_t step_budget, uint32_t stop_on_finish, void* stream) {
  if (!plans || !d_ctl || n == 0 || n > kMaxBatchJobs) {
    set_error("need 1.." + std::to_string(kMaxBatchJobs) + " plans and a control buffer");
    return GKR_EINVAL;
  }
  BatchArgs a;
  memset(&a, 0, sizeof(a));
  for (uint32_t i = 0; i < n; ++i) {
    if (!plans[i]) {
      set_error("null plan");
      return GKR_EINVAL;
    }
    for (uint32_t k = 0; k < i; ++k)
      if (plans[k] == plans[i]) {
        set_error("a plan appears twice in one run");
        return GKR_EINVAL;
      }
    a.jobs[i] = job_dev(*plans[i]);
  }
  a.njobs = n;
  a.step_budget = step_budget;
  a.stop_on_finish = stop_on_finish ? 1 : 0;
  a.ctl = d_ctl;
  // A run to the end on the whole device takes the plans that have not begun in
  // lockstep where that pays: stage k of every one of them in launch k. The persistent
  // kernel then finds those finished, and carries on those that an earlier run with a
  // limit began. A count of workgroups is a limit on the share of the device, which
  // the lockstep launches do not keep: with one the persistent kernel runs alone.
  // Plans that an earlier run has taken are left out: the launches of their stages
  // would find nothing to do (4 ms for a finished plan of depth 28).
  const bool whole = workgroups == 0 && step_budget == 0 && !stop_on_finish;
  gkr_plan* fresh[kMaxBatchJobs];
  uint32_t nfresh = 0;
  for (uint32_t i = 0; i < n; ++i)
    if (!plans[i]->queued.exchange(true, std::memory_order_relaxed)) fresh[nfresh++] = plans[i];
  const bool lockstep = whole && nfresh > 0 && lockstep_pays(fresh, nfresh);
  if (workgroups == 0) {
    int dev = 0, cus = 0;
    hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) {
      (void)hipGetLastError();
      cus = 256;
    }
    workgroups = (uint32_t)cus * batch_kernel_max_workgroups_per_cu();
    // to the end a workgroup per CU does best (64 uneven proofs 81.0 ms, against 84.6
    // with two per CU, which contend for the step counters, and 88.7 with 5 per 8 CUs)
    if (whole) workgroups = (uint32_t)cus;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  launch_fill_u32(d_ctl, 4, 0u, s);
  if (lockstep) run_lockstep(fresh, nfresh, d_ctl, s);
  launch_batch(a, workgroups, s);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error(std::string("kernel launch failed: ") + hipGetErrorString(e));
    return GKR_EDEVICE;
  }
  return GKR_OK;
}

int32_t gkr_plan_progress(const gkr_plan* p, uint32_t* done_steps, uint32_t* total_steps) {
  if (!p) {
    set_error("null plan");
    return GKR_EINVAL;
  }
  uint32_t cur = 0;
  if (hipMemcpy(&cur, p->ctr, 4, hipMemcpyDeviceToHost) != hipSuccess) {
    (void)hipGetLastError();
    set_error("reading plan progress failed");
    return GKR_EDEVICE;
  }
  if (done_steps) *done_steps = cur;
  if (total_steps) *total_steps = p->nsteps;
  return GKR_OK;
}

int32_t gkr_prove_batch(const gkr_job* jobs, uint32_t n, void* stream) {
  if (!jobs || n == 0) {
    set_error("no jobs");
    return GKR_EINVAL;
  }
  std::vector<gkr_plan*> plans(n, nullptr);
  int32_t rc = GKR_OK;
  for (uint32_t i = 0; i < n && rc == GKR_OK; ++i) rc = gkr_plan_create(&jobs[i], &plans[i]);
  uint32_t* ctl = nullptr;
  if (rc == GKR_OK && hipMalloc(&ctl, 16) != hipSuccess) {
    (void)hipGetLastError();
    set_error("device allocation failed");
    rc = GKR_ENOMEM;
  }
  for (uint32_t b = 0; b < n && rc == GKR_OK; b += kMaxBatchJobs) {
    const uint32_t m = std::min<uint32_t>(kMaxBatchJobs, n - b);
    rc = gkr_run_batch(plans.data() + b, m, ctl, 0, 0, 0, stream);
  }
  if (rc == GKR_OK && hipStreamSynchronize(static_cast<hipStream_t>(stream)) != hipSuccess) {
    (void)hipGetLastError();
    set_error("batch run failed");
    rc = GKR_EDEVICE;
  }
  if (ctl) hipFree(ctl);
  for (gkr_plan* p : plans) gkr_plan_destroy(p);
  return rc;
}

}  // extern "C"
