// A batch of proofs in lockstep: launch k runs stage k (one step, or two that do not
// depend on each other) of every proof of the batch.
//
// The persistent batch kernel hands tiles of many proofs' steps to resident
// workgroups; between two steps of a proof lie a tile's publication (an L2
// write-back), a counter and another workgroup's scan and L2 invalidation, so
// 64 uneven proofs (depth 8..32, 2^10..2^18 gates per layer) take 81 ms (155 when
// every tile of a reduction wrote its L2 back) although their products take 4. Here
// a proof's next step begins with the next launch: no tile protocol, and a step of
// the whole batch costs one launch and its longest member: 58.7 ms, 1,350 launches
// of 43 us, of which about 16 are a launch and the shortest steps (a round's serial
// transcript), 20 the products and tiles of all proofs, the rest the wait for the
// longest step, which a few uneven proofs pay most (gkr_run_batch weighs it). Holding
// long steps back until every proof has one lowers a launch to 23 us but takes
// 5,700 of them.
#include "gkr_bodies.hpp"
#include "gkr_profile.hpp"
#include "gkr_wide_bodies.hpp"

namespace gkr {

// Two workgroups per CU: the bodies' registers, as in the persistent kernel.
__global__ void __launch_bounds__(kBlock, 2) k_lock(LockArgs a) {
  __shared__ Step sh;
  // the step whose tiles include this workgroup: the first with blockIdx < end
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t n = a.n;
  uint32_t i = 0;
#pragma unroll
  for (uint32_t h = 0; h < kMaxLockSteps / 64; ++h) {
    const uint32_t k = 64 * h + lane;
    i += (uint32_t)__popcll(__ballot(k < n && a.end[k < n ? k : 0] <= blockIdx.x));
  }
  i = (uint32_t)__builtin_amdgcn_readfirstlane((int)i);
  const uint32_t tile = blockIdx.x - (i ? a.end[i - 1] : 0);
  const uint32_t* src = reinterpret_cast<const uint32_t*>(a.step[i]);
  uint32_t* dst = reinterpret_cast<uint32_t*>(&sh);
  const uint32_t on = *a.flag[i];
  for (uint32_t k = threadIdx.x; k < sizeof(Step) / 4; k += kBlock) dst[k] = src[k];
  __syncthreads();
  if (!on) return;
  switch (sh.type) {
    case ST_W_ROUND_A: body_wide_round<FormA>(sh, tile, sh.ntiles); break;
    case ST_W_ROUND_B: body_wide_round<FormB>(sh, tile, sh.ntiles); break;
    case ST_W_P1_GATES: body_wide_p1_gates(sh, tile, sh.ntiles); break;
    case ST_W_P1_ROUND: body_wide_p1_round(sh, tile, sh.ntiles); break;
    default: run_step_tile(sh, tile, sh.ntiles); break;
  }
}

struct LockJobs {
  uint32_t* ctr[kMaxBatchJobs];
  uint32_t* flag[kMaxBatchJobs];
  uint32_t nsteps[kMaxBatchJobs];
  uint32_t n;
  uint32_t* ctl;
};

// A job takes part when no step of it has begun.
__global__ void __launch_bounds__(64) k_lock_begin(LockJobs a) {
  const uint32_t i = threadIdx.x;
  if (i < a.n) *a.flag[i] = a.ctr[i][0] == 0 && a.ctr[i][1] == 0 ? 1u : 0u;
}

// The jobs that took part are finished (ctr[0] = their step count), counted in ctl.
__global__ void __launch_bounds__(64) k_lock_end(LockJobs a) {
  const uint32_t i = threadIdx.x;
  if (i < a.n && *a.flag[i]) {
    a.ctr[i][0] = a.nsteps[i];
    *a.flag[i] = 0;
    atomicAdd(&a.ctl[0], 1u);
    atomicAdd(&a.ctl[2], a.nsteps[i]);
  }
}

static LockJobs lock_jobs(const BatchArgs& a, uint32_t* const* flags) {
  LockJobs j;
  for (uint32_t i = 0; i < a.njobs; ++i) {
    j.ctr[i] = a.jobs[i].ctr;
    j.flag[i] = flags[i];
    j.nsteps[i] = a.jobs[i].nsteps;
  }
  j.n = a.njobs;
  j.ctl = a.ctl;
  return j;
}

void launch_lock_begin(const BatchArgs& a, uint32_t* const* flags, hipStream_t s) {
  k_lock_begin<<<1, 64, 0, s>>>(lock_jobs(a, flags));
}
void launch_lock_stage(const LockArgs& a, uint32_t tiles, hipStream_t s) {
  const int tok = prof_begin(s);
  k_lock<<<tiles, kBlock, 0, s>>>(a);
  if (tok >= 0) prof_end(tok, s, PC_BATCH, 0.0, 0.0);
}
void launch_lock_end(const BatchArgs& a, uint32_t* const* flags, hipStream_t s) {
  k_lock_end<<<1, 64, 0, s>>>(lock_jobs(a, flags));
}

}  // namespace gkr
