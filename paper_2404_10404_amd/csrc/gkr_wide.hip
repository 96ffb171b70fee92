// A sumcheck round over small tables: one field product per thread.
//
// With one pair per thread (k_round_a) a round whose tables do not fill the
// chip is a chain: six folds and two evaluation products one after another in
// one wave (8.7 us of the round's 20), then the sums, the hash and the launch.
// Here a workgroup takes 32 pairs and wave k takes table k: lanes 0..31 fold
// the pairs' lower entries and lanes 32..63 the upper ones, so all folds are one
// product deep; the folded entries meet in shared memory, and one wave (two
// for five tables) evaluates, lanes 0..31 at t = 0 and 32..63 at t = 2, one product
// each. A round of 2^9..2^13 pairs takes 13 us instead of 20 (three tables).
// Above 2^13 pairs the chip fills either way (a proof of 2^20 gates x 16 layers
// with the limit at 2^12: 11.89 ms, 2^13: 11.81, 2^14: 11.80).
#include "gkr_bodies.hpp"
#include "gkr_profile.hpp"
#include "gkr_wide_bodies.hpp"

namespace gkr {

template <class Form>
__global__ void __launch_bounds__(64 * Form::NT) k_wide_round(Step st) {
  body_wide_round<Form>(st, blockIdx.x, gridDim.x);
}
__global__ void __launch_bounds__(kBlock) k_wide_p1_gates(Step st) { body_wide_p1_gates(st, blockIdx.x, gridDim.x); }
__global__ void __launch_bounds__(64 * 3) k_wide_p1_round(Step st) { body_wide_p1_round(st, blockIdx.x, gridDim.x); }

void launch_wide_step(const Step& st, hipStream_t s) {
  const int tok = prof_begin(s);
  const dim3 grid(st.ntiles);
  ProfClass cls = PC_ROUND_WIDE;
  switch (st.type) {
    case ST_W_ROUND_A: k_wide_round<FormA><<<grid, dim3(64 * 3), 0, s>>>(st); break;
    case ST_W_ROUND_B: k_wide_round<FormB><<<grid, dim3(64 * 5), 0, s>>>(st); break;
    case ST_W_P1_GATES: k_wide_p1_gates<<<grid, dim3(kBlock), 0, s>>>(st); cls = PC_PHASE1_WIDE; break;
    case ST_W_P1_ROUND: k_wide_p1_round<<<grid, dim3(64 * 3), 0, s>>>(st); cls = PC_PHASE1_WIDE; break;
    default: break;
  }
  if (tok >= 0) prof_end(tok, s, cls, st.bytes, st.mulmods);
}

}  // namespace gkr
