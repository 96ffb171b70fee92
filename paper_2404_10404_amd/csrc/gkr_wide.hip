// A sumcheck round over small tables: one field product per thread.
//
// With one pair per thread (k_round_a) a round whose tables do not fill the
// chip is a chain: six folds and two evaluation products one after another in
// one wave (8.7 us of the round's 20), then the sums, the hash and the launch.
// Here a workgroup takes 32 pairs and wave k takes table k: lanes 0..31 fold
// the pairs' lower entries and lanes 32..63 the upper ones, so all folds are one
// product deep; the folded entries meet in shared memory, and one wave (two
// for five tables) evaluates, lanes 0..31 at t = 0 and 32..63 at t = 2, one product
// each. A round of 2^9..2^13 pairs takes 12 us instead of 20 (three tables).
// Above 2^15 pairs the chip is full either way and the extra pass through
// shared memory and the larger number of partial sums cost more than they save.
#include "gkr_bodies.hpp"
#include "gkr_profile.hpp"
#include "gkr_wide.hpp"

namespace gkr {

// Steps and pointers as in ST_ROUND_A / ST_ROUND_B (RoundPtrs); NT waves per workgroup.
template <class Form>
__global__ void __launch_bounds__(64 * Form::NT) k_wide_round(Step st) {
  constexpr int NT = Form::NT;
  using R = RoundPtrs<NT>;
  __shared__ Fr ent[NT][2 * kWidePairs];  // the tables' entries: lower, then upper ones of the pairs
  const uint32_t wid = threadIdx.x >> 6, lane = threadIdx.x & 63, p = lane & 31;
  const uint64_t half = st.q[0];
  const Fr* rprev = P<const Fr*>(st, R::kR);
  const uint64_t b = (uint64_t)blockIdx.x * kWidePairs + p;
  const bool act = b < half;
  const uint64_t e = lane < 32 ? b : b + half;
  Fr v = fr_zero();
  if (act) {
    const Fr* src = P<const Fr*>(st, 0);
    Fr* dst = P<Fr*>(st, NT);
#pragma unroll
    for (int k = 1; k < NT; ++k)
      if (wid == (uint32_t)k) {
        src = P<const Fr*>(st, k);
        dst = P<Fr*>(st, NT + k);
      }
    v = ldf(src, e);
    if (rprev) {
      const Fr a1 = ldf(src, e + 2 * half), r = ldf(rprev, 0);
      v = fr_add(v, fr_mul(r, fr_sub(a1, v)));
      stf(dst, e, v);
    }
  }
  ent[wid][lane] = v;
  __syncthreads();
  // wave 0: x0 x1 (+ x2 of three tables), wave 1 of five tables: x2 x3 + x4
  constexpr uint32_t kEval = NT == 3 ? 1 : 2;
  Fr* partials = P<Fr*>(st, R::kPart);
  if (wid < kEval) {
    auto at = [&](uint32_t k) {
      const Fr lo = ent[k][p];
      return lane < 32 ? opaque(lo) : opaque(fr_sub(fr_double(ent[k][32 + p]), lo));
    };
    const Fr x = at(2 * wid), y = at(2 * wid + 1);
    Fr t = fr_mul(x, y);
    if (NT == 3 || wid == 1) t = fr_add(t, at(NT - 1));
    t = half_wave_sum(t);
    if (p == 31) stf(partials, ((uint64_t)blockIdx.x * kEval + wid) * 2 + (lane >> 5), t);
    wait_vmem();
  }
  if (last_tile(&P<DevState*>(st, R::kS)->counter, gridDim.x))
    finish_reduced_round<false>(partials, gridDim.x * kEval, P<DevState*>(st, R::kS), P<Fr*>(st, R::kROut),
                                P<uint32_t*>(st, R::kMsg));
}

void launch_wide_step(const Step& st, hipStream_t s) {
  const int tok = prof_begin(s);
  const dim3 grid(st.ntiles);
  if (st.type == ST_W_ROUND_A) k_wide_round<FormA><<<grid, dim3(64 * 3), 0, s>>>(st);
  else k_wide_round<FormB><<<grid, dim3(64 * 5), 0, s>>>(st);
  if (tok >= 0) prof_end(tok, s, st.type == ST_W_ROUND_A ? PC_ROUND_A : PC_ROUND_B, st.bytes, st.mulmods);
}

}  // namespace gkr
