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
// Above 2^13 pairs (c2, sweep of the limit: 14.20 ms at 2^15, 14.06 at 2^14, 14.02
// at 2^13, 14.06 at 2^12) the chip fills either way and more than 256 workgroups
// queue on the round's counter.
#include "gkr_bodies.hpp"
#include "gkr_profile.hpp"
#include "gkr_wide.hpp"

namespace gkr {

// The end of a wide round, from the folded entries in shared memory (ent[k]: table
// k's lower, then upper entries of the workgroup's pairs; the workgroup has
// written them, not yet synchronised): waves 0.. evaluate and store the partial
// sums, the last workgroup runs the transcript step.
template <class Form>
__device__ __forceinline__ void wide_finish(const Fr (*ent)[2 * kWidePairs], Fr* partials, DevState* S, Fr* r_out,
                                            uint32_t* msg) {
  constexpr int NT = Form::NT;
  // wave 0: x0 x1 (+ x2 of three tables), wave 1 of five tables: x2 x3 + x4
  constexpr uint32_t kEval = NT == 3 ? 1 : 2;
  const uint32_t wid = threadIdx.x >> 6, lane = threadIdx.x & 63, p = lane & 31;
  __syncthreads();
  if (wid < kEval) {
    auto at = [&](uint32_t k) {
      const Fr lo = opaque(ent[k][p]);
      return lane < 32 ? lo : opaque(fr_sub(fr_double(opaque(ent[k][32 + p])), lo));
    };
    const Fr x = at(2 * wid), y = at(2 * wid + 1);
    Fr t = fr_mul(x, y);
    if (NT == 3 || wid == 1) t = fr_add(t, at(NT - 1));
    t = half_wave_sum(t);
    if (p == 31) stf(partials, ((uint64_t)blockIdx.x * kEval + wid) * 2 + (lane >> 5), t);
    wait_vmem();
  }
  if (last_tile(&S->counter, gridDim.x)) finish_reduced_round<false>(partials, gridDim.x * kEval, S, r_out, msg);
}

// Steps and pointers as in ST_ROUND_A / ST_ROUND_B (RoundPtrs); NT waves per workgroup.
template <class Form>
__global__ void __launch_bounds__(64 * Form::NT) k_wide_round(Step st) {
  constexpr int NT = Form::NT;
  using R = RoundPtrs<NT>;
  __shared__ Fr ent[NT][2 * kWidePairs];
  const uint32_t wid = threadIdx.x >> 6, lane = threadIdx.x & 63, p = lane & 31;
  const uint64_t half = st.q[0];
  const Fr* rprev = P<const Fr*>(st, R::kR);
  const uint64_t b = (uint64_t)blockIdx.x * kWidePairs + p;
  const uint64_t e = lane < 32 ? b : b + half;
  Fr v = fr_zero();
  if (b < half) {
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
  wide_finish<Form>(ent, P<Fr*>(st, R::kPart), P<DevState*>(st, R::kS), P<Fr*>(st, R::kROut),
                    P<uint32_t*>(st, R::kMsg));
}

// ST_W_P1_GATES: the phase-1 term of every gate and copy, tw[(k << n) | c] = T[z,c]
// W[y_z,c] for position k of the wiring by x (see phase1_entry), one per thread:
// an entry's gates one after another in its thread (k_p1_init_round) take 45 us
// where a row has up to six gates, this and the round below 22.
// p0 W, p1 tw, p2 xent, p3 aU, p4 bV, p5 Cu, p6 Cv; u0 n; q0 gates x copies.
__global__ void __launch_bounds__(kBlock) k_wide_p1_gates(Step st) {
  const uint32_t n = st.u[0];
  const uint64_t mask = (1ull << n) - 1;
  for (uint64_t t = (uint64_t)blockIdx.x * kBlock + threadIdx.x; t < st.q[0]; t += (uint64_t)gridDim.x * kBlock) {
    const uint2 e = P<const uint2*>(st, 2)[t >> n];
    const uint64_t c = t & mask;
    const Fr w = ldf(P<const Fr*>(st, 0), ((uint64_t)(e.y & 0x7fffffffu) << n) | c);
    const Fr T = fr_mul_add2(ldf(P<const Fr*>(st, 3), e.x), ldf(P<const Fr*>(st, 5), c), ldf(P<const Fr*>(st, 4), e.x),
                             ldf(P<const Fr*>(st, 6), c));
    stf(P<Fr*>(st, 1), t, fr_mul(T, w));
  }
}

// ST_W_P1_ROUND: the phase-1 tables from those terms, and round 1. Wave 0 loads W,
// wave 1 adds up G's entries (the MUL terms, and sum T over the ADD gates =
// Cu sum aU + Cv sum bV), wave 2 H's (the ADD terms). p0 W, p1 G, p2 H, p3 xrow,
// p4 xmid, p5 xent, p6 tw, p7 aU, p8 bV, p9 S, p10 partials, p11 r_out, p12 msg,
// p13 Cu, p14 Cv; u0 n; q0 pairs.
__global__ void __launch_bounds__(64 * 3) k_wide_p1_round(Step st) {
  __shared__ Fr ent[3][2 * kWidePairs];
  const uint32_t wid = threadIdx.x >> 6, lane = threadIdx.x & 63, p = lane & 31;
  const uint32_t n = st.u[0];
  const uint64_t half = st.q[0], mask = (1ull << n) - 1;
  const uint64_t b = (uint64_t)blockIdx.x * kWidePairs + p;
  const uint64_t e = lane < 32 ? b : b + half;
  Fr v = fr_zero();
  if (b < half) {
    if (wid == 0) {
      v = ldf(P<const Fr*>(st, 0), e);
    } else {
      const uint64_t x = e >> n, c = e & mask;
      const uint32_t k0 = P<const uint32_t*>(st, 3)[x], km = P<const uint32_t*>(st, 4)[x],
                     k1 = P<const uint32_t*>(st, 3)[x + 1];
      const Fr* tw = P<const Fr*>(st, 6);
      if (wid == 1) {
        for (uint32_t k = k0; k < km; ++k) v = fr_add(v, ldf(tw, ((uint64_t)k << n) | c));
        if (km < k1) {
          Fr sa = fr_zero(), sb = fr_zero();
          for (uint32_t k = km; k < k1; ++k) {
            const uint32_t z = P<const uint2*>(st, 5)[k].x;
            sa = fr_add(sa, ldf(P<const Fr*>(st, 7), z));
            sb = fr_add(sb, ldf(P<const Fr*>(st, 8), z));
          }
          v = fr_add(v, fr_mul_add2(sa, ldf(P<const Fr*>(st, 13), c), sb, ldf(P<const Fr*>(st, 14), c)));
        }
        stf(P<Fr*>(st, 1), e, v);
      } else {
        for (uint32_t k = km; k < k1; ++k) v = fr_add(v, ldf(tw, ((uint64_t)k << n) | c));
        stf(P<Fr*>(st, 2), e, v);
      }
    }
  }
  ent[wid][lane] = v;
  wide_finish<FormA>(ent, P<Fr*>(st, 10), P<DevState*>(st, 9), P<Fr*>(st, 11), P<uint32_t*>(st, 12));
}

void launch_wide_step(const Step& st, hipStream_t s) {
  const int tok = prof_begin(s);
  const dim3 grid(st.ntiles);
  ProfClass cls = PC_ROUND_A;
  switch (st.type) {
    case ST_W_ROUND_A: k_wide_round<FormA><<<grid, dim3(64 * 3), 0, s>>>(st); break;
    case ST_W_ROUND_B: k_wide_round<FormB><<<grid, dim3(64 * 5), 0, s>>>(st); cls = PC_ROUND_B; break;
    case ST_W_P1_GATES: k_wide_p1_gates<<<grid, dim3(kBlock), 0, s>>>(st); cls = PC_PHASE1_INIT; break;
    case ST_W_P1_ROUND: k_wide_p1_round<<<grid, dim3(64 * 3), 0, s>>>(st); cls = PC_PHASE1_INIT; break;
    default: break;
  }
  if (tok >= 0) prof_end(tok, s, cls, st.bytes, st.mulmods);
}

}  // namespace gkr
