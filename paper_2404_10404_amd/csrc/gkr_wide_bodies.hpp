// Bodies of the wide rounds (see gkr_wide.hip), for workgroups of any number of
// waves: one per table in the plain kernels, four in the lockstep kernel of a
// batch.
#pragma once

#include "gkr_bodies.hpp"
#include "gkr_wide.hpp"

namespace gkr {

// The end of a wide round, from the folded entries in shared memory (ent[k]: table
// k's lower, then upper entries of the tile's pairs; the workgroup has written
// them, not yet synchronised): waves 0.. evaluate and store the partial sums,
// the last tile runs the transcript step.
template <class Form>
__device__ __forceinline__ void wide_finish(const Fr (*ent)[2 * kWidePairs], Fr* partials, DevState* S, Fr* r_out,
                                            uint32_t* msg, uint32_t tile, uint32_t ntiles) {
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
    if (p == 31) put_partial(partials, ((uint64_t)tile * kEval + wid) * 2 + (lane >> 5), t);
    wait_vmem();
  }
  if (last_tile(&S->counter, ntiles)) finish_reduced_round<false>(partials, ntiles * kEval, S, r_out, msg);
}

// ST_W_ROUND_A / ST_W_ROUND_B: pointers as in ST_ROUND_A / ST_ROUND_B (RoundPtrs).
template <class Form>
__device__ __forceinline__ void body_wide_round(const Step& st, uint32_t tile, uint32_t ntiles) {
  constexpr int NT = Form::NT;
  using R = RoundPtrs<NT>;
  __shared__ Fr ent[NT][2 * kWidePairs];
  const uint32_t lane = threadIdx.x & 63, p = lane & 31;
  const uint64_t half = st.q[0];
  const Fr* rprev = P<const Fr*>(st, R::kR);
  const uint64_t b = (uint64_t)tile * kWidePairs + p;
  const uint64_t e = lane < 32 ? b : b + half;
  for (uint32_t tab = threadIdx.x >> 6; tab < NT; tab += blockDim.x >> 6) {
    Fr v = fr_zero();
    if (b < half) {
      const Fr* src = P<const Fr*>(st, 0);
      Fr* dst = P<Fr*>(st, NT);
#pragma unroll
      for (int k = 1; k < NT; ++k)
        if (tab == (uint32_t)k) {
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
    ent[tab][lane] = v;
  }
  wide_finish<Form>(ent, P<Fr*>(st, R::kPart), P<DevState*>(st, R::kS), P<Fr*>(st, R::kROut),
                    P<uint32_t*>(st, R::kMsg), tile, ntiles);
}

// ST_W_P1_GATES: the phase-1 term of every gate and copy, tw[(k << n) | c] = T[z,c]
// W[y_z,c] for position k of the wiring by x (see phase1_entry), one per thread:
// an entry's gates one after another in its thread (k_p1_init_round) take 45 us
// where a row has up to six gates, this and the round below 22.
// p0 W, p1 tw, p2 xent, p3 aU, p4 bV, p5 Cu, p6 Cv; u0 n; q0 gates x copies.
__device__ __forceinline__ void body_wide_p1_gates(const Step& st, uint32_t tile, uint32_t ntiles) {
  const uint32_t n = st.u[0];
  const uint64_t mask = (1ull << n) - 1;
  for (uint64_t t = (uint64_t)tile * kBlock + threadIdx.x; t < st.q[0]; t += (uint64_t)ntiles * kBlock) {
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
__device__ __forceinline__ void body_wide_p1_round(const Step& st, uint32_t tile, uint32_t ntiles) {
  __shared__ Fr ent[3][2 * kWidePairs];
  const uint32_t wid = threadIdx.x >> 6, lane = threadIdx.x & 63, p = lane & 31;
  const uint32_t n = st.u[0];
  const uint64_t half = st.q[0], mask = (1ull << n) - 1;
  const uint64_t b = (uint64_t)tile * kWidePairs + p;
  const uint64_t e = lane < 32 ? b : b + half;
  Fr v = fr_zero();
  if (wid < 3 && b < half) {
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
  if (wid < 3) ent[wid][lane] = v;
  wide_finish<FormA>(ent, P<Fr*>(st, 10), P<DevState*>(st, 9), P<Fr*>(st, 11), P<uint32_t*>(st, 12), tile, ntiles);
}

}  // namespace gkr
