// Phase 1 of a layer's sumcheck with the addition gates contracted over the
// copies (Section 2.3's bookkeeping tables for a layer of identical
// sub-circuits), for gfx950.
//
// Phase 1 sums W[x,c] G[x,c] + H[x,c] over (x, c), where a gate z = (x_z, y_z)
// with weight T[z,c] = aU[z] Cu[c] + bV[z] Cv[c] adds T W[y_z,c] to G (MUL), or T to
// G and T W[y_z,c] to H (ADD). Only the MUL gates need tables over (x, c):
//  - H is additive, and the ADD part of G is Cu[c] sa[x] + Cv[c] sb[x] with
//    sa[x] = sum_{ADD z: x_z = x} aU[z] (sb with bV). Over the sub-circuit
//    variables their sums over c are
//      sum_x Pu[x] sa[x] + Pv[x] sb[x] + h[x],
//      Pu[x] = sum_c Cu[c] W[x,c] (Pv with Cv),
//      h[x] = sum_{ADD z: x_z = x} aU[z] Pu[y_z] + bV[z] Pv[y_z]:
//    the five-table form of phase 2, on 2^sigma entries.
//  - For the copy variables, with the sub-circuit variables bound to rx,
//      G(rx,c) = Gm(rx,c) + Cu[c] sa(rx) + Cv[c] sb(rx),
//      H(rx,c) = Cu[c] A[c] + Cv[c] B[c],  A[c] = sum_y Aa[y] W[y,c] (B with Ab),
//    where Aa[y] = sum_{ADD z: y_z = y} aU[z] eq(rx, x_z) is a phase-2 table anyway.
//  - Gm's rows (x, .) without a MUL gate are zero until a fold pairs them with a
//    row that has one; which rows are zero at which level is known from the
//    wiring (a bit per row and level), so they are neither read, multiplied
//    nor written.
// The round polynomials, hence the proof bytes, are those of the three-table
// form: field sums in another order. Two passes over W (Pu and Pv; A and B) are
// added, one table of three leaves every round, and the table build does only
// the MUL gates' products.
#include <string.h>

#include <algorithm>

#include "gkr_bodies.hpp"
#include "gkr_contract.hpp"
#include "gkr_profile.hpp"
#include "gkr_general.hpp"
#include "gkr_split.hpp"

namespace gkr {

// Whether row `row` of the 2^k rows of a level is nonzero (levels one after
// another: bit 2^k + row). The row is the same in every lane: a scalar load.
__device__ __forceinline__ bool row_active(const uint32_t* act, uint32_t k, uint32_t row) {
  const uint32_t bit = (1u << k) + row;
  return (act[bit >> 5] >> (bit & 31)) & 1u;
}

// ST_S_SMALL: the 2^sigma tables sa, sb, h for x < q0 over the ADD gates of x.
// p0 xrow, p1 xmid, p2 xent (z, y | type << 31), p3 aU, p4 bV, p5 Pu, p6 Pv,
// p7 sa, p8 sb, p9 h.
__global__ void __launch_bounds__(kBlock) k_s_small(Step st) {
  const uint32_t* __restrict__ xrow = P<const uint32_t*>(st, 0);
  const uint32_t* __restrict__ xmid = P<const uint32_t*>(st, 1);
  const uint2* __restrict__ xent = P<const uint2*>(st, 2);
  const Fr *aU = P<const Fr*>(st, 3), *bV = P<const Fr*>(st, 4);
  const Fr *Pu = P<const Fr*>(st, 5), *Pv = P<const Fr*>(st, 6);
  for (uint64_t x = (uint64_t)blockIdx.x * kBlock + threadIdx.x; x < st.q[0]; x += (uint64_t)gridDim.x * kBlock) {
    Fr sa = fr_zero(), sb = fr_zero(), h = fr_zero();
    const uint32_t k1 = xrow[x + 1];
    for (uint32_t k = xmid[x]; k < k1; ++k) {
      const uint2 e = xent[k];
      const uint64_t y = e.y & 0x7fffffffu;
      const Fr a = ldf(aU, e.x), b = ldf(bV, e.x);
      sa = fr_add(sa, a);
      sb = fr_add(sb, b);
      h = fr_add(h, fr_mul_add2(a, ldf(Pu, y), b, ldf(Pv, y)));
    }
    stf(P<Fr*>(st, 7), x, sa);
    stf(P<Fr*>(st, 8), x, sb);
    stf(P<Fr*>(st, 9), x, h);
  }
}

// The MUL entry (x, c) of Gm: the sum of T[z,c] W[y_z,c] over x's MUL gates (at least one).
__device__ __forceinline__ Fr split_entry(const Fr* __restrict__ W, const uint2* __restrict__ xent,
                                          const Fr* __restrict__ aU, const Fr* __restrict__ bV, const Fr& cu,
                                          const Fr& cv, uint32_t k0, uint32_t k1, uint32_t n, uint64_t c) {
  Fr g = fr_zero();
  for (uint32_t k = k0; k < k1; ++k) {
    const uint2 e = xent[k];
    const uint64_t z = e.x, y = e.y & 0x7fffffffu;
    const Fr w = ldf(W, (y << n) | c);
    const Fr tw = fr_mul(fr_mul_add2(ldf(aU, z), cu, ldf(bV, z), cv), w);
    if (k == k0) g = tw;
    else g = fr_add(g, tw);
  }
  return g;
}

// ST_S_INIT_ROUND: Gm and round 1 in one pass. Tiles below u1 take the pairs b
// < q0 of the (x, c) table (rows x and x + 2^(sigma-1)); the others the q1 pairs
// of the five small tables. p0 W, p1 G, p2 xrow, p3 xmid, p4 xent, p5 aU, p6 bV,
// p7 Cu, p8 Cv, p9 S, p10 partials, p11 r_out, p12 msg, p13 the first small
// table, w0..w4 the entry offsets of all five from it; u0 n.
// ST_S_ROUND: a later round: folds both big tables and the small ones by the
// pending challenge and evaluates. p0 W src, p1 W dst, p2 G (in place), p3 act,
// p4..p8 small tables (in place), p9 S, p10 partials, p11 r_out, p12 msg,
// p13 rprev; u0 n, u1 tiles of the big part, u2 k (2^k rows before this round's
// pairing); q0 pairs, q1 small pairs.
// 2^14 rows of 2^12 copies, a quarter of them with MUL gates: the first pass takes
// 890 us and is bound by its products (VALU 76 % busy, 2.0 GiB moved); the later
// rounds move 1.001 times the bytes of W's levels and the active rows, at 4.3 TB/s
// of the 5.5 that the folding pattern reaches without arithmetic (VALU 72 % busy).
__global__ void __launch_bounds__(kBlock, 3) k_s_init_round(Step st) {
  const uint32_t nb = st.u[1];
  Fr acc[2] = {fr_zero(), fr_zero()};
  if (blockIdx.x < nb) {
    const Fr* __restrict__ W = P<const Fr*>(st, 0);
    Fr* __restrict__ G = P<Fr*>(st, 1);
    const uint32_t* __restrict__ xrow = P<const uint32_t*>(st, 2);
    const uint32_t* __restrict__ xmid = P<const uint32_t*>(st, 3);
    const uint2* __restrict__ xent = P<const uint2*>(st, 4);
    const Fr *aU = P<const Fr*>(st, 5), *bV = P<const Fr*>(st, 6);
    const uint32_t n = st.u[0];
    const uint64_t mask = (1ull << n) - 1, half = st.q[0], xh = half >> n;
    for (uint64_t b = (uint64_t)blockIdx.x * kBlock + threadIdx.x; b < half; b += (uint64_t)nb * kBlock) {
      // a wave's 64 entries lie in one row: its gates are the same in every lane
      const uint32_t x0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(b >> n)), x1 = x0 + (uint32_t)xh;
      const uint64_t c = b & mask;
      const uint32_t a0 = xrow[x0], e0 = xmid[x0], a1 = xrow[x1], e1 = xmid[x1];
      if (a0 == e0 && a1 == e1) continue;
      const Fr cu = ldf(P<const Fr*>(st, 7), c), cv = ldf(P<const Fr*>(st, 8), c);
      Fr g0 = fr_zero(), g1 = fr_zero();
      if (a0 != e0) {
        g0 = split_entry(W, xent, aU, bV, cu, cv, a0, e0, n, c);
        stf(G, b, g0);
      }
      if (a1 != e1) {
        g1 = split_entry(W, xent, aU, bV, cu, cv, a1, e1, n, c);
        stf(G, b + half, g1);
      }
      const Fr w0 = ldf(W, b), w1 = ldf(W, b + half);
      if (a0 != e0) acc[0] = fr_add(acc[0], fr_mul(w0, g0));
      acc[1] = fr_add(acc[1], fr_mul(fr_sub(fr_double(w1), w0), fr_sub(fr_double(g1), g0)));
    }
  } else {
    const Fr* base = P<const Fr*>(st, 13);
    const Fr* src[5];
    Fr* dst[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      src[k] = base + st.w[k];
      dst[k] = nullptr;
    }
    const Fr r = fr_zero();
    for (uint64_t b = (uint64_t)(blockIdx.x - nb) * kBlock + threadIdx.x; b < st.q[1];
         b += (uint64_t)(gridDim.x - nb) * kBlock)
      round_pair<FormB, false>(src, dst, b, st.q[1], r, acc[0], acc[1]);
  }
  write_partial<2>(acc, P<Fr*>(st, 10), blockIdx.x);
  if (last_tile(&P<DevState*>(st, 9)->counter, gridDim.x))
    finish_reduced_round<false>(P<const Fr*>(st, 10), gridDim.x, P<DevState*>(st, 9), P<Fr*>(st, 11),
                                P<uint32_t*>(st, 12));
}

__device__ __forceinline__ Fr fold_entry(const Fr& r, const Fr& a0, const Fr& a1) {
  return fr_add(a0, fr_mul(r, fr_sub(a1, a0)));
}

__global__ void __launch_bounds__(kBlock, 3) k_s_round(Step st) {
  const uint32_t nb = st.u[1];
  const Fr r = ldf(P<const Fr*>(st, 13), 0);
  Fr acc[2] = {fr_zero(), fr_zero()};
  if (blockIdx.x < nb) {
    const Fr* Ws = P<const Fr*>(st, 0);  // from the third round on the same table as Wd
    Fr* Wd = P<Fr*>(st, 1);
    Fr* G = P<Fr*>(st, 2);
    const uint32_t* __restrict__ act = P<const uint32_t*>(st, 3);
    const uint32_t n = st.u[0], k = st.u[2];
    const uint64_t half = st.q[0], m = 2 * half;
    const uint32_t rh = 1u << (k - 1);
    for (uint64_t b = (uint64_t)blockIdx.x * kBlock + threadIdx.x; b < half; b += (uint64_t)nb * kBlock) {
      const uint32_t x = (uint32_t)__builtin_amdgcn_readfirstlane((int)(b >> n));
      const bool f00 = row_active(act, k + 1, x), f01 = row_active(act, k + 1, x + 2 * rh);
      const bool f10 = row_active(act, k + 1, x + rh), f11 = row_active(act, k + 1, x + 3 * rh);
      const Fr a0 = ldf(Ws, b), a1 = ldf(Ws, b + m), c0 = ldf(Ws, b + half), c1 = ldf(Ws, b + half + m);
      Fr g00 = fr_zero(), g01 = fr_zero(), g10 = fr_zero(), g11 = fr_zero();
      if (f00) g00 = ldf(G, b);
      if (f01) g01 = ldf(G, b + m);
      if (f10) g10 = ldf(G, b + half);
      if (f11) g11 = ldf(G, b + half + m);
      const Fr wl = fold_entry(r, a0, a1);
      stf(Wd, b, wl);
      const Fr wh = fold_entry(r, c0, c1);
      stf(Wd, b + half, wh);
      Fr gl = fr_zero(), gh = fr_zero();
      if (f00 || f01) {
        gl = fold_entry(r, g00, g01);
        stf(G, b, gl);
        acc[0] = fr_add(acc[0], fr_mul(wl, gl));
      }
      if (f10 || f11) {
        gh = fold_entry(r, g10, g11);
        stf(G, b + half, gh);
      }
      if (f00 || f01 || f10 || f11)
        acc[1] = fr_add(acc[1], fr_mul(fr_sub(fr_double(wh), wl), fr_sub(fr_double(gh), gl)));
    }
  } else {
    const Fr* src[5];
    Fr* dst[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      src[k] = P<const Fr*>(st, 4 + k);
      dst[k] = P<Fr*>(st, 4 + k);
    }
    for (uint64_t b = (uint64_t)(blockIdx.x - nb) * kBlock + threadIdx.x; b < st.q[1];
         b += (uint64_t)(gridDim.x - nb) * kBlock)
      round_pair<FormB, true>(src, dst, b, st.q[1], r, acc[0], acc[1]);
  }
  write_partial<2>(acc, P<Fr*>(st, 10), blockIdx.x);
  if (last_tile(&P<DevState*>(st, 9)->counter, gridDim.x))
    finish_reduced_round<false>(P<const Fr*>(st, 10), gridDim.x, P<DevState*>(st, 9), P<Fr*>(st, 11),
                                P<uint32_t*>(st, 12));
}

// ST_S_WIDE_ROUND: ST_S_ROUND for small tables, with a product per thread as in the
// wide rounds: wave 2 g + t of a big tile folds table t (W, Gm) of its pairs
// 32 g .. 32 g + 31, the five waves of a small tile fold the five small tables of 32
// pairs; wave g then evaluates. Pointers and sizes as in ST_S_ROUND. A round with
// few pairs is one chain of products per thread otherwise (27 us, here 15).
__global__ void __launch_bounds__(64 * 5) k_s_wide_round(Step st) {
  const uint32_t nb = st.u[1], wid = threadIdx.x >> 6, lane = threadIdx.x & 63, p = lane & 31;
  const bool big = blockIdx.x < nb;
  const Fr r = ldf(P<const Fr*>(st, 13), 0);
  __shared__ Fr ent[5][64];
  Fr v = fr_zero();
  if (big && wid < 4) {
    const uint64_t half = st.q[0], m = 2 * half;
    const uint64_t b = (uint64_t)blockIdx.x * 64 + (wid >> 1) * 32 + p, e = lane < 32 ? b : b + half;
    if (b < half) {
      if ((wid & 1) == 0) {
        v = fold_entry(r, ldf(P<const Fr*>(st, 0), e), ldf(P<const Fr*>(st, 0), e + m));
        stf(P<Fr*>(st, 1), e, v);
      } else {
        Fr* G = P<Fr*>(st, 2);
        const uint32_t k = st.u[2], x = (uint32_t)(e >> st.u[0]);
        const bool f0 = row_active(P<const uint32_t*>(st, 3), k + 1, x);
        const bool f1 = row_active(P<const uint32_t*>(st, 3), k + 1, x + (2u << (k - 1)));
        if (f0 || f1) {
          v = fold_entry(r, f0 ? ldf(G, e) : fr_zero(), f1 ? ldf(G, e + m) : fr_zero());
          stf(G, e, v);
        }
      }
    }
  } else if (!big) {
    const uint64_t half = st.q[1], m = 2 * half;
    const uint64_t b = (uint64_t)(blockIdx.x - nb) * 32 + p, e = lane < 32 ? b : b + half;
    if (b < half) {
      Fr* t = P<Fr*>(st, 4);
#pragma unroll
      for (int k = 1; k < 5; ++k)
        if (wid == (uint32_t)k) t = P<Fr*>(st, 4 + k);
      v = fold_entry(r, ldf(t, e), ldf(t, e + m));
      stf(t, e, v);
    }
  }
  ent[wid][lane] = v;
  __syncthreads();
  if (wid < 2) {
    auto at = [&](uint32_t k) {
      const Fr lo = opaque(ent[k][p]);
      return lane < 32 ? lo : opaque(fr_sub(fr_double(opaque(ent[k][32 + p])), lo));
    };
    Fr t = fr_mul(at(2 * wid), at(2 * wid + 1));
    if (wid == 1 && !big) t = fr_add(t, at(4));
    t = half_wave_sum(t);
    if (p == 31) put_partial(P<Fr*>(st, 10), (2ull * blockIdx.x + wid) * 2 + (lane >> 5), t);
    wait_vmem();
  }
  if (last_tile(&P<DevState*>(st, 9)->counter, gridDim.x))
    finish_reduced_round<false>(P<const Fr*>(st, 10), 2 * gridDim.x, P<DevState*>(st, 9), P<Fr*>(st, 11),
                                P<uint32_t*>(st, 12));
}

// ST_S_P2_RAW: the phase-2 wiring tables over y < q0, which need eq(rx, .) on
// the sub-circuit variables only: Ma[y] = sum_{MUL z: y_z = y} aU[z] EL[x_z] (Mb
// with bV), Aa and Ab over the ADD gates. p0 yrow, p1 yent, p2 aU, p3 bV, p4 EL,
// p5 Ma, p6 Mb, p7 Aa, p8 Ab.
__global__ void __launch_bounds__(kBlock) k_s_p2_raw(Step st) {
  const uint32_t* __restrict__ yrow = P<const uint32_t*>(st, 0);
  const uint2* __restrict__ yent = P<const uint2*>(st, 1);
  const Fr *aU = P<const Fr*>(st, 2), *bV = P<const Fr*>(st, 3), *EL = P<const Fr*>(st, 4);
  for (uint64_t y = (uint64_t)blockIdx.x * kBlock + threadIdx.x; y < st.q[0]; y += (uint64_t)gridDim.x * kBlock) {
    Fr ma = fr_zero(), mb = fr_zero(), aa = fr_zero(), ab = fr_zero();
    const uint32_t k1 = yrow[y + 1];
    for (uint32_t k = yrow[y]; k < k1; ++k) {
      const uint2 e = yent[k];
      const Fr el = ldf(EL, e.y & 0x7fffffffu);
      const Fr a = fr_mul(ldf(aU, e.x), el), b = fr_mul(ldf(bV, e.x), el);
      if (e.y >> 31) {
        ma = fr_add(ma, a);
        mb = fr_add(mb, b);
      } else {
        aa = fr_add(aa, a);
        ab = fr_add(ab, b);
      }
    }
    stf(P<Fr*>(st, 5), y, ma);
    stf(P<Fr*>(st, 6), y, mb);
    stf(P<Fr*>(st, 7), y, aa);
    stf(P<Fr*>(st, 8), y, ab);
  }
}

// ST_S_P2_FINAL: Fa = vx Ma + Aa, Fb = vx Mb + Ab, Ka = vx Aa, Kb = vx Ab,
// Ks = su Ka + sv Kb for y < q0. p0 Fa, p1 Fb, p2 Ka (holding Aa), p3 Kb (Ab),
// p4 Ks, p5 S, p6 Ma, p7 Mb.
__global__ void __launch_bounds__(kBlock) k_s_p2_final(Step st) {
  const DevState* S = P<const DevState*>(st, 5);
  const Fr vx = opaque(S->vx), su = opaque(S->su), sv = opaque(S->sv);
  for (uint64_t y = (uint64_t)blockIdx.x * kBlock + threadIdx.x; y < st.q[0]; y += (uint64_t)gridDim.x * kBlock) {
    const Fr aa = ldf(P<const Fr*>(st, 2), y), ab = ldf(P<const Fr*>(st, 3), y);
    stf(P<Fr*>(st, 0), y, fr_add(fr_mul(vx, ldf(P<const Fr*>(st, 6), y)), aa));
    stf(P<Fr*>(st, 1), y, fr_add(fr_mul(vx, ldf(P<const Fr*>(st, 7), y)), ab));
    const Fr ka = fr_mul(vx, aa), kb = fr_mul(vx, ab);
    stf(P<Fr*>(st, 2), y, ka);
    stf(P<Fr*>(st, 3), y, kb);
    stf(P<Fr*>(st, 4), y, fr_mul_add2(su, ka, sv, kb));
  }
}

// ST_S_HANDOFF: the copy tables of phase 1 for c < q0: the last fold of W and Gm
// (two rows left) by the pending challenge, the ADD parts added. p0 A, p1 B,
// p2 Cu, p3 Cv, p4 sa, p5 sb (two entries left), p6 W src, p7 G, p8 act, p9 rprev,
// p10 Wc, p11 Gc, p12 Hc.
__global__ void __launch_bounds__(kBlock) k_s_handoff(Step st) {
  const Fr r = opaque(ldf(P<const Fr*>(st, 9), 0));
  const Fr *Ws = P<const Fr*>(st, 6), *G = P<const Fr*>(st, 7);
  const uint32_t* act = P<const uint32_t*>(st, 8);
  const bool f0 = row_active(act, 1, 0), f1 = row_active(act, 1, 1);
  const Fr sa = fold_entry(r, ldf(P<const Fr*>(st, 4), 0), ldf(P<const Fr*>(st, 4), 1));
  const Fr sb = fold_entry(r, ldf(P<const Fr*>(st, 5), 0), ldf(P<const Fr*>(st, 5), 1));
  const uint64_t ncop = st.q[0];
  for (uint64_t c = (uint64_t)blockIdx.x * kBlock + threadIdx.x; c < ncop; c += (uint64_t)gridDim.x * kBlock) {
    const Fr cu = ldf(P<const Fr*>(st, 2), c), cv = ldf(P<const Fr*>(st, 3), c);
    stf(P<Fr*>(st, 10), c, fold_entry(r, ldf(Ws, c), ldf(Ws, c + ncop)));
    Fr g = fr_mul_add2(cu, sa, cv, sb);
    if (f0 || f1)
      g = fr_add(g, fold_entry(r, f0 ? ldf(G, c) : fr_zero(), f1 ? ldf(G, c + ncop) : fr_zero()));
    stf(P<Fr*>(st, 11), c, g);
    stf(P<Fr*>(st, 12), c, fr_mul_add2(cu, ldf(P<const Fr*>(st, 0), c), cv, ldf(P<const Fr*>(st, 1), c)));
  }
}

void launch_split_step(const Step& st, hipStream_t s) {
  const int tok = prof_begin(s);
  const dim3 grid(st.ntiles), block(kBlock);
  ProfClass cls = PC_SMALL;
  switch (st.type) {
    case ST_S_SMALL: k_s_small<<<grid, block, 0, s>>>(st); break;
    case ST_S_INIT_ROUND: k_s_init_round<<<grid, block, 0, s>>>(st); cls = PC_PHASE1_SPLIT; break;
    case ST_S_ROUND: k_s_round<<<grid, block, 0, s>>>(st); cls = PC_ROUND_SPLIT; break;
    case ST_S_WIDE_ROUND: k_s_wide_round<<<grid, dim3(64 * 5), 0, s>>>(st); cls = PC_ROUND_WIDE; break;
    case ST_S_P2_RAW: k_s_p2_raw<<<grid, block, 0, s>>>(st); cls = PC_PHASE2_TABLES; break;
    case ST_S_P2_FINAL: k_s_p2_final<<<grid, block, 0, s>>>(st); cls = PC_PHASE2_TABLES; break;
    case ST_S_HANDOFF: k_s_handoff<<<grid, block, 0, s>>>(st); break;
    default: break;
  }
  if (tok >= 0) prof_end(tok, s, cls, st.bytes, st.mulmods);
}

// ---------------------------------------------------------------- host

namespace {

constexpr double kE = 32.0;
constexpr uint32_t kSplitMinLogCopies = 9, kSplitMinLogRows = 10, kSplitMinLogWidth = 23;
// Most pairs (log2) of a wide round: a layer of 2^22 gates took 2,000 us without,
// 1,953 up to 2^12 pairs, 1,927 up to 2^14, 1,925 up to 2^15, 1,927 up to 2^16.
constexpr uint32_t kSplitWideMaxLogHalf = 15;
constexpr uint32_t kSplitBlocks = 768;  // workgroups of a round over (x, c): three per CU

Step smk(uint32_t type, uint64_t items, uint64_t cap = 1u << 20) {
  Step st;
  memset(&st, 0, sizeof(st));
  st.type = type;
  st.ntiles = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((items + kBlock - 1) / kBlock, cap));
  return st;
}

}  // namespace

// The form trades three passes over three tables for two contractions more, and
// gains what Gm's empty rows leave out. Four layers, this form and the other, us:
//   entries (copies)   MUL 1/10        1/2             all
//   2^22 (2^9)         5,640 / 5,656   6,020 / 5,630   6,236 / 5,628
//   2^23 (2^10)        7,506 / 8,428   8,296 / 8,408   8,965 / 8,435
//   2^24 (2^11)       10,900 / 13,500 12,515 / 13,489 13,711 / 13,575 (3/4: 13,266 / 13,662)
//   2^23 (2^8)         7,750 / 8,163   8,544 / 8,191   9,097 / 8,158 (no matrix cores)
bool split_applies(uint32_t n, uint32_t sigma, uint64_t mul_gates) {
  const bool sparse = n + sigma > kSplitMinLogWidth ? 4 * mul_gates <= 3ull << sigma : 2 * mul_gates <= 1ull << sigma;
  return sparse && n >= kSplitMinLogCopies && sigma >= kSplitMinLogRows && n + sigma >= kSplitMinLogWidth &&
         cc_scratch_bytes(sigma, n) <= sizeof(Fr) << (n + sigma);
}

void emit_phase1_split(Program& pg, const Workspace& w, const LayerWiring& lw, const Fr* W, uint32_t n, uint32_t sigma,
                       uint64_t gates, uint64_t mul_gates, Fr* rx, uint32_t* proof, const Tuning& tun) {
  DevState* S = w.state;
  const uint64_t rows = 1ull << sigma, ncop = 1ull << n, full = rows << n;
  // Pu, Pv where phase 2 will have P, Q; sa, sb, h where it will have Fa, Fb, Ks
  if (void* cc = cc_scratch(w, n, sigma)) emit_contract_mfma(pg, W, w.Cu, w.Cv, w.P, w.Q, n, sigma, false, cc);
  else pg.copy_contract(W, w.Cu, w.Cv, w.P, w.Q, n, rows);
  Fr* small[5] = {w.P, w.Fa, w.Q, w.Fb, w.Ks};
  {
    Step st = smk(ST_S_SMALL, rows);
    st.p[0] = lw.xrow; st.p[1] = lw.xmid; st.p[2] = lw.xent; st.p[3] = w.aU; st.p[4] = w.bV; st.p[5] = w.P;
    st.p[6] = w.Q; st.p[7] = w.Fa; st.p[8] = w.Fb; st.p[9] = w.Ks; st.q[0] = rows;
    st.bytes = kE * (3.0 * rows + 4.0 * (gates - mul_gates)); st.mulmods = 1.5 * (gates - mul_gates);
    pg.steps.push_back(st);
  }
  const Fr* Ws = W;
  for (uint32_t j = 0; j < sigma; ++j) {
    const uint64_t half = full >> (j + 1), shalf = rows >> (j + 1);
    const uint32_t ns = (uint32_t)std::min<uint64_t>((shalf + kBlock - 1) / kBlock, 64);
    Step st = smk(j == 0 ? ST_S_INIT_ROUND : ST_S_ROUND, half, j == 0 ? 2 * kSplitBlocks : kSplitBlocks);
    st.u[0] = n; st.u[1] = st.ntiles; st.u[2] = sigma - j;
    st.ntiles += ns;
    if (j > 0 && half <= 1ull << kSplitWideMaxLogHalf) {
      st.type = ST_S_WIDE_ROUND;
      st.u[1] = (uint32_t)((half + 63) / 64);
      st.ntiles = st.u[1] + (uint32_t)((shalf + 31) / 32);
    }
    st.q[0] = half; st.q[1] = shalf;
    st.p[9] = S; st.p[10] = w.partials; st.p[11] = rx + j; st.p[12] = proof + 24 * j;
    if (j == 0) {
      st.p[0] = W; st.p[1] = w.G; st.p[2] = lw.xrow; st.p[3] = lw.xmid; st.p[4] = lw.xent; st.p[5] = w.aU;
      st.p[6] = w.bV; st.p[7] = w.Cu; st.p[8] = w.Cv;
      for (int k = 0; k < 5; ++k) st.w[k] = (uint32_t)(small[k] - small[0]);
      st.p[13] = small[0];
      const double a0 = split_active_share(mul_gates, rows, 0), a1 = split_active_share(mul_gates, rows, 1);
      st.bytes = kE * (mul_gates * ncop + a0 * full + a1 * full);  // gathers, Gm, W beside active rows
      st.mulmods = 2.5 * mul_gates * ncop + (a0 + a1) * half;
    } else {
      st.p[0] = Ws; st.p[1] = w.Wf; st.p[2] = w.G; st.p[3] = lw.act;
      for (int k = 0; k < 5; ++k) st.p[4 + k] = small[k];
      st.p[13] = rx + j - 1;
      Ws = w.Wf;
      const double a0 = split_active_share(mul_gates, rows, j - 1), a1 = split_active_share(mul_gates, rows, j);
      const double a2 = split_active_share(mul_gates, rows, j + 1);
      st.bytes = kE * half * (6.0 + 4.0 * a0 + 2.0 * a1); st.mulmods = half * (2.0 + 3.0 * a1 + a2);
    }
    pg.steps.push_back(st);
  }
  {
    const uint32_t bits[1] = {sigma};
    const Fr* pts[1] = {rx};
    const Fr* scl[1] = {nullptr};
    Fr* outs[1] = {w.EL};
    pg.eq(1, bits, pts, scl, outs);
  }
  // Ma, Mb where phase 2 will have P, Q (sa and sb keep their last two entries
  // in Fa, Fb until the hand-off)
  {
    Step st = smk(ST_S_P2_RAW, rows);
    st.p[0] = lw.yrow; st.p[1] = lw.yent; st.p[2] = w.aU; st.p[3] = w.bV; st.p[4] = w.EL; st.p[5] = w.P;
    st.p[6] = w.Q; st.p[7] = w.Ka; st.p[8] = w.Kb; st.q[0] = rows;
    st.bytes = kE * (3.0 * gates + 4.0 * rows); st.mulmods = 2.0 * gates;
    pg.steps.push_back(st);
  }
  // A, B where phase 2 will have U, V; H, which this form does not use, is the scratch
  emit_contract_mfma(pg, W, w.Ka, w.Kb, w.U, w.V, sigma, n, true, w.H);
  {
    Step st = smk(ST_S_HANDOFF, ncop);
    st.p[0] = w.U; st.p[1] = w.V; st.p[2] = w.Cu; st.p[3] = w.Cv; st.p[4] = w.Fa; st.p[5] = w.Fb; st.p[6] = Ws;
    st.p[7] = w.G; st.p[8] = lw.act; st.p[9] = rx + sigma - 1; st.p[10] = w.Wc; st.p[11] = w.Fc; st.p[12] = w.Kc;
    st.q[0] = ncop;
    st.bytes = kE * 11.0 * ncop; st.mulmods = 5.0 * ncop;
    pg.steps.push_back(st);
  }
  Fr* tc[3] = {w.Wc, w.Fc, w.Kc};
  const Fr* tc_src[3] = {w.Wc, w.Fc, w.Kc};
  const uint32_t s1 = sigma + n;
  emit_phase_a(pg, tc_src, tc, n, S, w.partials, rx + sigma, proof + 24 * sigma, &S->vx, proof + 24 * s1, tun);
}

void emit_p2_final(Program& pg, const Workspace& w, uint64_t rows) {
  Step st = smk(ST_S_P2_FINAL, rows);
  st.p[0] = w.Fa; st.p[1] = w.Fb; st.p[2] = w.Ka; st.p[3] = w.Kb; st.p[4] = w.Ks; st.p[5] = w.state; st.p[6] = w.P;
  st.p[7] = w.Q; st.q[0] = rows;
  st.bytes = kE * 9.0 * rows; st.mulmods = 5.5 * rows;
  pg.steps.push_back(st);
}

}  // namespace gkr
