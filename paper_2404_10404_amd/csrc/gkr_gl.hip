// The layered data-parallel prover over the Goldilocks field (Section 4.1,
// the field choice), for gfx950: kernels, the proof program and the C ABI.
//
// The protocol is the BN254 prover's (GKR layer relation, Libra's two-phase
// product sumcheck, claims combined with squeezed alpha and beta, bits bound
// from the most significant, copies in the low bits) with 8-byte canonical
// elements and this field's transcript rules:
//   accept         v = LE64(digest bytes 0..7); rehash with "GKRC" while v >= p
//   round(e0, e2)  one compression of LE64(e0) || LE64(e2) || 47 zero bytes || 0x01
//   values         vx, vy absorbed with "GKRV" as 8 bytes
// Elements are 8 bytes, so a wave's load of 64 consecutive entries is 512
// bytes; a product is four 32 x 32 multiplies and the reduction of gl.hpp.
// One kernel per step type. Phase 2 contracts the copy factors and big layers take
// phase 1 with the addition gates contracted over the copies, as the BN254 prover
// does; products are cheap here, so a round's finisher is one chain (the hash, spread
// over a wave's lanes) and the small rounds of a phase run in one workgroup.
#include <string.h>

#include <algorithm>
#include <new>
#include <string>
#include <vector>

#include "gkr_bodies.hpp"
#include "gkr_gl.hpp"
#include "gkr_profile.hpp"
#include "gkr_program.hpp"
#include "gkr_split.hpp"
#include "gkr_tuning.hpp"
#include "gl.hpp"

namespace gkr {

// ---------------------------------------------------------------- device helpers

typedef __attribute__((address_space(1))) uint64_t GlobalU64;

__device__ __forceinline__ uint64_t gld(const uint64_t* p, uint64_t i) { return ((const GlobalU64*)p)[i]; }
__device__ __forceinline__ void gst(uint64_t* p, uint64_t i, uint64_t v) { ((GlobalU64*)p)[i] = v; }

// Two adjacent elements (i even) as one 16-byte access.
typedef uint64_t U64x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) U64x2 GlobalU64x2;
__device__ __forceinline__ U64x2 gld2(const uint64_t* p, uint64_t i) { return *(const GlobalU64x2*)(p + i); }
__device__ __forceinline__ void gst2(uint64_t* p, uint64_t i, U64x2 v) { *(GlobalU64x2*)(p + i) = v; }

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int mask) {
  const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, mask, 64);
  const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), mask, 64);
  return ((uint64_t)hi << 32) | lo;
}

template <int Ctrl, int RowMask>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, Ctrl, RowMask, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), Ctrl, RowMask, 0xF, false);
  return ((uint64_t)hi << 32) | lo;
}

// Sum over the 64 lanes of a wave (all active) into lane 63, by DPP row operations.
__device__ __forceinline__ uint64_t gl_wave_sum63(uint64_t v) {
  v = gl_add(v, dpp_u64<0xB1, 0xF>(v));   // quad_perm [1,0,3,2]
  v = gl_add(v, dpp_u64<0x4E, 0xF>(v));   // quad_perm [2,3,0,1]
  v = gl_add(v, dpp_u64<0x141, 0xF>(v));  // row_half_mirror
  v = gl_add(v, dpp_u64<0x140, 0xF>(v));  // row_mirror
  v = gl_add(v, dpp_u64<0x142, 0xA>(v));  // row_bcast15 into rows 1 and 3
  v = gl_add(v, dpp_u64<0x143, 0xC>(v));  // row_bcast31 into rows 2 and 3
  return v;
}

// Sum of NV values over the workgroup (blockDim.x a multiple of 64); valid in thread 0.
template <int NV>
__device__ __forceinline__ void gl_block_sum(uint64_t (&v)[NV]) {
  __shared__ uint64_t red[NV][16];
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = gl_wave_sum63(v[k]);
  const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  if (lane == 63)
#pragma unroll
    for (int k = 0; k < NV; ++k) red[k][wid] = v[k];
  __syncthreads();
  if (threadIdx.x == 0)
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      uint64_t a = red[k][0];
      for (uint32_t w = 1; w < nw; ++w) a = gl_add(a, red[k][w]);
      v[k] = a;
    }
  __syncthreads();
}

// ---------------------------------------------------------------- transcript (device)

// The transcript runs in whole waves (sha256_wave.hpp): v = LE64 of the first
// two digest words, which the a-lanes hold.
__device__ __forceinline__ uint64_t gl_candidate(const ShaLanes& s) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)s.x[0], 8);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)s.x[1], 8);
  return (uint64_t)bswap32(lo) | ((uint64_t)bswap32(hi) << 32);
}

__device__ __forceinline__ uint64_t gl_accept_wave(ShaLanes& st) {
  uint64_t v = gl_candidate(st);
  for (int attempt = 0; attempt < 4096 && v >= kGlP; ++attempt) {
    sha_rehash_wave(st, sha_buf());
    v = gl_candidate(st);
  }
  return v;
}

__device__ __forceinline__ uint64_t gl_squeeze_wave(ShaLanes& st) {
  sha_rehash_wave(st, sha_buf());
  return gl_accept_wave(st);
}

// Word `lane mod 16` of the block that absorbs a round: e0, e2 and the end mark.
__device__ __forceinline__ uint32_t gl_round_word(uint64_t e0, uint64_t e2) {
  const uint32_t li = threadIdx.x & 15;
  const uint64_t e = li < 2 ? e0 : e2;
  const uint32_t v = (li & 1) ? (uint32_t)(e >> 32) : (uint32_t)e;
  return li < 4 ? bswap32(v) : (li == 15 ? 1u : 0u);
}

// SHA-256 of `len` 32-bit words (byte-swapped when swap: element words are
// little-endian) with the standard padding.
__device__ void sha256_words(const uint32_t* in, uint64_t len, int swap, uint32_t* out) {
  Sha256State sh = sha256_iv();
  const uint64_t full = len / 16;
  for (uint64_t b = 0; b < full; ++b) {
    Sha256Block blk;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const uint32_t v = in[b * 16 + i];
      blk.w[i] = swap ? bswap32(v) : v;
    }
    sh = sha256_compress_v(sh, blk);
  }
  const uint32_t rem = (uint32_t)(len - full * 16);
  Sha256Block blk;
#pragma unroll
  for (int i = 0; i < 16; ++i) blk.w[i] = 0;
  for (uint32_t i = 0; i < rem; ++i) {
    const uint32_t v = in[full * 16 + i];
    blk.w[i] = swap ? bswap32(v) : v;
  }
  blk.w[rem] = 0x80000000u;
  const uint64_t bits = len * 32;
  if (rem <= 13) {
    blk.w[14] = (uint32_t)(bits >> 32);
    blk.w[15] = (uint32_t)bits;
    sh = sha256_compress_v(sh, blk);
  } else {
    sh = sha256_compress_v(sh, blk);
#pragma unroll
    for (int i = 0; i < 16; ++i) blk.w[i] = 0;
    blk.w[14] = (uint32_t)(bits >> 32);
    blk.w[15] = (uint32_t)bits;
    sh = sha256_compress_v(sh, blk);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) out[k] = sh.h[k];
}

// ---------------------------------------------------------------- bodies

#define GTID ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x)
#define GSTRIDE ((uint64_t)gridDim.x * blockDim.x)
#define GTILE_ID ((uint64_t)tile * kBlock + threadIdx.x)
#define GTILE_STRIDE ((uint64_t)ntiles * kBlock)

// ST_GL_FORWARD: V[z*2^n + c] = W[x_z*2^n + c] (+ or *) W[y_z*2^n + c].
// p0 W, p1 V, p2 gate records (x | type << 31, y), u0 n, q0 count.
__global__ void __launch_bounds__(kBlock) k_gl_forward(Step st) {
  const uint64_t* __restrict__ W = P<const uint64_t*>(st, 0);
  uint64_t* __restrict__ V = P<uint64_t*>(st, 1);
  const uint2* __restrict__ gates = P<const uint2*>(st, 2);
  const uint32_t n = st.u[0];
  const uint64_t mask = (1ull << n) - 1;
  for (uint64_t g = GTID; g < st.q[0]; g += GSTRIDE) {
    const uint2 gate = gates[g >> n];
    const uint64_t c = g & mask;
    const uint64_t a = gld(W, ((uint64_t)(gate.x & 0x7fffffffu) << n) | c), b = gld(W, ((uint64_t)gate.y << n) | c);
    gst(V, g, (gate.x >> 31) ? gl_mul(a, b) : gl_add(a, b));
  }
}

// ST_GL_DIGEST: one level of a tree digest; chunk t (256 words) hashed by thread t.
// p0 in, p1 out, q0 nwords, q1 nchunks, u0 swap; a second vector as in ST_DIGEST.
__global__ void __launch_bounds__(kBlock) k_gl_digest(Step st) {
  for (uint64_t g = GTID; g < st.q[1] + st.q[3]; g += GSTRIDE) {
    const bool second = g >= st.q[1];
    const uint32_t* in = second ? P<const uint32_t*>(st, 2) : P<const uint32_t*>(st, 0);
    uint32_t* out = second ? P<uint32_t*>(st, 3) : P<uint32_t*>(st, 1);
    const uint64_t nwords = second ? st.q[2] : st.q[0], t = second ? g - st.q[1] : g;
    const uint64_t begin = t * kChunkWords;
    const uint64_t end = (begin + kChunkWords < nwords) ? begin + kChunkWords : nwords;
    sha256_words(in + begin, end - begin, second ? st.u[1] : st.u[0], out + 8 * t);
  }
}

// ST_GL_BEGIN: st = seed state (w0..7), absorb the circuit digest (w8..15) and
// the two vector digests; the reduction counter starts at zero.
// p0 S, p1 dig_in, p2 dig_out.
__global__ void __launch_bounds__(kBlock) k_gl_begin(Step st) {
  if (threadIdx.x >= 64) return;
  GlState* S = P<GlState*>(st, 0);
  sha_init(sha_buf());
  const uint32_t k = threadIdx.x & 7;
  ShaLanes sh;
#pragma unroll
  for (int q = 0; q < 4; ++q) sh.x[q] = sha_sel((threadIdx.x & 8) != 0, st.w[q], st.w[4 + q]);
  Fr circ;
#pragma unroll
  for (int q = 0; q < 8; ++q) circ.v[q] = st.w[8 + q];
  sha_absorb_words_wave(sh, sha_buf(), kTagDigest, lane_limb(circ));
  sha_absorb_words_wave(sh, sha_buf(), kTagDigest, P<const uint32_t*>(st, 1)[k]);
  sha_absorb_words_wave(sh, sha_buf(), kTagDigest, P<const uint32_t*>(st, 2)[k]);
  sha_lanes_store(S->st, sh);
  if (threadIdx.x == 0) S->counter = 0;
}

// ST_GL_SQUEEZE: u0 challenges into p1. p0 S.
__global__ void __launch_bounds__(kBlock) k_gl_squeeze(Step st) {
  if (threadIdx.x >= 64) return;
  GlState* S = P<GlState*>(st, 0);
  uint64_t* out = P<uint64_t*>(st, 1);
  sha_init(sha_buf());
  ShaLanes sh = sha_lanes_load(S->st);
  for (uint32_t k = 0; k < st.u[0]; ++k) {
    const uint64_t v = gl_squeeze_wave(sh);
    if (threadIdx.x == 0) out[k] = v;
  }
  sha_lanes_store(S->st, sh);
}

// ST_GL_LAYER_BEGIN: alpha, beta squeezed (u0 = 0) and claim = alpha vu + beta vv;
// on layer 0 (u0 = 1) alpha = 1, beta = 0, claim = vu. p0 S, p1 vu, p2 vv.
__global__ void __launch_bounds__(kBlock) k_gl_layer_begin(Step st) {
  if (threadIdx.x >= 64) return;
  GlState* S = P<GlState*>(st, 0);
  const uint64_t vu = *P<const uint64_t*>(st, 1), vv = *P<const uint64_t*>(st, 2);
  uint64_t a = 1, b = 0;  // the output layer has one claim
  if (!st.u[0]) {
    sha_init(sha_buf());
    ShaLanes sh = sha_lanes_load(S->st);
    a = gl_squeeze_wave(sh);
    b = gl_squeeze_wave(sh);
    sha_lanes_store(S->st, sh);
  }
  const uint64_t claim = st.u[0] ? vu : gl_add(gl_mul(a, vu), gl_mul(b, vv));
  if (threadIdx.x == 0) {
    S->alpha = a;
    S->beta = b;
    S->claim = claim;
  }
}

// ST_GL_EQ: up to four tables out_j[b] = scale_j prod_k (bit_k(b) ? r_k : 1 - r_k),
// bit 1 the most significant. u0..3 bits, u4 count; p0..3 points, p4..7 scales
// (null = 1), p8..11 outs.
__global__ void __launch_bounds__(kBlock) k_gl_eq(Step st) {
  uint64_t total = 0;
  for (uint32_t j = 0; j < st.u[4]; ++j) total += 1ull << st.u[j];
  for (uint64_t g = GTID; g < total; g += GSTRIDE) {
    uint64_t t = g;
    uint32_t j = 0;
    while (t >= (1ull << st.u[j])) {
      t -= 1ull << st.u[j];
      ++j;
    }
    const uint64_t* r = P<const uint64_t*>(st, j);
    const int k = st.u[j];
    const uint64_t* scale = P<const uint64_t*>(st, 4 + j);
    uint64_t acc = scale ? *scale : 1;
    for (int i = 0; i < k; ++i) {
      const uint64_t ri = r[i];
      acc = gl_mul(acc, ((t >> (k - 1 - i)) & 1) ? ri : gl_one_minus(ri));
    }
    gst(P<uint64_t*>(st, 8 + j), t, acc);
  }
}


// ST_GL_WSUM: sum_e V[e] A[e >> n] B[e & mask] into *p5.
// p0 V, p1 A, p2 B, p3 partials, p4 S, p5 dst, u0 n, q0 count.
__global__ void __launch_bounds__(kBlock) k_gl_wsum(Step st) {
  const uint64_t* V = P<const uint64_t*>(st, 0);
  const uint64_t* A = P<const uint64_t*>(st, 1);
  const uint64_t* B = P<const uint64_t*>(st, 2);
  uint64_t* partials = P<uint64_t*>(st, 3);
  GlState* S = P<GlState*>(st, 4);
  const uint32_t n = st.u[0];
  const uint64_t mask = (1ull << n) - 1;
  uint64_t acc[1] = {0};
  for (uint64_t e = GTID; e < st.q[0]; e += GSTRIDE)
    acc[0] = gl_add(acc[0], gl_mul(gl_mul(gld(V, e), gld(A, e >> n)), gld(B, e & mask)));
  gl_block_sum<1>(acc);
  if (threadIdx.x == 0) put_word(partials + blockIdx.x, acc[0]);
  if (last_tile(&S->counter, gridDim.x)) {
    uint64_t tot[1] = {0};
    for (uint32_t b = threadIdx.x; b < gridDim.x; b += blockDim.x) tot[0] = gl_add(tot[0], get_word(partials + b));
    gl_block_sum<1>(tot);
    if (threadIdx.x == 0) *P<uint64_t*>(st, 5) = tot[0];
  }
}

// ST_GL_P1: phase-1 tables over (x, c), T[z,c] = aU[z] Cu[c] + bV[z] Cv[c]:
//   G[x,c] = sum_{MUL z: x_z=x} T W[y_z,c] + sum_{ADD z: x_z=x} T,  H[x,c] = sum_{ADD} T W[y_z,c].
// p0 W, p1 G, p2 H, p3 xrow, p4 xent (z, y | type << 31), p5 aU, p6 bV, p7 Cu, p8 Cv, u0 n, q0 count.
__global__ void __launch_bounds__(kBlock) k_gl_p1(Step st) {
  const uint64_t* __restrict__ W = P<const uint64_t*>(st, 0);
  uint64_t* __restrict__ G = P<uint64_t*>(st, 1);
  uint64_t* __restrict__ H = P<uint64_t*>(st, 2);
  const uint32_t* __restrict__ xrow = P<const uint32_t*>(st, 3);
  const uint2* __restrict__ xent = P<const uint2*>(st, 4);
  const uint64_t *aU = P<const uint64_t*>(st, 5), *bV = P<const uint64_t*>(st, 6);
  const uint64_t *Cu = P<const uint64_t*>(st, 7), *Cv = P<const uint64_t*>(st, 8);
  const uint32_t n = st.u[0];
  const uint64_t mask = (1ull << n) - 1;
  for (uint64_t e = GTID; e < st.q[0]; e += GSTRIDE) {
    const uint64_t x = e >> n, c = e & mask;
    const uint64_t cu = gld(Cu, c), cv = gld(Cv, c);
    uint64_t g = 0, h = 0;
    const uint32_t k1 = xrow[x + 1];
    for (uint32_t k = xrow[x]; k < k1; ++k) {
      const uint2 r = xent[k];
      const uint64_t T = gl_add(gl_mul(gld(aU, r.x), cu), gl_mul(gld(bV, r.x), cv));
      const uint64_t tw = gl_mul(T, gld(W, ((uint64_t)(r.y & 0x7fffffffu) << n) | c));
      if (r.y >> 31) {
        g = gl_add(g, tw);
      } else {
        g = gl_add(g, T);
        h = gl_add(h, tw);
      }
    }
    gst(G, e, g);
    gst(H, e, h);
  }
}

// ---------------------------------------------------------------- phase 2
//
// Phase 2 sums W[y,c] F[y,c] + K[y,c] over (y, c). With the copy weights
// U[c] = EC[c] Cu[c], V[c] = EC[c] Cv[c] both tables have rank 2 per copy:
//   F[y,c] = U[c] Fa[y] + V[c] Fb[y],  K[y,c] = U[c] Ka[y] + V[c] Kb[y],
//   Fa = vx Mu + Au, Fb = vx Mv + Av, Ka = vx Au, Kb = vx Av, where
//   Mu[y] = sum_{MUL z: y_z = y} aU[z] EL[x_z] (Mv with bV; Au, Av over ADD gates).
// The sub-circuit rounds therefore run on the 2^sigma tables
//   sum_y P[y] Fa[y] + Q[y] Fb[y] + Ks[y],  P = sum_c U[c] W[., c], Q = sum_c V[c] W[., c],
//   Ks = su Ka + sv Kb (su = sum_c U[c], sv = sum_c V[c]),
// and the copy rounds on Wc[c] = W(ry_local, c), Fc[c] = U[c] Fa~ + V[c] Fb~,
// Kc[c] = U[c] Ka~ + V[c] Kb~: the same round polynomials as over the whole
// layer, with two passes over W instead of a pass per round.

// ST_GL_COPY_WEIGHTS (one workgroup): U = EC Cu, V = EC Cv for c < q0, and
// their sums into S->su, S->sv. p0 EC, p1 Cu, p2 Cv, p3 U, p4 V, p5 S.
__global__ void __launch_bounds__(kBlock) k_gl_copy_weights(Step st) {
  const uint64_t *EC = P<const uint64_t*>(st, 0), *Cu = P<const uint64_t*>(st, 1), *Cv = P<const uint64_t*>(st, 2);
  uint64_t *U = P<uint64_t*>(st, 3), *V = P<uint64_t*>(st, 4);
  GlState* S = P<GlState*>(st, 5);
  uint64_t acc[2] = {0, 0};
  for (uint64_t c = threadIdx.x; c < st.q[0]; c += blockDim.x) {
    const uint64_t e = gld(EC, c);
    const uint64_t u = gl_mul(e, gld(Cu, c)), v = gl_mul(e, gld(Cv, c));
    gst(U, c, u);
    gst(V, c, v);
    acc[0] = gl_add(acc[0], u);
    acc[1] = gl_add(acc[1], v);
  }
  gl_block_sum<2>(acc);
  if (threadIdx.x == 0) {
    S->su = acc[0];
    S->sv = acc[1];
  }
}

// ST_GL_P2T: the 2^sigma phase-2 tables for y < q0 from the wiring by y.
// p0 yrow, p1 yent (z, x | type << 31), p2 aU, p3 bV, p4 EL, p5 S,
// p6 Fa, p7 Fb, p8 Ka, p9 Kb, p10 Ks.
__device__ __forceinline__ void body_gl_p2t(const Step& st, uint32_t tile, uint32_t ntiles) {
  const uint32_t* __restrict__ yrow = P<const uint32_t*>(st, 0);
  const uint2* __restrict__ yent = P<const uint2*>(st, 1);
  const uint64_t *aU = P<const uint64_t*>(st, 2), *bV = P<const uint64_t*>(st, 3), *EL = P<const uint64_t*>(st, 4);
  const GlState* S = P<const GlState*>(st, 5);
  const uint64_t vx = S->vx, su = S->su, sv = S->sv;
  for (uint64_t y = GTILE_ID; y < st.q[0]; y += GTILE_STRIDE) {
    uint64_t mu = 0, mv = 0, au = 0, av = 0;
    const uint32_t k1 = yrow[y + 1];
    for (uint32_t k = yrow[y]; k < k1; ++k) {
      const uint2 r = yent[k];
      const uint64_t e = gld(EL, r.y & 0x7fffffffu);
      const uint64_t tu = gl_mul(gld(aU, r.x), e), tv = gl_mul(gld(bV, r.x), e);
      if (r.y >> 31) {
        mu = gl_add(mu, tu);
        mv = gl_add(mv, tv);
      } else {
        au = gl_add(au, tu);
        av = gl_add(av, tv);
      }
    }
    const uint64_t ka = gl_mul(vx, au), kb = gl_mul(vx, av);
    gst(P<uint64_t*>(st, 6), y, gl_add(gl_mul(vx, mu), au));
    gst(P<uint64_t*>(st, 7), y, gl_add(gl_mul(vx, mv), av));
    gst(P<uint64_t*>(st, 8), y, ka);
    gst(P<uint64_t*>(st, 9), y, kb);
    gst(P<uint64_t*>(st, 10), y, gl_add(gl_mul(su, ka), gl_mul(sv, kb)));
  }
}
__global__ void __launch_bounds__(kBlock) k_gl_p2t(Step st) { body_gl_p2t(st, blockIdx.x, gridDim.x); }

// Sum over the wave; valid in every lane.
__device__ __forceinline__ uint64_t gl_wave_sum(uint64_t v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = gl_add(v, shfl_xor_u64(v, off));
  return v;
}

// ST_GL_COPY_CONTRACT: P[y] = sum_c U[c] W[y 2^n + c], Q[y] likewise with V,
// one wave per row y < q0, two adjacent copies per lane (16-byte loads) from 2^7
// copies up. p0 W, p1 U, p2 V, p3 P, p4 Q, u0 n.
__device__ __forceinline__ void body_gl_copy_contract(const Step& st, uint32_t tile, uint32_t ntiles) {
  const uint64_t *W = P<const uint64_t*>(st, 0), *U = P<const uint64_t*>(st, 1), *V = P<const uint64_t*>(st, 2);
  const uint32_t n = st.u[0];
  const uint64_t ncop = 1ull << n;
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t wave = GTILE_ID >> 6, nwaves = GTILE_STRIDE >> 6;
  if (n < 7) {
    // one product per lane at most: an unreduced sum's own reduction would cost more
    // (2^22 rows of one entry: 2.6 ms a layer instead of 1.6)
    for (uint64_t y = wave; y < st.q[0]; y += nwaves) {
      uint64_t p = 0, q = 0;
      if (lane < ncop) {
        const uint64_t w = gld(W, (y << n) | lane);
        p = gl_mul(gld(U, lane), w);
        q = gl_mul(gld(V, lane), w);
      }
      p = gl_wave_sum(p);
      q = gl_wave_sum(q);
      if (lane == 0) {
        gst(P<uint64_t*>(st, 3), y, p);
        gst(P<uint64_t*>(st, 4), y, q);
      }
    }
    return;
  }
  for (uint64_t y = wave; y < st.q[0]; y += nwaves) {
    GlAcc ps, qs;
    for (uint64_t c = 2 * lane; c < ncop; c += 128) {
      const U64x2 w = gld2(W, (y << n) | c), u = gld2(U, c), v = gld2(V, c);
      gl_mac(ps, u.x, w.x);
      gl_mac(qs, v.x, w.x);
      gl_mac(ps, u.y, w.y);
      gl_mac(qs, v.y, w.y);
    }
    const uint64_t p = gl_wave_sum(gl_acc_value(ps)), q = gl_wave_sum(gl_acc_value(qs));
    if (lane == 0) {
      gst(P<uint64_t*>(st, 3), y, p);
      gst(P<uint64_t*>(st, 4), y, q);
    }
  }
}
__global__ void __launch_bounds__(kBlock) k_gl_copy_contract(Step st) { body_gl_copy_contract(st, blockIdx.x, gridDim.x); }

// ST_GL_LOCAL_VALUES: Ka~ = sum_y EqR[y] Ka[y], Kb~ likewise, y < q0, into S->ka_f,
// S->kb_f, a workgroup per 2^14 rows: a row is a chain of loads and a product, so
// one workgroup over 2^22 rows took 10 ms. p0 EqR, p1 Ka, p2 Kb, p3 S, p4 partials.
constexpr uint64_t kGlLocalValueRows = 1u << 14;

__device__ __forceinline__ void body_gl_local_values(const Step& st, uint32_t tile, uint32_t ntiles) {
  const uint64_t *E = P<const uint64_t*>(st, 0), *Ka = P<const uint64_t*>(st, 1), *Kb = P<const uint64_t*>(st, 2);
  GlState* S = P<GlState*>(st, 3);
  uint64_t acc[2] = {0, 0};
  for (uint64_t y = GTILE_ID; y < st.q[0]; y += GTILE_STRIDE) {
    const uint64_t e = gld(E, y);
    acc[0] = gl_add(acc[0], gl_mul(e, gld(Ka, y)));
    acc[1] = gl_add(acc[1], gl_mul(e, gld(Kb, y)));
  }
  gl_block_sum<2>(acc);
  if (ntiles > 1) {
    uint64_t* partials = P<uint64_t*>(st, 4);
    if (threadIdx.x == 0) {
      put_word(partials + 2 * tile, acc[0]);
      put_word(partials + 2 * tile + 1, acc[1]);
    }
    if (!last_tile(&S->counter, ntiles)) return;
    acc[0] = acc[1] = 0;
    for (uint32_t b = threadIdx.x; b < ntiles; b += kBlock) {
      acc[0] = gl_add(acc[0], get_word(partials + 2 * b));
      acc[1] = gl_add(acc[1], get_word(partials + 2 * b + 1));
    }
    gl_block_sum<2>(acc);
  }
  if (threadIdx.x == 0) {
    S->ka_f = acc[0];
    S->kb_f = acc[1];
  }
}
__global__ void __launch_bounds__(kBlock) k_gl_local_values(Step st) { body_gl_local_values(st, blockIdx.x, gridDim.x); }

// ST_GL_LOCAL_CONTRACT: part[ch 2^n + c] = sum over the 2^u1 rows y of chunk
// ch of EqR[y] W[y 2^n + c], for ch 2^n + c < q0. p0 W, p1 EqR, p2 part, u0 n.
// Two adjacent columns per thread (n >= 1). Bound by memory; with reduced
// products and 8-byte loads 2^26 entries took 174 us.
__device__ __forceinline__ void body_gl_local_contract(const Step& st, uint32_t tile, uint32_t ntiles) {
  const uint64_t *W = P<const uint64_t*>(st, 0), *E = P<const uint64_t*>(st, 1);
  uint64_t* part = P<uint64_t*>(st, 2);
  const uint32_t n = st.u[0], lr = st.u[1];
  const uint64_t mask = (1ull << n) - 1;
  if (n == 0) {
    for (uint64_t g = GTILE_ID; g < st.q[0]; g += GTILE_STRIDE) {
      GlAcc acc;
      for (uint64_t y = g << lr; y < (g + 1) << lr; ++y) gl_mac(acc, gld(E, y), gld(W, y));
      gst(part, g, gl_acc_value(acc));
    }
    return;
  }
  for (uint64_t g = 2 * GTILE_ID; g < st.q[0]; g += 2 * GTILE_STRIDE) {
    const uint64_t ch = g >> n, c = g & mask;
    const uint64_t y0 = ch << lr, y1 = y0 + (1ull << lr);
    GlAcc a, b;
    for (uint64_t y = y0; y < y1; ++y) {
      const U64x2 w = gld2(W, (y << n) | c);
      const uint64_t e = gld(E, y);
      gl_mac(a, e, w.x);
      gl_mac(b, e, w.y);
    }
    gst2(part, g, U64x2{gl_acc_value(a), gl_acc_value(b)});
  }
}
__global__ void __launch_bounds__(kBlock) k_gl_local_contract(Step st) { body_gl_local_contract(st, blockIdx.x, gridDim.x); }

// ST_GL_COPY_TABLES: for c < q0, Wc[c] = sum of the u0 chunk partials,
// Fc = U Fa~ + V Fb~, Kc = U Ka~ + V Kb~ (Fa~, Fb~ the first entries of the
// folded Fa, Fb tables). p0 part, p1 U, p2 V, p3 Fa, p4 Fb, p5 S, p6 Wc, p7 Fc, p8 Kc.
// tpc lanes (up to a wave) per column, summed with shuffles inside aligned
// lane groups: few copies come with many chunks.
__global__ void __launch_bounds__(kBlock) k_gl_copy_tables(Step st) {
  const uint64_t* part = P<const uint64_t*>(st, 0);
  const uint64_t *U = P<const uint64_t*>(st, 1), *V = P<const uint64_t*>(st, 2);
  const uint64_t fa = *P<const uint64_t*>(st, 3), fb = *P<const uint64_t*>(st, 4);
  const GlState* S = P<const GlState*>(st, 5);
  const uint64_t ka = S->ka_f, kb = S->kb_f, ncop = st.q[0];
  const uint32_t R = st.u[0];
  const uint32_t rlog = 31 - __clz(R);
  const uint32_t tpc_log = rlog < 6 ? rlog : 6;
  const uint32_t tpc = 1u << tpc_log, lane = threadIdx.x & (tpc - 1);
  const uint64_t cols_per_tile = kBlock >> tpc_log;
  const uint32_t tile = blockIdx.x, ntiles = gridDim.x;
  for (uint64_t base = (uint64_t)tile * cols_per_tile; base < ncop; base += (uint64_t)ntiles * cols_per_tile) {
    const uint64_t c = base + (threadIdx.x >> tpc_log);
    uint64_t w = 0;
    if (c < ncop)
      for (uint32_t ch = lane; ch < R; ch += tpc) w = gl_add(w, gld(part, (uint64_t)ch * ncop + c));
    for (uint32_t off = tpc / 2; off >= 1; off >>= 1) {
      const uint64_t o = ((uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)(w >> 32), off, 64) << 32) |
                         (uint32_t)__shfl_xor((int)(uint32_t)w, off, 64);
      w = gl_add(w, o);
    }
    if (lane == 0 && c < ncop) {
      const uint64_t u = gld(U, c), v = gld(V, c);
      gst(P<uint64_t*>(st, 6), c, w);
      gst(P<uint64_t*>(st, 7), c, gl_add(gl_mul(u, fa), gl_mul(v, fb)));
      gst(P<uint64_t*>(st, 8), c, gl_add(gl_mul(u, ka), gl_mul(v, kb)));
    }
  }
}

// ---------------------------------------------------------------- rounds

// The transcript step of a grid round (the whole workgroup; e0, e2 in thread
// 0): the hash in wave 0 with its schedule from wave 2 gives r; then the
// message (e0, e1 = claim - e0, e2) and the claim at r.
__device__ __forceinline__ void gl_round_step(GlState* S, uint64_t e0, uint64_t e2, uint64_t* r_out, uint64_t* msg) {
  __shared__ uint64_t e_sh[2];
  __shared__ ShaHelper help;
  const uint32_t wid = threadIdx.x >> 6;
  ShaLanes sh;
  if (wid == 0) {
    sh = sha_lanes_load(S->st);
    sha_init(sha_buf());
  }
  if (threadIdx.x == 0) {
    e_sh[0] = e0;
    e_sh[1] = e2;
    help.ready = 0;
  }
  __syncthreads();
  const uint64_t f0 = e_sh[0], f2 = e_sh[1];
  if (wid == 2) {
    sha_help(gl_round_word(f0, f2), sha_buf(), &help, 0);
  } else if (wid == 0) {
    const uint64_t claim = S->claim;
    sh = sha_compress_wave<true>(sh, gl_round_word(f0, f2), sha_buf(), &help, 0);
    const uint64_t r = gl_accept_wave(sh);
    sha_lanes_store(S->st, sh);
    if (threadIdx.x == 0) {
      const uint64_t e1 = gl_sub(claim, f0);
      *r_out = r;
      msg[0] = f0;
      msg[1] = e1;
      msg[2] = f2;
      S->claim = gl_interp3(f0, e1, f2, r);
    }
  }
}

// The summand of a round over NT tables at one point: T0 T1 + T2 (NT = 3) or
// T0 T1 + T2 T3 + T4 (NT = 5).
template <int NT>
__device__ __forceinline__ uint64_t gl_form(const uint64_t (&v)[NT]) {
  if constexpr (NT == 3) return gl_add(gl_mul(v[0], v[1]), v[2]);
  else return gl_add(gl_add(gl_mul(v[0], v[1]), gl_mul(v[2], v[3])), v[4]);
}

// Evaluation of pair b of NT tables at t = 0 and t = 2, after an optional
// fold of the source by r (entry i of the folded table is
// src[i] + r (src[i + 2 half] - src[i])).
template <int NT>
__device__ __forceinline__ void gl_pair(const uint64_t* const* src, uint64_t* const* dst, bool fold, uint64_t r,
                                        uint64_t b, uint64_t half, uint64_t& acc0, uint64_t& acc2) {
  uint64_t lo[NT], hi[NT];
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    if (fold) {
      const uint64_t m = 2 * half;
      const uint64_t a0 = gld(src[k], b), a1 = gld(src[k], b + m);
      const uint64_t b0 = gld(src[k], b + half), b1 = gld(src[k], b + half + m);
      lo[k] = gl_add(a0, gl_mul(r, gl_sub(a1, a0)));
      hi[k] = gl_add(b0, gl_mul(r, gl_sub(b1, b0)));
      gst(dst[k], b, lo[k]);
      gst(dst[k], b + half, hi[k]);
    } else {
      lo[k] = gld(src[k], b);
      hi[k] = gld(src[k], b + half);
    }
  }
  acc0 = gl_add(acc0, gl_form<NT>(lo));
  uint64_t t2[NT];
#pragma unroll
  for (int k = 0; k < NT; ++k) t2[k] = gl_sub(gl_double(hi[k]), lo[k]);
  acc2 = gl_add(acc2, gl_form<NT>(t2));
}

// Pairs b and b + 1 (b even, half even) of NT tables: gl_pair for both, with
// 16-byte loads and stores.
template <int NT>
__device__ __forceinline__ void gl_pair2(const uint64_t* const* src, uint64_t* const* dst, bool fold, uint64_t r,
                                         uint64_t b, uint64_t half, uint64_t& acc0, uint64_t& acc2) {
  uint64_t lo[2][NT], hi[2][NT];
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    if (fold) {
      const uint64_t m = 2 * half;
      const U64x2 a0 = gld2(src[k], b), a1 = gld2(src[k], b + m);
      const U64x2 b0 = gld2(src[k], b + half), b1 = gld2(src[k], b + half + m);
      lo[0][k] = gl_add(a0.x, gl_mul(r, gl_sub(a1.x, a0.x)));
      lo[1][k] = gl_add(a0.y, gl_mul(r, gl_sub(a1.y, a0.y)));
      hi[0][k] = gl_add(b0.x, gl_mul(r, gl_sub(b1.x, b0.x)));
      hi[1][k] = gl_add(b0.y, gl_mul(r, gl_sub(b1.y, b0.y)));
      gst2(dst[k], b, U64x2{lo[0][k], lo[1][k]});
      gst2(dst[k], b + half, U64x2{hi[0][k], hi[1][k]});
    } else {
      const U64x2 a = gld2(src[k], b), c = gld2(src[k], b + half);
      lo[0][k] = a.x;
      lo[1][k] = a.y;
      hi[0][k] = c.x;
      hi[1][k] = c.y;
    }
  }
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    acc0 = gl_add(acc0, gl_form<NT>(lo[e]));
    uint64_t t2[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) t2[k] = gl_sub(gl_double(hi[e][k]), lo[e][k]);
    acc2 = gl_add(acc2, gl_form<NT>(t2));
  }
}

// The end of a grid round: the workgroup's sums, and in the last tile the total
// and the round's transcript step.
__device__ __forceinline__ void gl_finish_round(uint64_t (&acc)[2], GlState* S, uint64_t* partials, uint64_t* r_out,
                                                uint64_t* msg) {
  gl_block_sum<2>(acc);
  if (threadIdx.x == 0) {
    put_word(partials + 2 * blockIdx.x, acc[0]);
    put_word(partials + 2 * blockIdx.x + 1, acc[1]);
  }
  if (last_tile(&S->counter, gridDim.x)) {
    uint64_t tot[2] = {0, 0};
    for (uint32_t b = threadIdx.x; b < gridDim.x; b += blockDim.x) {
      tot[0] = gl_add(tot[0], get_word(partials + 2 * b));
      tot[1] = gl_add(tot[1], get_word(partials + 2 * b + 1));
    }
    gl_block_sum<2>(tot);
    gl_round_step(S, tot[0], tot[1], r_out, msg);
  }
}

// ST_GL_ROUND (NT = 3) / ST_GL_ROUND5 (NT = 5): one grid-wide round of the
// NT-table sum (optional fold by the previous challenge, evaluation at
// t = 0, 2), then in the last tile the round's transcript step. p0..p(NT-1)
// src, pNT..p(2NT-1) dst, then (from B = 2 NT) pB rprev (null: no fold),
// pB+1 S, pB+2 partials, pB+3 r_out, pB+4 msg; q0 half.
template <int NT>
__global__ void __launch_bounds__(kBlock) k_gl_round(Step st) {
  constexpr int B = 2 * NT;
  const uint64_t* src[NT];
  uint64_t* dst[NT];
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    src[k] = P<const uint64_t*>(st, k);
    dst[k] = P<uint64_t*>(st, NT + k);
  }
  const uint64_t* rprev = P<const uint64_t*>(st, B);
  GlState* S = P<GlState*>(st, B + 1);
  uint64_t* partials = P<uint64_t*>(st, B + 2);
  const bool fold = rprev != nullptr;
  const uint64_t r = fold ? *rprev : 0;
  const uint64_t half = st.q[0];
  uint64_t acc[2] = {0, 0};
  if ((half & 1) == 0) {
    for (uint64_t b = 2 * GTID; b < half; b += 2 * GSTRIDE) gl_pair2<NT>(src, dst, fold, r, b, half, acc[0], acc[1]);
  } else {
    for (uint64_t b = GTID; b < half; b += GSTRIDE) gl_pair<NT>(src, dst, fold, r, b, half, acc[0], acc[1]);
  }
  gl_finish_round(acc, S, partials, P<uint64_t*>(st, B + 3), P<uint64_t*>(st, B + 4));
}

// ---------------------------------------------------------------- contracted phase 1
//
// Phase 1 with the addition gates contracted over the copies, as in the BN254
// prover (gkr_split.hip states the identities): tables over (x, c) only for W and
// the MUL gates' Gm, whose rows without a MUL gate are neither read nor
// written; the ADD gates in five 2^sigma tables; two more passes over W.

__device__ __forceinline__ bool gl_row_active(const uint32_t* act, uint32_t k, uint32_t row) {
  const uint32_t bit = (1u << k) + row;
  return (act[bit >> 5] >> (bit & 31)) & 1u;
}

// ST_GL_S_SMALL: sa, sb, h over the ADD gates of x < q0. p0 xrow, p1 xmid, p2 xent,
// p3 aU, p4 bV, p5 Pu, p6 Pv, p7 sa, p8 sb, p9 h.
__global__ void __launch_bounds__(kBlock) k_gl_s_small(Step st) {
  const uint32_t* __restrict__ xrow = P<const uint32_t*>(st, 0);
  const uint32_t* __restrict__ xmid = P<const uint32_t*>(st, 1);
  const uint2* __restrict__ xent = P<const uint2*>(st, 2);
  const uint64_t *aU = P<const uint64_t*>(st, 3), *bV = P<const uint64_t*>(st, 4);
  const uint64_t *Pu = P<const uint64_t*>(st, 5), *Pv = P<const uint64_t*>(st, 6);
  for (uint64_t x = GTID; x < st.q[0]; x += GSTRIDE) {
    uint64_t sa = 0, sb = 0, h = 0;
    const uint32_t k1 = xrow[x + 1];
    for (uint32_t k = xmid[x]; k < k1; ++k) {
      const uint2 e = xent[k];
      const uint64_t y = e.y & 0x7fffffffu, a = gld(aU, e.x), b = gld(bV, e.x);
      sa = gl_add(sa, a);
      sb = gl_add(sb, b);
      h = gl_add(h, gl_add(gl_mul(a, gld(Pu, y)), gl_mul(b, gld(Pv, y))));
    }
    gst(P<uint64_t*>(st, 7), x, sa);
    gst(P<uint64_t*>(st, 8), x, sb);
    gst(P<uint64_t*>(st, 9), x, h);
  }
}

// Two adjacent entries (x, c), (x, c + 1) of Gm over x's MUL gates (at least one).
__device__ __forceinline__ U64x2 gl_split_entry(const uint64_t* __restrict__ W, const uint2* __restrict__ xent,
                                                const uint64_t* __restrict__ aU, const uint64_t* __restrict__ bV,
                                                U64x2 cu, U64x2 cv, uint32_t k0, uint32_t k1, uint32_t n, uint64_t c) {
  U64x2 g = {0, 0};
  for (uint32_t k = k0; k < k1; ++k) {
    const uint2 e = xent[k];
    const uint64_t a = gld(aU, e.x), b = gld(bV, e.x);
    const U64x2 w = gld2(W, ((uint64_t)(e.y & 0x7fffffffu) << n) | c);
    g.x = gl_add(g.x, gl_mul(gl_add(gl_mul(a, cu.x), gl_mul(b, cv.x)), w.x));
    g.y = gl_add(g.y, gl_mul(gl_add(gl_mul(a, cu.y), gl_mul(b, cv.y)), w.y));
  }
  return g;
}

__device__ __forceinline__ U64x2 gl_fold2(uint64_t r, U64x2 a0, U64x2 a1) {
  return U64x2{gl_add(a0.x, gl_mul(r, gl_sub(a1.x, a0.x))), gl_add(a0.y, gl_mul(r, gl_sub(a1.y, a0.y)))};
}
__device__ __forceinline__ U64x2 gl_at2(U64x2 lo, U64x2 hi) {  // 2 hi - lo
  return U64x2{gl_sub(gl_double(hi.x), lo.x), gl_sub(gl_double(hi.y), lo.y)};
}
__device__ __forceinline__ uint64_t gl_dot2(U64x2 a, U64x2 b) { return gl_add(gl_mul(a.x, b.x), gl_mul(a.y, b.y)); }

// ST_GL_S_INIT_ROUND: Gm and round 1. Tiles below u1 take the pairs b < q0 of the
// (x, c) table, two adjacent ones per thread; the others the q1 pairs of the
// small tables. p0 W, p1 G, p2 xrow, p3 xmid, p4 xent, p5 aU, p6 bV, p7 Cu, p8 Cv,
// p9 S, p10 partials, p11 r_out, p12 msg, p13 the first small table, w0..w4 the
// entry offsets of all five from it; u0 n.
__global__ void __launch_bounds__(kBlock) k_gl_s_init_round(Step st) {
  const uint32_t nb = st.u[1];
  uint64_t acc[2] = {0, 0};
  if (blockIdx.x < nb) {
    const uint64_t* __restrict__ W = P<const uint64_t*>(st, 0);
    uint64_t* __restrict__ G = P<uint64_t*>(st, 1);
    const uint32_t* __restrict__ xrow = P<const uint32_t*>(st, 2);
    const uint32_t* __restrict__ xmid = P<const uint32_t*>(st, 3);
    const uint2* __restrict__ xent = P<const uint2*>(st, 4);
    const uint64_t *aU = P<const uint64_t*>(st, 5), *bV = P<const uint64_t*>(st, 6);
    const uint32_t n = st.u[0];
    const uint64_t mask = (1ull << n) - 1, half = st.q[0];
    for (uint64_t b = 2 * GTID; b < half; b += 2ull * nb * kBlock) {
      // a wave's 128 entries lie in one row: its gates are the same in every lane
      const uint32_t x0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(b >> n)), x1 = x0 + (uint32_t)(half >> n);
      const uint64_t c = b & mask;
      const uint32_t a0 = xrow[x0], e0 = xmid[x0], a1 = xrow[x1], e1 = xmid[x1];
      if (a0 == e0 && a1 == e1) continue;
      const U64x2 cu = gld2(P<const uint64_t*>(st, 7), c), cv = gld2(P<const uint64_t*>(st, 8), c);
      const U64x2 w0 = gld2(W, b), w1 = gld2(W, b + half);
      U64x2 g0 = {0, 0}, g1 = {0, 0};
      if (a0 != e0) {
        g0 = gl_split_entry(W, xent, aU, bV, cu, cv, a0, e0, n, c);
        gst2(G, b, g0);
        acc[0] = gl_add(acc[0], gl_dot2(w0, g0));
      }
      if (a1 != e1) {
        g1 = gl_split_entry(W, xent, aU, bV, cu, cv, a1, e1, n, c);
        gst2(G, b + half, g1);
      }
      acc[1] = gl_add(acc[1], gl_dot2(gl_at2(w0, w1), gl_at2(g0, g1)));
    }
  } else {
    const uint64_t* src[5];
    uint64_t* dst[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      src[k] = P<const uint64_t*>(st, 13) + st.w[k];
      dst[k] = nullptr;
    }
    for (uint64_t b = (uint64_t)(blockIdx.x - nb) * kBlock + threadIdx.x; b < st.q[1];
         b += (uint64_t)(gridDim.x - nb) * kBlock)
      gl_pair<5>(src, dst, false, 0, b, st.q[1], acc[0], acc[1]);
  }
  gl_finish_round(acc, P<GlState*>(st, 9), P<uint64_t*>(st, 10), P<uint64_t*>(st, 11), P<uint64_t*>(st, 12));
}

// ST_GL_S_ROUND: a later round: folds by the pending challenge and evaluates.
// p0 W src, p1 W dst, p2 G (in place), p3 act, p4..p8 small tables (in place),
// p9 S, p10 partials, p11 r_out, p12 msg, p13 rprev; u0 n, u1 tiles of the big
// part, u2 k (2^k rows before this round's pairing); q0 pairs, q1 small pairs.
__global__ void __launch_bounds__(kBlock) k_gl_s_round(Step st) {
  const uint32_t nb = st.u[1];
  const uint64_t r = *P<const uint64_t*>(st, 13);
  uint64_t acc[2] = {0, 0};
  if (blockIdx.x < nb) {
    const uint64_t* Ws = P<const uint64_t*>(st, 0);  // from the third round on the same table as Wd
    uint64_t *Wd = P<uint64_t*>(st, 1), *G = P<uint64_t*>(st, 2);
    const uint32_t* __restrict__ act = P<const uint32_t*>(st, 3);
    const uint32_t n = st.u[0], k = st.u[2], rh = 1u << (k - 1);
    const uint64_t half = st.q[0], m = 2 * half;
    for (uint64_t b = 2 * GTID; b < half; b += 2ull * nb * kBlock) {
      const uint32_t x = (uint32_t)__builtin_amdgcn_readfirstlane((int)(b >> n));
      const bool f00 = gl_row_active(act, k + 1, x), f01 = gl_row_active(act, k + 1, x + 2 * rh);
      const bool f10 = gl_row_active(act, k + 1, x + rh), f11 = gl_row_active(act, k + 1, x + 3 * rh);
      const U64x2 a0 = gld2(Ws, b), a1 = gld2(Ws, b + m), c0 = gld2(Ws, b + half), c1 = gld2(Ws, b + half + m);
      U64x2 g00 = {0, 0}, g01 = {0, 0}, g10 = {0, 0}, g11 = {0, 0};
      if (f00) g00 = gld2(G, b);
      if (f01) g01 = gld2(G, b + m);
      if (f10) g10 = gld2(G, b + half);
      if (f11) g11 = gld2(G, b + half + m);
      const U64x2 wl = gl_fold2(r, a0, a1), wh = gl_fold2(r, c0, c1);
      gst2(Wd, b, wl);
      gst2(Wd, b + half, wh);
      U64x2 gl = {0, 0}, gh = {0, 0};
      if (f00 || f01) {
        gl = gl_fold2(r, g00, g01);
        gst2(G, b, gl);
        acc[0] = gl_add(acc[0], gl_dot2(wl, gl));
      }
      if (f10 || f11) {
        gh = gl_fold2(r, g10, g11);
        gst2(G, b + half, gh);
      }
      if (f00 || f01 || f10 || f11) acc[1] = gl_add(acc[1], gl_dot2(gl_at2(wl, wh), gl_at2(gl, gh)));
    }
  } else {
    const uint64_t* src[5];
    uint64_t* dst[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      src[k] = P<const uint64_t*>(st, 4 + k);
      dst[k] = P<uint64_t*>(st, 4 + k);
    }
    for (uint64_t b = (uint64_t)(blockIdx.x - nb) * kBlock + threadIdx.x; b < st.q[1];
         b += (uint64_t)(gridDim.x - nb) * kBlock)
      gl_pair<5>(src, dst, true, r, b, st.q[1], acc[0], acc[1]);
  }
  gl_finish_round(acc, P<GlState*>(st, 9), P<uint64_t*>(st, 10), P<uint64_t*>(st, 11), P<uint64_t*>(st, 12));
}

// ST_GL_S_P2_RAW: Ma, Mb, Aa, Ab for y < q0 (see ST_GL_P2T). p0 yrow, p1 yent,
// p2 aU, p3 bV, p4 EL, p5 Ma, p6 Mb, p7 Aa, p8 Ab.
__global__ void __launch_bounds__(kBlock) k_gl_s_p2_raw(Step st) {
  const uint32_t* __restrict__ yrow = P<const uint32_t*>(st, 0);
  const uint2* __restrict__ yent = P<const uint2*>(st, 1);
  const uint64_t *aU = P<const uint64_t*>(st, 2), *bV = P<const uint64_t*>(st, 3), *EL = P<const uint64_t*>(st, 4);
  for (uint64_t y = GTID; y < st.q[0]; y += GSTRIDE) {
    uint64_t mu = 0, mv = 0, au = 0, av = 0;
    const uint32_t k1 = yrow[y + 1];
    for (uint32_t k = yrow[y]; k < k1; ++k) {
      const uint2 e = yent[k];
      const uint64_t l = gld(EL, e.y & 0x7fffffffu), tu = gl_mul(gld(aU, e.x), l), tv = gl_mul(gld(bV, e.x), l);
      if (e.y >> 31) {
        mu = gl_add(mu, tu);
        mv = gl_add(mv, tv);
      } else {
        au = gl_add(au, tu);
        av = gl_add(av, tv);
      }
    }
    gst(P<uint64_t*>(st, 5), y, mu);
    gst(P<uint64_t*>(st, 6), y, mv);
    gst(P<uint64_t*>(st, 7), y, au);
    gst(P<uint64_t*>(st, 8), y, av);
  }
}

// ST_GL_S_P2_FINAL: Fa, Fb, Ka (holding Aa), Kb (Ab), Ks for y < q0. p0 Fa, p1 Fb,
// p2 Ka, p3 Kb, p4 Ks, p5 S, p6 Ma, p7 Mb.
__global__ void __launch_bounds__(kBlock) k_gl_s_p2_final(Step st) {
  const GlState* S = P<const GlState*>(st, 5);
  const uint64_t vx = S->vx, su = S->su, sv = S->sv;
  for (uint64_t y = GTID; y < st.q[0]; y += GSTRIDE) {
    const uint64_t au = gld(P<const uint64_t*>(st, 2), y), av = gld(P<const uint64_t*>(st, 3), y);
    const uint64_t ka = gl_mul(vx, au), kb = gl_mul(vx, av);
    gst(P<uint64_t*>(st, 0), y, gl_add(gl_mul(vx, gld(P<const uint64_t*>(st, 6), y)), au));
    gst(P<uint64_t*>(st, 1), y, gl_add(gl_mul(vx, gld(P<const uint64_t*>(st, 7), y)), av));
    gst(P<uint64_t*>(st, 2), y, ka);
    gst(P<uint64_t*>(st, 3), y, kb);
    gst(P<uint64_t*>(st, 4), y, gl_add(gl_mul(su, ka), gl_mul(sv, kb)));
  }
}

// ST_GL_S_LOCAL2: as ST_GL_LOCAL_CONTRACT with two weight vectors p1, p3 into
// p2, p4; two adjacent columns per thread (n >= 1).
__global__ void __launch_bounds__(kBlock) k_gl_s_local2(Step st) {
  const uint64_t *W = P<const uint64_t*>(st, 0), *A = P<const uint64_t*>(st, 1), *B = P<const uint64_t*>(st, 3);
  const uint32_t n = st.u[0], lr = st.u[1];
  const uint64_t mask = (1ull << n) - 1;
  for (uint64_t g = 2 * GTID; g < st.q[0]; g += 2 * GSTRIDE) {
    const uint64_t ch = g >> n, c = g & mask;
    const uint64_t y0 = ch << lr, y1 = y0 + (1ull << lr);
    GlAcc ax, ay, bx, by;
    for (uint64_t y = y0; y < y1; ++y) {
      const U64x2 w = gld2(W, (y << n) | c);
      const uint64_t ea = gld(A, y), eb = gld(B, y);
      gl_mac(ax, ea, w.x);
      gl_mac(ay, ea, w.y);
      gl_mac(bx, eb, w.x);
      gl_mac(by, eb, w.y);
    }
    gst2(P<uint64_t*>(st, 2), g, U64x2{gl_acc_value(ax), gl_acc_value(ay)});
    gst2(P<uint64_t*>(st, 4), g, U64x2{gl_acc_value(bx), gl_acc_value(by)});
  }
}

// ST_GL_S_HANDOFF: the copy tables of phase 1 for c < q0. p0, p1 the chunk partials
// of A and B (u0 chunks, chunk ch's columns from ch q0), p2 Cu, p3 Cv, p4 sa, p5 sb
// (two entries left), p6 W src, p7 G, p8 act, p9 rprev, p10 Wc, p11 Gc, p12 Hc.
// 16 lanes per column add its chunks.
__global__ void __launch_bounds__(kBlock) k_gl_s_handoff(Step st) {
  const uint64_t r = *P<const uint64_t*>(st, 9);
  const uint64_t *Ws = P<const uint64_t*>(st, 6), *G = P<const uint64_t*>(st, 7);
  const uint32_t* act = P<const uint32_t*>(st, 8);
  const uint64_t sa0 = gld(P<const uint64_t*>(st, 4), 0), sa1 = gld(P<const uint64_t*>(st, 4), 1);
  const uint64_t sb0 = gld(P<const uint64_t*>(st, 5), 0), sb1 = gld(P<const uint64_t*>(st, 5), 1);
  const uint64_t sa = gl_add(sa0, gl_mul(r, gl_sub(sa1, sa0))), sb = gl_add(sb0, gl_mul(r, gl_sub(sb1, sb0)));
  const uint64_t ncop = st.q[0];
  const uint32_t lane = threadIdx.x & 15;
  for (uint64_t base = (uint64_t)blockIdx.x * (kBlock / 16); base < ncop; base += (uint64_t)gridDim.x * (kBlock / 16)) {
    const uint64_t c = base + threadIdx.x / 16;
    uint64_t a = 0, b = 0;
    if (c < ncop)
      for (uint32_t ch = lane; ch < st.u[0]; ch += 16) {
        a = gl_add(a, gld(P<const uint64_t*>(st, 0), ch * ncop + c));
        b = gl_add(b, gld(P<const uint64_t*>(st, 1), ch * ncop + c));
      }
    for (int off = 8; off >= 1; off >>= 1) {
      a = gl_add(a, shfl_xor_u64(a, off));
      b = gl_add(b, shfl_xor_u64(b, off));
    }
    if (lane == 0 && c < ncop) {
      const uint64_t cu = gld(P<const uint64_t*>(st, 2), c), cv = gld(P<const uint64_t*>(st, 3), c);
      const uint64_t w0 = gld(Ws, c), w1 = gld(Ws, c + ncop);
      const uint64_t g0 = gl_row_active(act, 1, 0) ? gld(G, c) : 0, g1 = gl_row_active(act, 1, 1) ? gld(G, c + ncop) : 0;
      gst(P<uint64_t*>(st, 10), c, gl_add(w0, gl_mul(r, gl_sub(w1, w0))));
      gst(P<uint64_t*>(st, 11), c, gl_add(gl_add(gl_mul(cu, sa), gl_mul(cv, sb)), gl_add(g0, gl_mul(r, gl_sub(g1, g0)))));
      gst(P<uint64_t*>(st, 12), c, gl_add(gl_mul(cu, a), gl_mul(cv, b)));
    }
  }
}

// ---------------------------------------------------------------- tails

// ST_GL_TAIL / ST_GL_TAIL5: the remaining u0 rounds in one workgroup, then
// the final fold; the final value of table 0 goes to *final_out and, when
// proof_value is not null, to the proof and into the transcript. q0 = table
// size before the pending fold (if any). p0..p(NT-1) src, pNT..p(2NT-1) dst,
// then (from B = 2 NT) pB rpending, pB+1 S, pB+2 r_out, pB+3 msg,
// pB+4 final_out, pB+5 proof_value.
constexpr int kGlTailThreads = 1024;

// Levels of at most 2^kGlTailLdsLog(NT) entries live in shared memory (48 and 40 KiB),
// larger ones stay in their tables.
__host__ __device__ constexpr uint32_t gl_tail_lds_log(int nt) { return nt == 3 ? 11 : 10; }

template <int NT>
__global__ void __launch_bounds__(kGlTailThreads) k_gl_tail(Step st) {
  constexpr int B = 2 * NT;
  const uint64_t* src[NT];
  uint64_t* dst[NT];
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    src[k] = P<const uint64_t*>(st, k);
    dst[k] = P<uint64_t*>(st, NT + k);
  }
  const uint64_t* rpending = P<const uint64_t*>(st, B);
  GlState* S = P<GlState*>(st, B + 1);
  uint64_t* r_out = P<uint64_t*>(st, B + 2);
  uint64_t* msg = P<uint64_t*>(st, B + 3);
  // The folded tables stay in shared memory once they fit, packed (a level of m
  // entries takes NT m words, table k from k m). A pair's entries are folded and
  // evaluated by one thread, so a round is one pass, one sum and the hash: 5 us
  // at 2^12 entries, where a grid-wide round costs 12.
  extern __shared__ uint64_t lvl[];
  constexpr uint32_t kLds = 1u << gl_tail_lds_log(NT);
  __shared__ uint64_t r_sh[2], e_sh[2][2], red[2][kGlTailThreads / 64];
  __shared__ ShaHelper help;
  const uint32_t wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint32_t rounds = st.u[0];
  const bool pending = rpending != nullptr;
  uint64_t size = st.q[0];
  ShaLanes sh;
  uint64_t claim = 0;
  if (wid == 0) {
    sh = sha_lanes_load(S->st);
    sha_init(sha_buf());
  }
  if (wid == 1) claim = S->claim;
  if (threadIdx.x == 0) {
    r_sh[1] = pending ? *rpending : 0;
    help.ready = 0;
  }
  __syncthreads();
  bool in_lds = false;  // whether the current level is in lvl
  for (uint32_t j = 0; j < rounds; ++j) {
    const bool fold = pending || j > 0;
    const uint64_t r = r_sh[(j + 1) & 1];
    if (fold) size /= 2;
    const uint32_t half = (uint32_t)(size / 2);
    const uint32_t old = (uint32_t)(fold ? 2 * size : size);  // entries of the level read
    uint64_t acc[2] = {0, 0};
    uint64_t lo[NT], hi[NT];
    const bool to_lds = size <= kLds;
    // a level that lives in shared memory is read whole before any of it is
    // overwritten (it has at most one pair per thread); a level in its tables
    // is overwritten entry by entry by the thread that read it
    for (uint32_t b0 = 0; b0 < half; b0 += kGlTailThreads) {
      const uint32_t b = b0 + threadIdx.x;
      const bool act = b < half;
      if (act) {
#pragma unroll
        for (int k = 0; k < NT; ++k) {
          auto at = [&](uint32_t i) { return in_lds ? lvl[k * old + i] : gld(src[k], i); };
          if (fold) {
            const uint32_t m = 2 * half;
            const uint64_t a0 = at(b), a1 = at(b + m), c0 = at(b + half), c1 = at(b + half + m);
            lo[k] = gl_add(a0, gl_mul(r, gl_sub(a1, a0)));
            hi[k] = gl_add(c0, gl_mul(r, gl_sub(c1, c0)));
          } else {
            lo[k] = at(b);
            hi[k] = at(b + half);
          }
        }
      }
      if (in_lds) __syncthreads();
      if (act) {
#pragma unroll
        for (int k = 0; k < NT; ++k) {
          if (to_lds) {
            lvl[k * (uint32_t)size + b] = lo[k];
            lvl[k * (uint32_t)size + b + half] = hi[k];
          } else if (fold) {
            gst(dst[k], b, lo[k]);
            gst(dst[k], b + half, hi[k]);
          }
        }
        acc[0] = gl_add(acc[0], gl_form<NT>(lo));
        uint64_t t2[NT];
#pragma unroll
        for (int k = 0; k < NT; ++k) t2[k] = gl_sub(gl_double(hi[k]), lo[k]);
        acc[1] = gl_add(acc[1], gl_form<NT>(t2));
      }
    }
    in_lds = to_lds;
    if (!to_lds && fold)
#pragma unroll
      for (int k = 0; k < NT; ++k) src[k] = dst[k];
    const uint32_t nw = half >= kGlTailThreads ? kGlTailThreads / 64 : (half + 63) / 64;  // waves with pairs
    if (wid < nw) {
      acc[0] = gl_wave_sum63(acc[0]);
      acc[1] = gl_wave_sum63(acc[1]);
      if (lane == 63) {
        red[0][wid] = acc[0];
        red[1][wid] = acc[1];
      }
    }
    __syncthreads();
    if (wid < 3) {
      uint64_t e0 = red[0][0], e2 = red[1][0];
      for (uint32_t w = 1; w < nw; ++w) {
        e0 = gl_add(e0, red[0][w]);
        e2 = gl_add(e2, red[1][w]);
      }
      if (wid == 0) {
        sh = sha_compress_wave<true>(sh, gl_round_word(e0, e2), sha_buf(), &help, 3 * j);
        const uint64_t rr = gl_accept_wave(sh);
        if (lane == 0) {
          r_sh[j & 1] = rr;
          r_out[j] = rr;
        }
      } else if (wid == 2) {
        sha_help(gl_round_word(e0, e2), sha_buf(), &help, 3 * j);
      } else {
        // wave 1: the claim through the previous round, then this round's message
        if (j > 0) {
          const uint32_t q = (j - 1) & 1;
          claim = gl_interp3(e_sh[q][0], gl_sub(claim, e_sh[q][0]), e_sh[q][1], r_sh[q]);
        }
        if (lane == 0) {
          e_sh[j & 1][0] = e0;
          e_sh[j & 1][1] = e2;
          msg[3 * j] = e0;
          msg[3 * j + 1] = gl_sub(claim, e0);
          msg[3 * j + 2] = e2;
        }
      }
    }
    __syncthreads();
  }
  // the last fold, every table's final entry to its first place (the copy
  // tables read them there), and the last claim move
  if (wid == 0) {
    const bool fold = pending || rounds > 0;
    const uint64_t r = r_sh[(rounds + 1) & 1];
    uint64_t v = 0;
#pragma unroll
    for (int k = NT - 1; k >= 0; --k) {
      if (fold) {
        const uint64_t a0 = in_lds ? lvl[2 * k] : gld(src[k], 0), a1 = in_lds ? lvl[2 * k + 1] : gld(src[k], 1);
        v = gl_add(a0, gl_mul(r, gl_sub(a1, a0)));
        if (lane == 0) gst(dst[k], 0, v);
      } else {
        v = gld(src[k], 0);
      }
    }
    uint64_t* proof_value = P<uint64_t*>(st, B + 5);
    if (lane == 0) *P<uint64_t*>(st, B + 4) = v;
    if (proof_value) {
      if (lane == 0) *proof_value = v;
      sha_lanes_store(sha_buf()->msg, sh);
      if (lane < 3)
        sha_buf()->msg[8 + lane] = lane == 0 ? kTagValue : bswap32((uint32_t)(lane == 1 ? v : v >> 32));
      sh = sha_message_wave<11>(sha_buf());
    }
    sha_lanes_store(S->st, sh);
  } else if (wid == 1 && rounds > 0) {
    const uint32_t q = (rounds - 1) & 1;
    claim = gl_interp3(e_sh[q][0], gl_sub(claim, e_sh[q][0]), e_sh[q][1], r_sh[q]);
    if (lane == 0) S->claim = claim;
  }
}

#undef GTID
#undef GSTRIDE

static size_t gl_tail_lds(const Step& st, int nt) {
  const uint64_t eval = st.p[2 * nt] ? st.q[0] / 2 : st.q[0];  // p[2 NT]: the pending challenge
  return 8 * nt * std::min<uint64_t>(eval, 1ull << gl_tail_lds_log(nt));
}

// Largest table (log2 of its entries) a tail evaluates: three steps above the
// tuned limit of the BN254 tails, whose products cost ten times as much, at most
// 2^12 (c2 shape: 6595 us per proof at 2^10, 6545 at 2^11, 6510 at 2^12, 6768 at
// 2^13 for three tables).
static uint32_t gl_tail_log(const Tuning& tun) { return std::min<uint32_t>(tun.tail_log + 3, 12); }

// Two independent steps in one launch (Step::join), as in the BN254 prover.
__global__ void __launch_bounds__(kBlock) k_gl_p2_pair(Step a, Step b) {
  if (blockIdx.x < a.ntiles) body_gl_p2t(a, blockIdx.x, a.ntiles);
  else body_gl_copy_contract(b, blockIdx.x - a.ntiles, b.ntiles);
}
__global__ void __launch_bounds__(kBlock) k_gl_local_pair(Step a, Step b) {
  if (blockIdx.x < a.ntiles) body_gl_local_values(a, blockIdx.x, a.ntiles);
  else body_gl_local_contract(b, blockIdx.x - a.ntiles, b.ntiles);
}

bool launch_gl_pair(const Step& st, const Step& next, hipStream_t s) {
  const bool p2 = st.type == ST_GL_P2T && next.type == ST_GL_COPY_CONTRACT;
  if (!p2 && !(st.type == ST_GL_LOCAL_VALUES && next.type == ST_GL_LOCAL_CONTRACT)) return false;
  const int tok = prof_begin(s);
  const dim3 grid(st.ntiles + next.ntiles), block(kBlock);
  if (p2) k_gl_p2_pair<<<grid, block, 0, s>>>(st, next);
  else k_gl_local_pair<<<grid, block, 0, s>>>(st, next);
  if (tok >= 0)
    prof_end(tok, s, p2 ? PC_COPY_CONTRACT : PC_LOCAL_CONTRACT, st.bytes + next.bytes, st.mulmods + next.mulmods);
  return true;
}

void launch_gl_step(const Step& st, hipStream_t s) {
  const int tok = prof_begin(s);
  const dim3 grid(st.ntiles), block(kBlock);
  ProfClass cls = PC_SMALL;
  switch (st.type) {
    case ST_GL_FORWARD: k_gl_forward<<<grid, block, 0, s>>>(st); cls = PC_FORWARD; break;
    case ST_GL_DIGEST: k_gl_digest<<<grid, block, 0, s>>>(st); cls = PC_DIGEST; break;
    case ST_GL_BEGIN: k_gl_begin<<<grid, block, 0, s>>>(st); cls = PC_TRANSCRIPT; break;
    case ST_GL_SQUEEZE: k_gl_squeeze<<<grid, block, 0, s>>>(st); cls = PC_TRANSCRIPT; break;
    case ST_GL_LAYER_BEGIN: k_gl_layer_begin<<<grid, block, 0, s>>>(st); cls = PC_TRANSCRIPT; break;
    case ST_GL_EQ: k_gl_eq<<<grid, block, 0, s>>>(st); cls = PC_EQ; break;
    case ST_GL_WSUM: k_gl_wsum<<<grid, block, 0, s>>>(st); cls = PC_CLAIM; break;
    case ST_GL_P1: k_gl_p1<<<grid, block, 0, s>>>(st); cls = PC_PHASE1_INIT; break;
    case ST_GL_ROUND: k_gl_round<3><<<grid, block, 0, s>>>(st); cls = PC_ROUND_A; break;
    case ST_GL_TAIL: k_gl_tail<3><<<grid, dim3(kGlTailThreads), gl_tail_lds(st, 3), s>>>(st); cls = PC_TAIL_A; break;
    case ST_GL_ROUND5: k_gl_round<5><<<grid, block, 0, s>>>(st); cls = PC_ROUND_B; break;
    case ST_GL_TAIL5: k_gl_tail<5><<<grid, dim3(kGlTailThreads), gl_tail_lds(st, 5), s>>>(st); cls = PC_TAIL_B; break;
    case ST_GL_COPY_WEIGHTS: k_gl_copy_weights<<<grid, block, 0, s>>>(st); cls = PC_SMALL; break;
    case ST_GL_P2T: k_gl_p2t<<<grid, block, 0, s>>>(st); cls = PC_PHASE2_TABLES; break;
    case ST_GL_COPY_CONTRACT: k_gl_copy_contract<<<grid, block, 0, s>>>(st); cls = PC_COPY_CONTRACT; break;
    case ST_GL_LOCAL_VALUES: k_gl_local_values<<<grid, block, 0, s>>>(st); cls = PC_SMALL; break;
    case ST_GL_LOCAL_CONTRACT: k_gl_local_contract<<<grid, block, 0, s>>>(st); cls = PC_LOCAL_CONTRACT; break;
    case ST_GL_COPY_TABLES: k_gl_copy_tables<<<grid, block, 0, s>>>(st); cls = PC_SMALL; break;
    case ST_GL_S_SMALL: k_gl_s_small<<<grid, block, 0, s>>>(st); break;
    case ST_GL_S_INIT_ROUND: k_gl_s_init_round<<<grid, block, 0, s>>>(st); cls = PC_PHASE1_SPLIT; break;
    case ST_GL_S_ROUND: k_gl_s_round<<<grid, block, 0, s>>>(st); cls = PC_ROUND_SPLIT; break;
    case ST_GL_S_P2_RAW: k_gl_s_p2_raw<<<grid, block, 0, s>>>(st); cls = PC_PHASE2_TABLES; break;
    case ST_GL_S_P2_FINAL: k_gl_s_p2_final<<<grid, block, 0, s>>>(st); cls = PC_PHASE2_TABLES; break;
    case ST_GL_S_LOCAL2: k_gl_s_local2<<<grid, block, 0, s>>>(st); cls = PC_LOCAL_CONTRACT; break;
    case ST_GL_S_HANDOFF: k_gl_s_handoff<<<grid, block, 0, s>>>(st); break;
    default: break;
  }
  if (tok >= 0) prof_end(tok, s, cls, st.bytes, st.mulmods);
}

// ---------------------------------------------------------------- proof program (host)

namespace {

constexpr uint32_t kGlSweepTiles = 65535u * 8;
constexpr double kGE = 8.0;  // bytes per element

uint32_t gl_tiles(uint64_t n, uint32_t cap) {
  uint64_t g = (n + kBlock - 1) / kBlock;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (uint32_t)g;
}

Step gl_mk(uint32_t type, uint32_t ntiles) {
  Step st;
  memset(&st, 0, sizeof(st));
  st.type = type;
  st.ntiles = ntiles < 1 ? 1 : ntiles;
  return st;
}

size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }

struct GlWs {
  uint64_t* layer[GKR_MAX_DEPTH + 1];
  uint64_t *G, *H, *Wf, *aU, *bV, *Cu, *Cv, *EL, *EC, *partials, *chal;
  uint64_t *U, *V, *P, *Q, *Fa, *Fb, *Ka, *Kb, *Ks, *EqR, *Wc, *Fc, *Kc, *wpart;
  uint32_t *dig_a, *dig_b, *dig_in, *dig_out;
  GlState* S;
};

GlWs gl_bind(const gkr_circuit& c, void* base, const uint64_t* d_inputs, uint64_t* d_outputs) {
  const GlPlan& p = c.gl;
  char* b = static_cast<char*>(base);
  GlWs w;
  memset(&w, 0, sizeof(w));
  auto U = [&](size_t o) { return reinterpret_cast<uint64_t*>(b + o); };
  for (uint32_t i = 1; i < c.depth; ++i) w.layer[i] = U(p.off_layer[i]);
  w.layer[0] = d_outputs;
  w.layer[c.depth] = const_cast<uint64_t*>(d_inputs);
  w.G = U(p.off_G); w.H = U(p.off_H); w.Wf = U(p.off_Wf);
  w.aU = U(p.off_aU); w.bV = U(p.off_bV); w.Cu = U(p.off_Cu); w.Cv = U(p.off_Cv);
  w.EL = U(p.off_EL); w.EC = U(p.off_EC);
  w.U = U(p.off_U); w.V = U(p.off_V); w.P = U(p.off_P); w.Q = U(p.off_Q); w.Fa = U(p.off_Fa); w.Fb = U(p.off_Fb);
  w.Ka = U(p.off_Ka); w.Kb = U(p.off_Kb); w.Ks = U(p.off_Ks); w.EqR = U(p.off_EqR); w.Wc = U(p.off_Wc);
  w.Fc = U(p.off_Fc); w.Kc = U(p.off_Kc); w.wpart = U(p.off_wpart);
  w.partials = U(p.off_partials);
  w.chal = U(p.off_chal);
  w.dig_a = reinterpret_cast<uint32_t*>(b + p.off_dig_a);
  w.dig_b = reinterpret_cast<uint32_t*>(b + p.off_dig_b);
  w.dig_in = reinterpret_cast<uint32_t*>(b + p.off_dig_in);
  w.dig_out = reinterpret_cast<uint32_t*>(b + p.off_dig_out);
  w.S = reinterpret_cast<GlState*>(b + p.off_state);
  return w;
}

void gl_eq(std::vector<Step>& steps, int count, const uint32_t* bits, const uint64_t* const* pts,
           const uint64_t* const* scl, uint64_t* const* outs) {
  Step st = gl_mk(ST_GL_EQ, 1);
  uint64_t total = 0;
  for (int j = 0; j < count; ++j) {
    st.u[j] = bits[j]; st.p[j] = pts[j]; st.p[4 + j] = scl[j]; st.p[8 + j] = outs[j];
    total += 1ull << bits[j];
  }
  st.u[4] = count;
  st.ntiles = gl_tiles(total, 1u << 30);
  st.bytes = kGE * total;
  steps.push_back(st);
}

// One phase: grid-wide rounds while the table exceeds 2^tail_log, then the tail.
// The rounds of one phase over NT tables (3: W X + Y; 5: A B + C D + E):
// grid-wide rounds while the evaluated table exceeds the tail size, then one
// workgroup.
template <int NT>
void gl_phase(std::vector<Step>& steps, const uint64_t* const* src0, uint64_t* const* dst, uint32_t nrounds,
              GlState* S, uint64_t* partials, uint64_t* r_out, uint64_t* msg, uint64_t* final_out,
              uint64_t* proof_value, const Tuning& tun) {
  constexpr int B = 2 * NT;
  const uint64_t* src[NT];
  for (int k = 0; k < NT; ++k) src[k] = src0[k];
  uint64_t eval = 1ull << nrounds;
  uint32_t j = 0;
  const uint64_t* pending = nullptr;
  while (j < nrounds && eval > (1ull << gl_tail_log(tun))) {
    const uint64_t half = eval / 2;
    Step st = gl_mk(NT == 3 ? ST_GL_ROUND : ST_GL_ROUND5, gl_tiles((half + 1) / 2, tun.max_round_blocks));
    for (int k = 0; k < NT; ++k) {
      st.p[k] = src[k];
      st.p[NT + k] = dst[k];
    }
    st.p[B] = pending; st.p[B + 1] = S; st.p[B + 2] = partials; st.p[B + 3] = r_out + j; st.p[B + 4] = msg + 3 * j;
    st.q[0] = half;
    st.bytes = kGE * NT * (pending ? 6.0 : 2.0) * half;
    st.mulmods = (pending ? 2.0 * NT : 0.0) * half + (NT == 3 ? 4.0 : 6.0) * half;
    steps.push_back(st);
    if (pending)
      for (int k = 0; k < NT; ++k) src[k] = dst[k];
    pending = r_out + j;
    ++j;
    eval /= 2;
  }
  Step st = gl_mk(NT == 3 ? ST_GL_TAIL : ST_GL_TAIL5, 1);
  for (int k = 0; k < NT; ++k) {
    st.p[k] = src[k];
    st.p[NT + k] = dst[k];
  }
  st.p[B] = pending; st.p[B + 1] = S; st.p[B + 2] = r_out + j; st.p[B + 3] = msg + 3 * j; st.p[B + 4] = final_out;
  st.p[B + 5] = proof_value;
  st.q[0] = pending ? 2 * eval : eval;
  st.u[0] = nrounds - j;
  st.bytes = kGE * 3.0 * NT * eval;
  steps.push_back(st);
}

// Row chunks of the local contraction: about 2^18 threads in all.
uint32_t gl_ychunks(uint32_t sigma, uint32_t n) {
  const uint64_t want = (n >= 18) ? 1 : (1ull << (18 - n));
  return (uint32_t)std::min<uint64_t>(want, 1ull << sigma);
}

void gl_copy_contract(std::vector<Step>& steps, const uint64_t* W, const uint64_t* U, const uint64_t* V, uint64_t* Pt,
                      uint64_t* Qt, uint32_t n, uint64_t rows) {
  Step st = gl_mk(ST_GL_COPY_CONTRACT, gl_tiles(rows * 64, kGlSweepTiles));
  st.p[0] = W; st.p[1] = U; st.p[2] = V; st.p[3] = Pt; st.p[4] = Qt; st.u[0] = n;
  st.q[0] = rows;
  st.bytes = kGE * (double)(rows << n); st.mulmods = 2.0 * (double)(rows << n);
  steps.push_back(st);
}

// Layers whose phase 1 takes the contracted form. Four layers with it and without
// (half of the gates MUL), us: 2^22 entries 2,605 / 2,456, 2^23 2,979 / 3,084 (with
// 2^8 copies 3,478 / 3,406), 2^24 3,893 / 4,478; all gates MUL 2^23 3,047 / 3,081.
constexpr uint32_t kGlSplitMinLogCopies = 9, kGlSplitMinLogRows = 8, kGlSplitMinLogWidth = 23;

bool gl_split_applies(uint32_t n, uint32_t sigma) {
  return n >= kGlSplitMinLogCopies && sigma >= kGlSplitMinLogRows && n + sigma >= kGlSplitMinLogWidth;
}

// Phase 1 of layer i in the contracted form; leaves EL in w.EL and Ma, Mb, Aa, Ab in
// w.P, w.Q, w.Ka, w.Kb. H, which this form does not use, holds the chunk
// partials of A and B.
void gl_emit_phase1_split(std::vector<Step>& steps, const gkr_circuit& c, uint32_t i, const GlWs& w, uint64_t* rx,
                          uint64_t* msg, const Tuning& tun) {
  const uint32_t n = c.n, sigma = c.sigma[i + 1], s1 = sigma + n;
  const LayerWiring& lw = c.wiring[i];
  const uint64_t rows = 1ull << sigma, ncop = 1ull << n, full = rows << n;
  const double gates = (double)(1ull << c.sigma[i]), muls = (double)c.mul_gates[i];
  const uint64_t* W = w.layer[i + 1];
  gl_copy_contract(steps, W, w.Cu, w.Cv, w.P, w.Q, n, rows);
  uint64_t* small[5] = {w.P, w.Fa, w.Q, w.Fb, w.Ks};
  {
    Step st = gl_mk(ST_GL_S_SMALL, gl_tiles(rows, kGlSweepTiles));
    st.p[0] = lw.xrow; st.p[1] = lw.xmid; st.p[2] = lw.xent; st.p[3] = w.aU; st.p[4] = w.bV; st.p[5] = w.P;
    st.p[6] = w.Q; st.p[7] = w.Fa; st.p[8] = w.Fb; st.p[9] = w.Ks; st.q[0] = rows;
    st.bytes = kGE * (3.0 * rows + 4.0 * (gates - muls)); st.mulmods = 2.0 * (gates - muls);
    steps.push_back(st);
  }
  const uint64_t* Ws = W;
  for (uint32_t j = 0; j < sigma; ++j) {
    const uint64_t half = full >> (j + 1), shalf = rows >> (j + 1);
    Step st = gl_mk(j == 0 ? ST_GL_S_INIT_ROUND : ST_GL_S_ROUND, gl_tiles((half + 1) / 2, j == 0 ? 2048 : 1024));
    st.u[0] = n; st.u[1] = st.ntiles; st.u[2] = sigma - j;
    st.ntiles += (uint32_t)std::min<uint64_t>((shalf + kBlock - 1) / kBlock, 64);
    st.q[0] = half; st.q[1] = shalf;
    st.p[9] = w.S; st.p[10] = w.partials; st.p[11] = rx + j; st.p[12] = msg + 3 * j;
    if (j == 0) {
      st.p[0] = W; st.p[1] = w.G; st.p[2] = lw.xrow; st.p[3] = lw.xmid; st.p[4] = lw.xent; st.p[5] = w.aU;
      st.p[6] = w.bV; st.p[7] = w.Cu; st.p[8] = w.Cv; st.p[13] = small[0];
      for (int k = 0; k < 5; ++k) st.w[k] = (uint32_t)(small[k] - small[0]);
      const double a0 = split_active_share(muls, rows, 0), a1 = split_active_share(muls, rows, 1);
      st.bytes = kGE * (muls * ncop + a0 * full + a1 * full);
      st.mulmods = 3.0 * muls * ncop + (a0 + a1) * half;
    } else {
      st.p[0] = Ws; st.p[1] = w.Wf; st.p[2] = w.G; st.p[3] = lw.act; st.p[13] = rx + j - 1;
      for (int k = 0; k < 5; ++k) st.p[4 + k] = small[k];
      Ws = w.Wf;
      const double a0 = split_active_share(muls, rows, j - 1), a1 = split_active_share(muls, rows, j);
      const double a2 = split_active_share(muls, rows, j + 1);
      st.bytes = kGE * half * (6.0 + 4.0 * a0 + 2.0 * a1); st.mulmods = half * (2.0 + 3.0 * a1 + a2);
    }
    steps.push_back(st);
  }
  {
    const uint32_t bits[1] = {sigma};
    const uint64_t* pts[1] = {rx};
    const uint64_t* scl[1] = {nullptr};
    uint64_t* outs[1] = {w.EL};
    gl_eq(steps, 1, bits, pts, scl, outs);
  }
  {
    Step st = gl_mk(ST_GL_S_P2_RAW, gl_tiles(rows, kGlSweepTiles));
    st.p[0] = lw.yrow; st.p[1] = lw.yent; st.p[2] = w.aU; st.p[3] = w.bV; st.p[4] = w.EL; st.p[5] = w.P; st.p[6] = w.Q;
    st.p[7] = w.Ka; st.p[8] = w.Kb; st.q[0] = rows;
    st.bytes = kGE * (3.0 * gates + 4.0 * rows); st.mulmods = 2.0 * gates;
    steps.push_back(st);
  }
  const uint32_t R = gl_ychunks(sigma, n);
  uint64_t *partA = w.H, *partB = w.H + (uint64_t)R * ncop;
  {
    uint32_t lr = 0;
    while ((1ull << (lr + 1)) * R <= rows) ++lr;
    Step st = gl_mk(ST_GL_S_LOCAL2, gl_tiles((uint64_t)R * ncop / 2, kGlSweepTiles));
    st.p[0] = W; st.p[1] = w.Ka; st.p[2] = partA; st.p[3] = w.Kb; st.p[4] = partB; st.u[0] = n; st.u[1] = lr;
    st.q[0] = (uint64_t)R * ncop;
    st.bytes = kGE * (double)(full + 2 * (uint64_t)R * ncop); st.mulmods = 2.0 * full;
    steps.push_back(st);
  }
  {
    Step st = gl_mk(ST_GL_S_HANDOFF, gl_tiles(16 * ncop, kGlSweepTiles));
    st.p[0] = partA; st.p[1] = partB; st.p[2] = w.Cu; st.p[3] = w.Cv; st.p[4] = w.Fa; st.p[5] = w.Fb; st.p[6] = Ws;
    st.p[7] = w.G; st.p[8] = lw.act; st.p[9] = rx + sigma - 1; st.p[10] = w.Wc; st.p[11] = w.Fc; st.p[12] = w.Kc;
    st.u[0] = R; st.q[0] = ncop;
    st.bytes = kGE * (double)((2 * R + 9) * ncop); st.mulmods = 6.0 * ncop;
    steps.push_back(st);
  }
  const uint64_t* src[3] = {w.Wc, w.Fc, w.Kc};
  uint64_t* dst[3] = {w.Wc, w.Fc, w.Kc};
  gl_phase<3>(steps, src, dst, n, w.S, w.partials, rx + sigma, msg + 3 * sigma, &w.S->vx, msg + 3 * s1, tun);
}

uint64_t gl_layer_proof_words(const gkr_circuit& c, uint32_t i) { return 6ull * c.s(i + 1) + 2; }

void gl_emit_proof(std::vector<Step>& steps, const gkr_circuit& c, const GlWs& w, uint64_t seed, uint64_t* proof,
                   const Tuning& tun) {
  const uint32_t d = c.depth, n = c.n;
  // forward evaluation: layer d is the caller's inputs, layer 0 the caller's outputs
  for (int i = (int)d - 1; i >= 0; --i) {
    Step st = gl_mk(ST_GL_FORWARD, gl_tiles(1ull << c.s(i), kGlSweepTiles));
    st.p[0] = w.layer[i + 1]; st.p[1] = w.layer[i]; st.p[2] = c.wiring[i].gates; st.u[0] = n;
    st.q[0] = 1ull << c.s(i);
    st.bytes = kGE * 3.0 * (1ull << c.s(i));
    st.mulmods = (double)(c.mul_gates[i] << n);
    steps.push_back(st);
  }
  // statement
  const DigestJob jobs[2] = {{reinterpret_cast<const uint32_t*>(w.layer[d]), 2ull << c.s(d), w.dig_in},
                             {reinterpret_cast<const uint32_t*>(w.layer[0]), 2ull << c.s(0), w.dig_out}};
  emit_digests(steps, ST_GL_DIGEST, jobs, 2, w.dig_a, w.dig_b, reinterpret_cast<uint32_t*>(w.partials),
               kGE * 2 * kMaxRoundBlocks / 32);
  {
    Step st = gl_mk(ST_GL_BEGIN, 1);
    st.p[0] = w.S; st.p[1] = w.dig_in; st.p[2] = w.dig_out;
    uint8_t msg[22];
    memcpy(msg, "SISU-GKR-GL-v1", 14);
    for (int k = 0; k < 8; ++k) msg[14 + k] = (uint8_t)(seed >> (8 * k));
    sha256_bytes(msg, sizeof(msg), st.w);
    memcpy(st.w + 8, c.digest, 32);
    steps.push_back(st);
  }
  // output point and claim
  uint64_t* g = w.chal;
  {
    Step st = gl_mk(ST_GL_SQUEEZE, 1);
    st.p[0] = w.S; st.p[1] = g; st.u[0] = c.s(0);
    steps.push_back(st);
    const uint32_t bits[2] = {c.sigma[0], n};
    const uint64_t* pts[2] = {g, g + c.sigma[0]};
    const uint64_t* scl[2] = {nullptr, nullptr};
    uint64_t* outs[2] = {w.aU, w.Cu};
    gl_eq(steps, 2, bits, pts, scl, outs);
    Step ws = gl_mk(ST_GL_WSUM, gl_tiles(1ull << c.s(0), tun.max_round_blocks));
    ws.p[0] = w.layer[0]; ws.p[1] = w.aU; ws.p[2] = w.Cu; ws.p[3] = w.partials; ws.p[4] = w.S;
    ws.p[5] = &w.S->scratch[0]; ws.u[0] = n; ws.q[0] = 1ull << c.s(0);
    ws.bytes = kGE * (1ull << c.s(0));
    steps.push_back(ws);
  }
  // layers
  uint64_t* chal = g + c.s(0);
  uint64_t* pr = proof;
  for (uint32_t i = 0; i < d; ++i) {
    const uint32_t sg = c.sigma[i], sg1 = c.sigma[i + 1], s1 = c.s(i + 1);
    const uint64_t* u = (i == 0) ? g : chal - 2 * c.s(i);
    const uint64_t* v = (i == 0) ? g : chal - c.s(i);
    uint64_t* rx = chal;
    uint64_t* ry = chal + s1;
    {
      Step st = gl_mk(ST_GL_LAYER_BEGIN, 1);
      st.p[0] = w.S; st.p[1] = (i == 0) ? &w.S->scratch[0] : &w.S->vx; st.p[2] = &w.S->vy; st.u[0] = i == 0;
      steps.push_back(st);
    }
    {
      const uint32_t bits[4] = {sg, sg, n, n};
      const uint64_t* pts[4] = {u, v, u + sg, v + sg};
      const uint64_t* scl[4] = {&w.S->alpha, &w.S->beta, nullptr, nullptr};
      uint64_t* outs[4] = {w.aU, w.bV, w.Cu, w.Cv};
      gl_eq(steps, 4, bits, pts, scl, outs);
    }
    const LayerWiring& lw = c.wiring[i];
    const uint64_t ncop = 1ull << n, rows = 1ull << sg1;
    const bool split = tun.matrix_cores && gl_split_applies(n, sg1);
    if (split) gl_emit_phase1_split(steps, c, i, w, rx, pr, tun);
    if (!split) {
      Step st = gl_mk(ST_GL_P1, gl_tiles(1ull << s1, kGlSweepTiles));
      st.p[0] = w.layer[i + 1]; st.p[1] = w.G; st.p[2] = w.H; st.p[3] = lw.xrow; st.p[4] = lw.xent;
      st.p[5] = w.aU; st.p[6] = w.bV; st.p[7] = w.Cu; st.p[8] = w.Cv; st.u[0] = n; st.q[0] = 1ull << s1;
      st.bytes = kGE * (double)((1ull << c.s(i)) + 2 * (1ull << s1));
      st.mulmods = 3.0 * (1ull << c.s(i));
      steps.push_back(st);
    }
    if (!split) {
      const uint64_t* src[3] = {w.layer[i + 1], w.G, w.H};
      uint64_t* dst[3] = {w.Wf, w.G, w.H};
      gl_phase<3>(steps, src, dst, s1, w.S, w.partials, rx, pr, &w.S->vx, pr + 3 * s1, tun);
    }
    {
      // (EL is there already after the contracted phase 1)
      const uint32_t bits[2] = {n, sg1};
      const uint64_t* pts[2] = {rx + sg1, rx};
      const uint64_t* scl[2] = {nullptr, nullptr};
      uint64_t* outs[2] = {w.EC, w.EL};
      gl_eq(steps, split ? 1 : 2, bits, pts, scl, outs);
    }
    // phase 2 with the copy factors contracted
    {
      Step st = gl_mk(ST_GL_COPY_WEIGHTS, 1);
      st.p[0] = w.EC; st.p[1] = w.Cu; st.p[2] = w.Cv; st.p[3] = w.U; st.p[4] = w.V; st.p[5] = w.S; st.q[0] = ncop;
      st.bytes = kGE * 5.0 * ncop; st.mulmods = 2.0 * ncop;
      steps.push_back(st);
    }
    if (split) {
      Step st = gl_mk(ST_GL_S_P2_FINAL, gl_tiles(rows, kGlSweepTiles));
      st.p[0] = w.Fa; st.p[1] = w.Fb; st.p[2] = w.Ka; st.p[3] = w.Kb; st.p[4] = w.Ks; st.p[5] = w.S; st.p[6] = w.P;
      st.p[7] = w.Q; st.q[0] = rows;
      st.bytes = kGE * 9.0 * rows; st.mulmods = 6.0 * rows;
      steps.push_back(st);
    } else {
      Step st = gl_mk(ST_GL_P2T, gl_tiles(rows, kGlSweepTiles));
      st.p[0] = lw.yrow; st.p[1] = lw.yent; st.p[2] = w.aU; st.p[3] = w.bV; st.p[4] = w.EL; st.p[5] = w.S;
      st.p[6] = w.Fa; st.p[7] = w.Fb; st.p[8] = w.Ka; st.p[9] = w.Kb; st.p[10] = w.Ks; st.q[0] = rows;
      st.bytes = kGE * 5.0 * rows; st.mulmods = 2.0 * (double)(1ull << sg) + 6.0 * rows;
      steps.push_back(st);
    }
    gl_copy_contract(steps, w.layer[i + 1], w.U, w.V, w.P, w.Q, n, rows);
    steps.back().join = split ? 0 : 1;  // independent of the phase-2 tables
    {
      const uint64_t* src[5] = {w.P, w.Fa, w.Q, w.Fb, w.Ks};
      uint64_t* dst[5] = {w.P, w.Fa, w.Q, w.Fb, w.Ks};
      gl_phase<5>(steps, src, dst, sg1, w.S, w.partials, ry, pr + 3 * s1 + 1, &w.S->scratch[1], nullptr, tun);
    }
    {
      const uint32_t bits[1] = {sg1};
      const uint64_t* pts[1] = {ry};
      const uint64_t* scl[1] = {nullptr};
      uint64_t* outs[1] = {w.EqR};
      gl_eq(steps, 1, bits, pts, scl, outs);
    }
    {
      Step st = gl_mk(ST_GL_LOCAL_VALUES, (uint32_t)std::min<uint64_t>(std::max<uint64_t>(1, rows / kGlLocalValueRows), 256));
      st.p[0] = w.EqR; st.p[1] = w.Ka; st.p[2] = w.Kb; st.p[3] = w.S; st.p[4] = w.partials; st.q[0] = rows;
      st.bytes = kGE * 3.0 * rows; st.mulmods = 2.0 * rows;
      steps.push_back(st);
    }
    const uint32_t R = gl_ychunks(sg1, n);
    {
      uint32_t lr = 0;
      while ((1ull << (lr + 1)) * R <= rows) ++lr;  // rows per chunk = rows / R
      Step st = gl_mk(ST_GL_LOCAL_CONTRACT, gl_tiles(n ? (uint64_t)R * ncop / 2 : R, kGlSweepTiles));
      st.p[0] = w.layer[i + 1]; st.p[1] = w.EqR; st.p[2] = w.wpart; st.u[0] = n; st.u[1] = lr;
      st.q[0] = (uint64_t)R * ncop;
      st.bytes = kGE * (double)(rows * ncop + (uint64_t)R * ncop); st.mulmods = (double)(rows * ncop);
      st.join = 1;  // independent of the local values
      steps.push_back(st);
    }
    {
      uint32_t tl = 0;
      while ((1u << (tl + 1)) <= R && tl < 6) ++tl;  // lanes per column, as in the kernel
      Step st = gl_mk(ST_GL_COPY_TABLES, gl_tiles(ncop << tl, kGlSweepTiles));
      st.p[0] = w.wpart; st.p[1] = w.U; st.p[2] = w.V; st.p[3] = w.Fa; st.p[4] = w.Fb; st.p[5] = w.S;
      st.p[6] = w.Wc; st.p[7] = w.Fc; st.p[8] = w.Kc; st.u[0] = R; st.q[0] = ncop;
      st.bytes = kGE * (double)((uint64_t)R * ncop + 5 * ncop); st.mulmods = 4.0 * ncop;
      steps.push_back(st);
    }
    {
      const uint64_t* src[3] = {w.Wc, w.Fc, w.Kc};
      uint64_t* dst[3] = {w.Wc, w.Fc, w.Kc};
      gl_phase<3>(steps, src, dst, n, w.S, w.partials, ry + sg1, pr + 3 * s1 + 1 + 3 * sg1, &w.S->vy,
                  pr + 6 * s1 + 1, tun);
    }
    pr += gl_layer_proof_words(c, i);
    chal += 2 * s1;
  }
}

}  // namespace

void plan_gl_workspace(gkr_circuit& c) {
  GlPlan& p = c.gl;
  memset(&p, 0, sizeof(p));
  const uint32_t d = c.depth, n = c.n;
  uint32_t sp = 0, sig = 0;
  size_t chal = c.s(0);
  for (uint32_t i = 0; i < d; ++i) {
    sp = std::max(sp, c.s(i + 1));
    chal += 2ull * c.s(i + 1);
  }
  for (uint32_t i = 0; i <= d; ++i) sig = std::max(sig, c.sigma[i]);
  const size_t E = 8;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes);
    return o;
  };
  for (uint32_t i = 1; i < d; ++i) p.off_layer[i] = take(E << c.s(i));
  p.off_G = take(E << sp);
  p.off_H = take(E << sp);
  p.off_Wf = take(E << (sp ? sp - 1 : 0));
  p.off_aU = take(E << sig);
  p.off_bV = take(E << sig);
  p.off_Cu = take(E << n);
  p.off_Cv = take(E << n);
  p.off_EL = take(E << sig);
  p.off_EC = take(E << n);
  p.off_partials = take(E * 2 * (size_t)kMaxRoundBlocks);
  p.off_U = take(E << n);
  p.off_V = take(E << n);
  p.off_P = take(E << sig);
  p.off_Q = take(E << sig);
  p.off_Fa = take(E << sig);
  p.off_Fb = take(E << sig);
  p.off_Ka = take(E << sig);
  p.off_Kb = take(E << sig);
  p.off_Ks = take(E << sig);
  p.off_EqR = take(E << sig);
  p.off_Wc = take(E << n);
  p.off_Fc = take(E << n);
  p.off_Kc = take(E << n);
  {
    uint64_t wp = 1;
    for (uint32_t i = 0; i < d; ++i) wp = std::max<uint64_t>(wp, (uint64_t)gl_ychunks(c.sigma[i + 1], n) << n);
    p.off_wpart = take(E * wp);
  }
  const uint64_t big = 1ull << std::max(c.s(0), c.s(d));
  const uint64_t words = (2 * big + kChunkWords - 1) / kChunkWords * 8;
  p.off_dig_a = take(4 * words);
  p.off_dig_b = take(4 * words);
  p.off_dig_in = take(32);
  p.off_dig_out = take(32);
  p.off_chal = take(E * (chal + 8));
  p.off_state = take(sizeof(GlState));
  c.plan.total = off;
}

size_t gl_proof_bytes(const gkr_circuit& c) {
  size_t t = 0;
  for (uint32_t i = 0; i < c.depth; ++i) t += gl_layer_proof_words(c, i) * 8;
  return t;
}

}  // namespace gkr

using namespace gkr;

extern "C" int32_t gkr_gl_prove_circuit(const gkr_circuit* c, const uint64_t* d_inputs, uint64_t seed,
                                        uint64_t* d_outputs, uint8_t* d_proof, size_t proof_cap, size_t* proof_len,
                                        void* d_ws, size_t ws_bytes, void* stream) {
  if (!c || !d_inputs || !d_outputs || !d_proof) {
    set_error("null argument");
    return GKR_EINVAL;
  }
  if (c->field != GKR_FIELD_GOLDILOCKS) {
    set_error("gkr_gl_prove_circuit takes circuits created for the Goldilocks field");
    return GKR_EINVAL;
  }
  if ((reinterpret_cast<uintptr_t>(d_inputs) & 15) ||
      ((reinterpret_cast<uintptr_t>(d_outputs) | reinterpret_cast<uintptr_t>(d_proof)) & 7)) {
    set_error("d_inputs must be 16-byte aligned, d_outputs and d_proof 8-byte aligned");
    return GKR_EINVAL;
  }
  const size_t need = gl_proof_bytes(*c);
  if (proof_len) *proof_len = need;
  if (proof_cap < need) {
    set_error("proof buffer too small: " + std::to_string(proof_cap) + " < " + std::to_string(need));
    return GKR_EBUFSZ;
  }
  int32_t rc = check_ws(c, d_ws, ws_bytes);
  if (rc) return rc;
  try {
    const GlWs w = gl_bind(*c, d_ws, d_inputs, d_outputs);
    Program pg;
    gl_emit_proof(pg.steps, *c, w, seed, reinterpret_cast<uint64_t*>(d_proof), current_tuning());
    pg.run(static_cast<hipStream_t>(stream));
  } catch (const std::bad_alloc&) {
    set_error("host allocation failed");
    return GKR_ENOMEM;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error(std::string("kernel launch failed: ") + hipGetErrorString(e));
    return GKR_EDEVICE;
  }
  return GKR_OK;
}
