// Step bodies of the GKR prover kernels (device code, included by the plain
// kernels and by the persistent batch kernel).
//
// Grid-wide bodies run with 256-thread workgroups (four 64-wide waves); the
// single-workgroup tails take any multiple of 64 threads from 128 to 1024
// (512 in the plain kernels, 256 in the batch kernel). Field
// elements are 32-byte records in Montgomery form, loaded and stored as two
// 16-byte vectors, so consecutive threads touch consecutive records and every
// access of a table sweep is coalesced. Gate g = z*2^n + c keeps the copy
// index in the low bits: a gather W[(y_z << n) | c] over consecutive c is
// contiguous.
//
// A body works over (tile, ntiles): tile plays the role of the workgroup index
// and ntiles of the grid size. The plain path launches one kernel per step
// with grid = ntiles; the persistent batch kernel hands tiles of many proofs'
// steps to resident workgroups.
//
// Reductions over a whole table (the round polynomials of the sumcheck) end in
// the last tile to finish: each tile stores its partial sums past its L2 and
// counts itself on an atomic counter; the tile that brings the counter to
// ntiles adds the partials and runs the round's Fiat-Shamir step: its first wave hashes the sums and takes the
// challenge, its second wave moves the claim through the previous round
// (the products by r stay off the chain of hashes).
// Challenges and claims never leave device memory, so a proof is a plain
// sequence of launches on one stream.
#pragma once

#include "gkr_device.hpp"
#include "gkr_kernels.hpp"
#include "fr_row.hpp"
#include "sha256_wave.hpp"

namespace gkr {


// ---------------------------------------------------------- transcript

// A challenge is the chaining value's candidate (254 bits, little-endian),
// accepted when it is below p; until then the state is rehashed with "GKRC".
// The challenge is v * 2^-256 mod p, so v itself is its Montgomery form: the
// limbs are used as they are. Each attempt is accepted with probability
// p / 2^254 > 3/4; the bound on attempts only guarantees termination. The
// hashing runs in whole waves (sha256_wave.hpp).

// The shared words of a workgroup's hashing wave.
__device__ __forceinline__ ShaBuf* sha_buf() {
  __shared__ __attribute__((aligned(16))) ShaBuf buf;
  return &buf;
}

__device__ __forceinline__ Fr fr_one_canonical() { return fr_make(1, 0, 0, 0, 0, 0, 0, 0); }

// The value of lane `src` (a constant) in every lane of the wave.
__device__ __forceinline__ Fr lane_fr(const Fr& a, int src) {
  Fr r;
#pragma unroll
  for (int k = 0; k < 8; ++k) r.v[k] = (uint32_t)__builtin_amdgcn_readlane((int)a.v[k], src);
  return r;
}

// Word `lane mod 16` of the block that absorbs a round: the Montgomery forms
// of the sums e0 and e2 (16 limbs in shared memory) with the round mark.
__device__ __forceinline__ uint32_t round_word(const Fr* e) {
  const uint32_t li = sha_lane() & 15;
  const uint32_t v = reinterpret_cast<const uint32_t*>(e)[li];
  return bswap32(li == 15 ? v | kRoundMark : v);
}

// The transcript half of a round, in a whole wave: one SHA-256 compression
// absorbs the round's sums (e in shared memory), and the accepted hash value
// is the challenge r in Montgomery form. No product precedes the hash, and the
// running claim is not needed (e1 enters only the message).
template <bool Helped>
__device__ __forceinline__ void round_hash_wave(ShaLanes& state, const Fr* e,
                                                ShaHelper* help, uint32_t base) {
  state = sha_compress_wave<Helped>(state, round_word(e), sha_buf(), help, base);
  sha_accept_wave(state, sha_buf());
}

// The challenge of an accepted state to one or two places (r_sh in shared memory).
__device__ __forceinline__ void store_challenge(const ShaLanes& state, Fr* r_sh, Fr* r_out) {
  const uint32_t lane = sha_lane();
  if (lane == 0 || lane == 8) {
    uint32_t v[4];
    sha_candidate_limbs(state, v);
    const uint32_t o = lane ? 0 : 4;
    if (r_sh) {
#pragma unroll
      for (int k = 0; k < 4; ++k) r_sh->v[o + k] = v[k];
    }
    GlobalU4* q = (GlobalU4*)r_out;
    q[lane ? 0 : 1] = U32x4{v[0], v[1], v[2], v[3]};
  }
}

// The product half: the next claim g(r) = e0 + r (e1 - e0) + r (r - 1)
// (e2 - 2 e1 + e0) / 2, evaluated as e0 + r (A + r B) with B = (e2 - 2 e1 +
// e0) / 2 and A = e1 - e0 - B, and the message (e0, e1, e2, canonical) stored
// by lanes 1..3 (one element each) to msg_out. The products run in different
// lanes: two rounds of products, both in every lane of the wave.
__device__ __forceinline__ Fr round_claim_wave(const Fr& r, const Fr& e0, const Fr& e1, const Fr& e2,
                                               uint32_t* msg_out) {
  const int lane = threadIdx.x & 63;
  const Fr B = fr_half(fr_add(fr_sub(e2, fr_double(e1)), e0));
  const Fr A = fr_sub(fr_sub(e1, e0), B);
  // lane 0: r B; lanes 1..3: canonical e0, e1, e2 (register selects over
  // opaque candidates: no private array for the optimizer to index)
  Fr c1 = e0, c2 = e1, c3 = e2, one = fr_one_canonical();
#pragma unroll
  for (int k = 0; k < 8; ++k) asm volatile("" : "+v"(c1.v[k]), "+v"(c2.v[k]), "+v"(c3.v[k]), "+v"(one.v[k]));
  Fr a = r, b = B;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    a.v[k] = lane == 1 ? c1.v[k] : (lane == 2 ? c2.v[k] : (lane == 3 ? c3.v[k] : a.v[k]));
    b.v[k] = lane == 0 ? b.v[k] : one.v[k];
  }
  const Fr prod = fr_mul(a, b);
  if (lane >= 1 && lane <= 3) stf(reinterpret_cast<Fr*>(msg_out), lane - 1, prod);
  const Fr t = fr_mul(r, fr_add(A, lane_fr(prod, 0)));
  return fr_add(e0, t);
}

// A phase's final value (a whole wave; v the same in every lane): store it,
// write it to the proof and absorb it.
__device__ __forceinline__ void finish_value_wave(ShaLanes& state, const Fr& v, Fr* v_out,
                                                  uint32_t* proof_out) {
  const Fr c = fr_from_mont(v);
  sha_absorb_words_wave(state, sha_buf(), kTagValue, bswap32(lane_limb(c)));
  if ((threadIdx.x & 63) == 0) {
    *v_out = v;
    stf(reinterpret_cast<Fr*>(proof_out), 0, c);
  }
}

// ---------------------------------------------------------------- bodies

#define GTID ((uint64_t)tile * kBlock + threadIdx.x)
#define GSTRIDE ((uint64_t)ntiles * kBlock)

// ST_TO_MONT: p0 canonical in, p1 out, q0 count.
__device__ __forceinline__ void body_to_mont(const Step& st, uint32_t tile, uint32_t ntiles) {
  const Fr* in = P<const Fr*>(st, 0);
  Fr* out = P<Fr*>(st, 1);
  for (uint64_t i = GTID; i < st.q[0]; i += GSTRIDE) stf(out, i, fr_to_mont(ldf(in, i)));
}

// ST_FROM_MONT: p0 in, p1 canonical out, q0 count.
__device__ __forceinline__ void body_from_mont(const Step& st, uint32_t tile, uint32_t ntiles) {
  const Fr* in = P<const Fr*>(st, 0);
  Fr* out = P<Fr*>(st, 1);
  for (uint64_t i = GTID; i < st.q[0]; i += GSTRIDE) stf(out, i, fr_from_mont(ldf(in, i)));
}

// ST_FORWARD: V_i[z*2^n + c] = W[x_z*2^n + c] (+ or *) W[y_z*2^n + c].
// p0 W, p1 V, p2 gate records, u0 n, u1 log2 gates, u2 log2 columns of a block, q0 count.
// Bound by memory; a row is read twice on average (see forward_block_log).
__device__ __forceinline__ void body_forward(const Step& st, uint32_t tile, uint32_t ntiles) {
  const Fr* __restrict__ W = P<const Fr*>(st, 0);
  Fr* __restrict__ V = P<Fr*>(st, 1);
  const uint2* __restrict__ gates = P<const uint2*>(st, 2);
  const uint32_t n = st.u[0];
  for (uint64_t g = GTID; g < st.q[0]; g += GSTRIDE) {
    const RowCol zc = block_order(g, st.u[1], st.u[2]);
    const uint64_t c = zc.col;
    const uint2 gate = gates[zc.row];
    const uint64_t x = gate.x & 0x7fffffffu, y = gate.y;
    const Fr a = ldf(W, (x << n) | c), b = ldf(W, (y << n) | c);
    stf(V, zc.row << n | c, (gate.x >> 31) ? fr_mul(a, b) : fr_add(a, b));
  }
}

// ST_DIGEST: one level of a tree digest; chunk t of q0 words (256 words, 1 KiB,
// per chunk) is hashed by thread t; element words are byte-swapped (limbs are
// little-endian). p0 in, p1 out, q0 nwords, q1 nchunks, u0 swap; p2, p3, q2, q3, u1 the
// same of a second vector (q3 = 0: none), whose chunks come after.
__device__ __forceinline__ void body_digest(const Step& st, uint32_t tile, uint32_t ntiles) {
  for (uint64_t g = GTID; g < st.q[1] + st.q[3]; g += GSTRIDE) {
    const bool second = g >= st.q[1];
    const uint32_t* in = second ? P<const uint32_t*>(st, 2) : P<const uint32_t*>(st, 0);
    uint32_t* out = second ? P<uint32_t*>(st, 3) : P<uint32_t*>(st, 1);
    const uint64_t nwords = second ? st.q[2] : st.q[0], t = second ? g - st.q[1] : g;
    const uint32_t swap = second ? st.u[1] : st.u[0];
    const uint64_t begin = t * kChunkWords;
    const uint64_t end = (begin + kChunkWords < nwords) ? begin + kChunkWords : nwords;
    const uint64_t len = end - begin;  // a multiple of 8 words
    Sha256State sh = sha256_iv();
    const uint4* src = reinterpret_cast<const uint4*>(in + begin);
    const uint64_t full = len / 16;
    for (uint64_t b = 0; b < full; ++b) {
      Sha256Block blk;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint4 v = src[b * 4 + q];
        blk.w[4 * q + 0] = swap ? bswap32(v.x) : v.x;
        blk.w[4 * q + 1] = swap ? bswap32(v.y) : v.y;
        blk.w[4 * q + 2] = swap ? bswap32(v.z) : v.z;
        blk.w[4 * q + 3] = swap ? bswap32(v.w) : v.w;
      }
      sh = sha256_compress_v(sh, blk);
    }
    Sha256Block blk;
#pragma unroll
    for (int i = 0; i < 16; ++i) blk.w[i] = 0;
    if (len - full * 16 == 8) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint4 v = src[full * 4 + q];
        blk.w[4 * q + 0] = swap ? bswap32(v.x) : v.x;
        blk.w[4 * q + 1] = swap ? bswap32(v.y) : v.y;
        blk.w[4 * q + 2] = swap ? bswap32(v.z) : v.z;
        blk.w[4 * q + 3] = swap ? bswap32(v.w) : v.w;
      }
      blk.w[8] = 0x80000000u;
    } else {
      blk.w[0] = 0x80000000u;
    }
    const uint64_t bits = len * 32;
    blk.w[14] = (uint32_t)(bits >> 32);
    blk.w[15] = (uint32_t)bits;
    sh = sha256_compress_v(sh, blk);
#pragma unroll
    for (int k = 0; k < 8; ++k) out[t * 8 + k] = sh.h[k];
  }
}

// ST_DIGEST_WAVE: one level of one or two tree digests with few chunks, a
// workgroup per chunk: p0 in, p1 out, q0 words, q1 chunks, u0 swap; the same of
// the second vector in p2, p3, q2, q3, u1 (tiles from q1 on). The blocks of a
// chunk chain, so a thread hashing a chunk alone needs 17 x 5,900 cycles (55 us
// per level); here the schedules of all blocks are written first, 16 at a time
// (one per row of 16 lanes), and one wave runs the rounds: 17 x 3,140 cycles.
__device__ __forceinline__ void body_digest_wave(const Step& st, uint32_t tile, uint32_t) {
  constexpr uint32_t kMaxBlocks = kChunkWords / 16 + 1;
  __shared__ __attribute__((aligned(16))) uint32_t wk[kMaxBlocks][64];
  __shared__ __attribute__((aligned(16))) uint32_t one4[4];
  const bool second = tile >= st.q[1];
  const uint32_t* in = second ? P<const uint32_t*>(st, 2) : P<const uint32_t*>(st, 0);
  uint32_t* out = second ? P<uint32_t*>(st, 3) : P<uint32_t*>(st, 1);
  const uint64_t nwords = second ? st.q[2] : st.q[0], t = second ? tile - st.q[1] : tile;
  const uint32_t swap = second ? st.u[1] : st.u[0];
  const uint64_t begin = t * kChunkWords;
  const uint32_t len = (uint32_t)(begin + kChunkWords < nwords ? kChunkWords : nwords - begin);
  const uint32_t nblk = (len + 3 + 15) / 16, li = threadIdx.x & 15;
  const uint32_t c0 = kSha256K[li], c1 = kSha256K[16 + li], c2 = kSha256K[32 + li], c3 = kSha256K[48 + li];
  if (threadIdx.x < 4) one4[threadIdx.x] = 1;
  // (whole waves: the schedule reads its neighbours' lanes)
  for (uint32_t b0 = 0; b0 < nblk; b0 += kBlock / 16) {
    const uint32_t b = b0 + threadIdx.x / 16;
    const uint32_t i = 16 * b + li;
    uint32_t w = 0;
    if (i < len) {
      w = in[begin + i];
      if (swap) w = bswap32(w);
    } else if (i == len) {
      w = 0x80000000u;
    } else if (i == 16 * nblk - 1) {
      w = len * 32;
    }
    const uint32_t w1 = sha_schedule(w), w2 = sha_schedule(w1), w3 = sha_schedule(w2);
    if (b < nblk) {
      wk[b][li] = w + c0;
      wk[b][16 + li] = w1 + c1;
      wk[b][32 + li] = w2 + c2;
      wk[b][48 + li] = w3 + c3;
    }
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    ShaLanes sh = sha_lanes_iv();
    for (uint32_t b = 0; b < nblk; ++b) sh = sha_compress_given(sh, wk[b], one4);
    sha_lanes_store(out + 8 * t, sh);
  }
}

// ST_TRANSCRIPT_BEGIN: st = seed state (w0..7), then absorb the circuit digest
// (w8..15) and the two vector digests; also zeroes the reduction counter and
// clears the pending round.
// p0 S, p1 dig_in, p2 dig_out.
__device__ __forceinline__ void body_transcript_begin(const Step& st, uint32_t, uint32_t) {
  if (threadIdx.x >= 64) return;
  DevState* S = P<DevState*>(st, 0);
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
  if (threadIdx.x == 0) {
    S->counter = 0;
    S->pending = 0;
  }
}

// ST_SQUEEZE: u0 challenges into p1 (Montgomery form). p0 S.
__device__ __forceinline__ void body_squeeze(const Step& st, uint32_t, uint32_t) {
  if (threadIdx.x >= 64) return;
  DevState* S = P<DevState*>(st, 0);
  Fr* out = P<Fr*>(st, 1);
  sha_init(sha_buf());
  ShaLanes sh = sha_lanes_load(S->st);
  for (uint32_t k = 0; k < st.u[0]; ++k) {
    sha_rehash_wave(sh, sha_buf());
    sha_accept_wave(sh, sha_buf());
    store_challenge(sh, nullptr, out + k);
  }
  sha_lanes_store(S->st, sh);
}

// ST_LAYER_BEGIN: draw alpha, beta (layer > 0) and set the claim to
// alpha * vu + beta * vv; on layer 0 (u0 = 1) alpha = 1, beta = 0 and claim = vu.
// p0 S, p1 vu, p2 vv.
__device__ __forceinline__ void body_layer_begin(const Step& st, uint32_t, uint32_t) {
  if (threadIdx.x >= 64) return;
  DevState* S = P<DevState*>(st, 0);
  const Fr vu = opaque(*P<const Fr*>(st, 1)), vv = opaque(*P<const Fr*>(st, 2));
  if (st.u[0]) {
    if (threadIdx.x == 0) {
      S->alpha = fr_one();
      S->beta = fr_zero();
      S->claim = vu;
    }
    return;
  }
  sha_init(sha_buf());
  ShaLanes sh = sha_lanes_load(S->st);
  const Fr a = sha_squeeze_wave(sh, sha_buf());
  const Fr b = sha_squeeze_wave(sh, sha_buf());
  sha_lanes_store(S->st, sh);
  const Fr claim = fr_mul_add2(opaque(a), vu, opaque(b), vv);
  if (threadIdx.x == 0) {
    S->alpha = a;
    S->beta = b;
    S->claim = claim;
  }
}

// ST_EQ: up to four tables out_j[b] = scale_j * prod_k (bit_k(b) ? r_k : 1 - r_k),
// bit 1 = MSB. u0..3 bits, u4 count; p0..3 points, p4..7 scales (null = 1), p8..11 outs.
// A workgroup first computes, for every table, the 16 products of each group
// of four variables (groups from the last variable on; the scale in the first
// group, which may be short), a thread per product; an entry is then a product
// of bits / 4 of them. An entry alone in its thread took bits + 3 products one
// after another: 17 us for 12 bits, now 8.
constexpr uint32_t kEqGroups = 4 * ((GKR_MAX_LOG_WIDTH + 3) / 4);

__device__ __forceinline__ void body_eq(const Step& st, uint32_t tile, uint32_t ntiles) {
  __shared__ Fr grp[kEqGroups][16];
  uint64_t total = 0;
  uint32_t groups = 0;
  for (uint32_t j = 0; j < st.u[4]; ++j) {
    total += 1ull << st.u[j];
    groups += (st.u[j] + 3) / 4;
  }
  for (uint32_t t = threadIdx.x; t < 16 * groups; t += kBlock) {
    const uint32_t c = t & 15;
    uint32_t g = t >> 4, j = 0;
    while (g >= (st.u[j] + 3) / 4) {
      g -= (st.u[j] + 3) / 4;
      ++j;
    }
    // group g of table j: bits 4 g .. 4 g + 3 of the index (from the low end)
    const Fr* r = P<const Fr*>(st, j);
    const Fr* scale = P<const Fr*>(st, 4 + j);
    const uint32_t k = st.u[j], have = k - 4 * g < 4 ? k - 4 * g : 4;
    auto factor = [&](uint32_t b) {
      if (b >= have) return fr_one();
      const Fr ri = opaque(ldf(r, k - 1 - 4 * g - b));
      return (c >> b) & 1 ? ri : fr_one_minus(ri);
    };
    Fr v = fr_mul(factor(0), factor(1));
    if (have > 2) v = fr_mul(v, fr_mul(factor(2), factor(3)));
    if (g == 0 && scale) v = fr_mul(v, opaque(*scale));
    grp[t >> 4][c] = v;
  }
  __syncthreads();
  for (uint64_t g = (uint64_t)tile * kBlock + threadIdx.x; g < total; g += (uint64_t)ntiles * kBlock) {
    uint64_t t = g;
    uint32_t j = 0, base = 0;
    while (t >= (1ull << st.u[j])) {
      t -= 1ull << st.u[j];
      base += (st.u[j] + 3) / 4;
      ++j;
    }
    const uint32_t k = st.u[j];
    Fr v;
    if (k == 0) {
      const Fr* scale = P<const Fr*>(st, 4 + j);
      v = scale ? *scale : fr_one();
    } else {
      v = grp[base][t & 15];
      for (uint32_t q = 1; 4 * q < k; ++q) v = fr_mul(v, opaque(grp[base + q][(t >> (4 * q)) & 15]));
    }
    stf(P<Fr*>(st, 8 + j), t, v);
  }
  __syncthreads();  // the batch kernel may run another tile next
}

// ST_WSUM: sum_e V[e] A[e >> n] B[e & mask] into *p5.
// p0 V, p1 A, p2 B, p3 partials, p4 S, p5 dst, u0 n, q0 count.
__device__ __forceinline__ void body_wsum(const Step& st, uint32_t tile, uint32_t ntiles) {
  const Fr* V = P<const Fr*>(st, 0);
  const Fr* A = P<const Fr*>(st, 1);
  const Fr* B = P<const Fr*>(st, 2);
  const uint32_t n = st.u[0];
  const uint64_t mask = (1ull << n) - 1;
  Fr acc[1] = {fr_zero()};
  for (uint64_t e = GTID; e < st.q[0]; e += GSTRIDE)
    acc[0] = fr_add(acc[0], fr_mul(fr_mul(ldf(V, e), ldf(A, e >> n)), ldf(B, e & mask)));
  write_partial<1>(acc, P<Fr*>(st, 3), tile);
}
__device__ __forceinline__ void finish_wsum(const Step& st, uint32_t ntiles) {
  Fr tot[1];
  sum_partials<1>(P<const Fr*>(st, 3), ntiles, tot);
  if (threadIdx.x == 0) *P<Fr*>(st, 5) = tot[0];
}

// Phase-1 bookkeeping tables over (x, c):
//   G[x,c] = sum_{MUL z: x_z=x} T[z,c] W[y_z,c] + sum_{ADD z: x_z=x} T[z,c]
//   H[x,c] = sum_{ADD z: x_z=x} T[z,c] W[y_z,c]
// with T[z,c] = aU[z] Cu[c] + bV[z] Cv[c] (the factored eq of both claims).
// p0 W, p1 G, p2 H, p3 xrow, p4 xent, p5 aU, p6 bV, p7 Cu, p8 Cv, u0 n.
__device__ __forceinline__ void phase1_entry(const Step& st, uint64_t e, Fr& g, Fr& h) {
  const Fr* __restrict__ W = P<const Fr*>(st, 0);
  const uint32_t* __restrict__ xrow = P<const uint32_t*>(st, 3);
  const uint2* __restrict__ xent = P<const uint2*>(st, 4);
  const Fr* __restrict__ aU = P<const Fr*>(st, 5);
  const Fr* __restrict__ bV = P<const Fr*>(st, 6);
  const uint32_t n = st.u[0];
  const uint64_t mask = (1ull << n) - 1;
  const uint64_t x = e >> n, c = e & mask;
  const Fr cu = ldf(P<const Fr*>(st, 7), c), cv = ldf(P<const Fr*>(st, 8), c);
  g = fr_zero();
  h = fr_zero();
  // The first gate's terms are assigned, not added to zero: with 2^n >= 64
  // copies every lane of a wave walks the same gate list (the entries of one
  // x), so these branches do not diverge and an entry with one gate costs no
  // additions.
  const uint32_t k0 = xrow[x], k1 = xrow[x + 1];
  for (uint32_t k = k0; k < k1; ++k) {
    const uint2 ent = xent[k];
    const uint64_t z = ent.x, y = ent.y & 0x7fffffffu;
    const Fr T = fr_mul_add2(ldf(aU, z), cu, ldf(bV, z), cv);
    const Fr tw = fr_mul(T, ldf(W, (y << n) | c));
    if (k == k0) {
      if (ent.y >> 31) {
        g = tw;
      } else {
        g = T;
        h = tw;
      }
    } else if (ent.y >> 31) {
      g = fr_add(g, tw);
    } else {
      g = fr_add(g, T);
      h = fr_add(h, tw);
    }
  }
}

// ST_P1_INIT: the tables alone; q0 count.
__device__ __forceinline__ void body_p1_init(const Step& st, uint32_t tile, uint32_t ntiles) {
  Fr* G = P<Fr*>(st, 1);
  Fr* H = P<Fr*>(st, 2);
  for (uint64_t e = GTID; e < st.q[0]; e += GSTRIDE) {
    Fr g, h;
    phase1_entry(st, e, g, h);
    stf(G, e, g);
    stf(H, e, h);
  }
}

// ST_P1_INIT_ROUND: the tables and the first round together: b builds entries
// b and b + half and evaluates the round-1 pair at t = 0, 2. With Lazy the
// t = 0 products of a thread's pairs are summed unreduced (a 512-bit
// accumulator, one reduction per 16 pairs; a thread takes many pairs here; a
// second accumulator for t = 2 would not fit the registers of three
// workgroups per CU); the batch kernel, which holds every body, takes the
// reduced form (Lazy = false) to stay within its registers.
// q0 half; p9 S, p10 partials, p11 r_out, p12 msg.
template <bool Lazy>
__device__ __forceinline__ void body_p1_init_round(const Step& st, uint32_t tile, uint32_t ntiles) {
  const Fr* W = P<const Fr*>(st, 0);
  Fr* G = P<Fr*>(st, 1);
  Fr* H = P<Fr*>(st, 2);
  const uint64_t half = st.q[0];
  Fr acc[2] = {fr_zero(), fr_zero()};
  FrWide e0 = frw_zero();
  uint32_t lazy = 0;
  // Lazy: the running sums wait in shared memory (a slot per thread), out of
  // the registers the gate walks need
  __shared__ Fr sacc[Lazy ? 2 : 1][Lazy ? kBlock : 1];
  __shared__ FrWide swide[Lazy ? kBlock : 1];
  if constexpr (Lazy) {
    sacc[0][threadIdx.x] = fr_zero();
    sacc[1][threadIdx.x] = fr_zero();
    swide[threadIdx.x] = frw_zero();
  }
  for (uint64_t b = GTID; b < half; b += GSTRIDE) {
    Fr g0, h0, g1, h1;
    phase1_entry(st, b, g0, h0);
    phase1_entry(st, b + half, g1, h1);
    stf(G, b, g0);
    stf(H, b, h0);
    stf(G, b + half, g1);
    stf(H, b + half, h1);
    const Fr w0 = ldf(W, b), w1 = ldf(W, b + half);
    const Fr w2 = fr_sub(fr_double(w1), w0), g2 = fr_sub(fr_double(g1), g0), h2 = fr_sub(fr_double(h1), h0);
    if constexpr (!Lazy) {
      acc[0] = fr_add(acc[0], fr_add(fr_mul(w0, g0), h0));
      acc[1] = fr_add(acc[1], fr_add(fr_mul(w2, g2), h2));
      continue;
    }
    FrWide ew = swide[threadIdx.x];
    frw_mac(ew, w0, g0);
    Fr a0 = fr_add(sacc[0][threadIdx.x], h0);
    sacc[1][threadIdx.x] = fr_add(sacc[1][threadIdx.x], fr_add(fr_mul(w2, g2), h2));
    if (++lazy == 16) {
      a0 = fr_add(a0, frw_reduce<16>(ew));
      ew = frw_zero();
      lazy = 0;
    }
    swide[threadIdx.x] = ew;
    sacc[0][threadIdx.x] = a0;
  }
  if constexpr (Lazy) {
    acc[0] = sacc[0][threadIdx.x];
    acc[1] = sacc[1][threadIdx.x];
    if (lazy) acc[0] = fr_add(acc[0], frw_reduce<16>(swide[threadIdx.x]));
  }
  write_partial<2>(acc, P<Fr*>(st, 10), tile);
}

// Sum of the partials, then the round's transcript step in wave 0: the hash
// of (e0, e2) gives r, and the round becomes the pending one. Meanwhile wave 1
// moves the claim through the previous pending round (if any) and writes that
// round's message, so the products by r stay off the chain of hashes.
// With Late (the batch kernel, which has no registers to spare) the transcript
// state and constants are loaded after the sum instead of during it.
template <bool Late>
__device__ __forceinline__ void finish_reduced_round(const Fr* partials, uint32_t ntiles, DevState* S, Fr* r_out,
                                     uint32_t* msg) {
  const uint32_t wid = threadIdx.x >> 6;
  __shared__ Fr e_sh[2];
  __shared__ ShaHelper help;
  // wave 0 fetches the transcript state while the partials are summed; wave 2
  // writes the hash's schedule
  ShaLanes st;
  auto fetch = [&] {
    if (wid == 0) {
      st = sha_lanes_load(S->st);
      sha_init(sha_buf());
    }
  };
  if constexpr (!Late) fetch();
  if (threadIdx.x == 0) help.ready = 0;
  if constexpr (Late) {
    Fr tot[2];
    sum_partials<2>(partials, ntiles, tot);
    if (threadIdx.x == 0) {
      e_sh[0] = tot[0];
      e_sh[1] = tot[1];
    }
  } else {
    // lanes 0..31 of each wave take the sums at t = 0, lanes 32..63 those at t = 2
    __shared__ Fr red[16][2];
    const uint32_t lane = threadIdx.x & 63, pt = lane >> 5, nw = blockDim.x >> 6;
    const uint32_t busy = (ntiles + 31) / 32 < nw ? (ntiles + 31) / 32 : nw;  // waves with partials
    if (wid < busy) {
      Fr v = fr_zero();
      for (uint32_t i = wid * 32 + (lane & 31); i < ntiles; i += nw * 32) v = fr_add(v, get_partial(partials, 2ull * i + pt));
      v = half_wave_sum(v);
      if ((lane & 31) == 31) red[wid][pt] = v;
    }
    __syncthreads();
    if (wid == 0) {
      Fr v = red[0][pt];
      for (uint32_t w = 1; w < busy; ++w) v = fr_add(v, red[w][pt]);
      if ((lane & 31) == 0) e_sh[pt] = v;
    }
  }
  bool pend = false;
  Fr claim, pe0, pe2, pr;
  uint32_t* pmsg = nullptr;
  if (wid == 1) {
    pend = S->pending != 0;
    if (pend) {
      claim = S->claim;
      pe0 = S->pend_e0;
      pe2 = S->pend_e2;
      pr = S->pend_r;
      pmsg = S->pend_msg;
    }
  }
  if constexpr (Late) fetch();
  // wave 1 has read the pending round before wave 0 overwrites it
  __syncthreads();
  if (wid == 0) {
    round_hash_wave<true>(st, e_sh, &help, 0);
    sha_lanes_store(S->st, st);
    store_challenge(st, nullptr, r_out);
    store_challenge(st, nullptr, &S->pend_r);
    if (threadIdx.x == 0) {
      S->pend_e0 = e_sh[0];
      S->pend_e2 = e_sh[1];
      S->pend_msg = msg;
      S->pending = 1;
    }
  } else if (wid == 2) {
    sha_help(round_word(e_sh), sha_buf(), &help, 0);
  } else if (wid == 1 && pend) {
    claim = round_claim_wave(pr, pe0, fr_sub(claim, pe0), pe2, pmsg);
    if (threadIdx.x == 64) S->claim = claim;
  }
}

template <bool Late>
__device__ __forceinline__ void finish_p1_init_round(const Step& st, uint32_t ntiles) {
  finish_reduced_round<Late>(P<const Fr*>(st, 10), ntiles, P<DevState*>(st, 9), P<Fr*>(st, 11), P<uint32_t*>(st, 12));
}

// Entries b and b + half of one table of a round. With Fold the source has
// 4*half entries and is first folded by r (entry i of the folded table is
// src[i] + r (src[i + 2 half] - src[i])); the folded entries are stored to dst.
template <bool Fold>
__device__ __forceinline__ void pair_entries(const Fr* src, Fr* dst, uint64_t b, uint64_t half, const Fr& r,
                                             Fr& lo, Fr& hi) {
  if constexpr (Fold) {
    const uint64_t m = 2 * half;
    const Fr a0 = ldf(src, b), a1 = ldf(src, b + m);
    const Fr b0 = ldf(src, b + half), b1 = ldf(src, b + half + m);
    lo = fr_add(a0, fr_mul(r, fr_sub(a1, a0)));
    hi = fr_add(b0, fr_mul(r, fr_sub(b1, b0)));
    stf(dst, b, lo);
    stf(dst, b + half, hi);
  } else {
    lo = ldf(src, b);
    hi = ldf(src, b + half);
  }
}

// One pair b of a round: the round polynomial's terms at t = 0 (the entry b)
// and t = 2 (2 * entry(b + half) - entry(b)). The last table of a form is
// additive, the others multiply in pairs (0,1), (2,3). Tables are visited one
// group at a time (scheduling barriers between groups) so that only one
// group's operands are live.
template <class Form, bool Fold>
__device__ __forceinline__ void round_pair(const Fr* const* src, Fr* const* dst, uint64_t b,
                                           uint64_t half, const Fr& r, Fr& acc0, Fr& acc2) {
  constexpr int NT = Form::NT;
  {
    Fr lo, hi;
    pair_entries<Fold>(src[NT - 1], dst[NT - 1], b, half, r, lo, hi);
    acc0 = fr_add(acc0, lo);
    acc2 = fr_add(acc2, fr_sub(fr_double(hi), lo));
  }
  if constexpr (NT == 3) {
    __builtin_amdgcn_sched_barrier(0);
    Fr xl, xh, yl, yh;
    pair_entries<Fold>(src[0], dst[0], b, half, r, xl, xh);
    pair_entries<Fold>(src[1], dst[1], b, half, r, yl, yh);
    acc0 = fr_add(acc0, fr_mul(xl, yl));
    acc2 = fr_add(acc2, fr_mul(fr_sub(fr_double(xh), xl), fr_sub(fr_double(yh), yl)));
  } else {
    // both product pairs of a FormB pair at once: one reduction per point
    __builtin_amdgcn_sched_barrier(0);
    Fr pl, ph, fl, fh;
    pair_entries<Fold>(src[0], dst[0], b, half, r, pl, ph);
    pair_entries<Fold>(src[1], dst[1], b, half, r, fl, fh);
    __builtin_amdgcn_sched_barrier(0);
    Fr ql, qh, gl, gh;
    pair_entries<Fold>(src[2], dst[2], b, half, r, ql, qh);
    pair_entries<Fold>(src[3], dst[3], b, half, r, gl, gh);
    acc0 = fr_add(acc0, fr_mul_add2(pl, fl, ql, gl));
    acc2 = fr_add(acc2, fr_mul_add2(fr_sub(fr_double(ph), pl), fr_sub(fr_double(fh), fl),
                                    fr_sub(fr_double(qh), ql), fr_sub(fr_double(gh), gl)));
  }
  __builtin_amdgcn_sched_barrier(0);
}

// The pairs [b0, half) with stride `stride` of one round, accumulated.
template <class Form>
__device__ __forceinline__ void round_range(const Fr* const* src, Fr* const* dst, uint64_t b0, uint64_t stride,
                                            uint64_t half, bool fold, const Fr& r, Fr& acc0, Fr& acc2) {
  if (fold) {
    for (uint64_t b = b0; b < half; b += stride) round_pair<Form, true>(src, dst, b, half, r, acc0, acc2);
  } else {
    for (uint64_t b = b0; b < half; b += stride) round_pair<Form, false>(src, dst, b, half, r, acc0, acc2);
  }
}

// ST_ROUND_A / ST_ROUND_B: one sumcheck round (optional fold by the previous
// challenge, evaluation at t = 0, 2); q0 half. Pointers: src[0..NT),
// dst[NT..2NT), then rprev, S, partials, r_out, msg (RoundPtrs).
template <class Form>
__device__ __forceinline__ void body_round(const Step& st, uint32_t tile, uint32_t ntiles) {
  using R = RoundPtrs<Form::NT>;
  const Fr* src[Form::NT];
  Fr* dst[Form::NT];
#pragma unroll
  for (int k = 0; k < Form::NT; ++k) {
    src[k] = P<const Fr*>(st, k);
    dst[k] = P<Fr*>(st, Form::NT + k);
  }
  const Fr* rprev = P<const Fr*>(st, R::kR);
  const bool fold = rprev != nullptr;
  const Fr r = fold ? ldf(rprev, 0) : fr_zero();
  const uint64_t half = st.q[0];
  Fr acc[2] = {fr_zero(), fr_zero()};
  round_range<Form>(src, dst, GTID, GSTRIDE, half, fold, r, acc[0], acc[1]);
  write_partial<2>(acc, P<Fr*>(st, R::kPart), tile);
}
template <class Form, bool Late>
__device__ __forceinline__ void finish_round_step(const Step& st, uint32_t ntiles) {
  using R = RoundPtrs<Form::NT>;
  finish_reduced_round<Late>(P<const Fr*>(st, R::kPart), ntiles, P<DevState*>(st, R::kS), P<Fr*>(st, R::kROut),
                       P<uint32_t*>(st, R::kMsg));
}

// Table k of NT pointers, for a k that varies across lanes: a chain of
// register selects. Each candidate passes through an empty asm statement, so
// the optimizer cannot turn the chain back into an indexed load from a
// private array (which would put the pointers in scratch memory and add a
// dependent load to every task).
template <int NT, class T>
__device__ __forceinline__ T pick(T const (&a)[NT], uint32_t k) {
  uint64_t p = reinterpret_cast<uint64_t>(a[0]);
#pragma unroll
  for (int q = 1; q < NT; ++q) {
    uint64_t c = reinterpret_cast<uint64_t>(a[q]);
    asm volatile("" : "+v"(c));
    p = k == (uint32_t)q ? c : p;
  }
  return reinterpret_cast<T>(p);
}

// ST_TAIL_A / ST_TAIL_B: the remaining u0 rounds of a phase in one workgroup
// (at least 128 threads), then the final fold. q0 = table size before the
// pending fold (if any). Pointers: src, dst, rpending, S, r_out, msg,
// final_out, proof_value. The final value of table 0 is stored in *final_out
// and, if proof_value is not null, written to the proof and absorbed.
// The transcript chain of the rounds needs only the sums e0 and e2 of each
// round (the hash absorbs them; the challenge is the hash value), not the
// running claim, so the two chains run in different waves:
//  - wave 0 holds the transcript state and hashes each round's e0, e2 as soon
//    as the sums are in, then publishes r;
//  - wave 1 holds the claim: while wave 0 hashes round j, it moves the claim
//    through round j - 1 (e1 = claim - e0, products by r) and writes that
//    round's message (in round 0, through the round a grid finisher left
//    pending, if any); the last round's claim moves after the final fold, and
//    nothing is left pending;
//  - waves 1.. (the workers) fold the tables by the previous challenge (one
//    task per entry, in place after the first round) and evaluate them at
//    t = 0 and t = 2 (one task per pair and t).
template <class Form>
__device__ __forceinline__ void body_tail(const Step& st, uint32_t, uint32_t) {
  constexpr int NT = Form::NT;
  const Fr* src[NT];
  Fr* dst[NT];
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    src[k] = P<const Fr*>(st, k);
    dst[k] = P<Fr*>(st, NT + k);
  }
  const Fr* rpending = P<const Fr*>(st, 2 * NT);
  DevState* S = P<DevState*>(st, 2 * NT + 1);
  Fr* r_out = P<Fr*>(st, 2 * NT + 2);
  uint32_t* msg = P<uint32_t*>(st, 2 * NT + 3);
  Fr* final_out = P<Fr*>(st, 2 * NT + 4);
  uint32_t* proof_value = P<uint32_t*>(st, 2 * NT + 5);
  const uint32_t wid = threadIdx.x >> 6;
  const uint32_t w = threadIdx.x - 64, nw = blockDim.x - 64;  // worker index and count
  uint64_t size = st.q[0];
  const uint32_t rounds = st.u[0];
  __shared__ Fr r_sh, e_sh[2];  // the last round's challenge and sums (e0, e2)
  __shared__ Fr red1[2];
  bool fold = rpending != nullptr;
  ShaLanes state;  // wave 0
  // wave 1: the claim and the pending round it has not moved through yet
  Fr claim = fr_zero(), pe0 = fr_zero(), pe2 = fr_zero(), pr = fr_zero();
  uint32_t* pmsg = nullptr;
  bool pend = false;
  if (wid == 0) {
    state = sha_lanes_load(S->st);
    sha_init(sha_buf());
  }
  if (wid == 1) {
    claim = S->claim;
    pend = S->pending != 0;
    if (pend) {
      pe0 = S->pend_e0;
      pe2 = S->pend_e2;
      pr = S->pend_r;
      pmsg = S->pend_msg;
    }
  }
  if (threadIdx.x == 0) r_sh = fold ? ldf(rpending, 0) : fr_zero();
  __syncthreads();
  for (uint32_t j = 0;; ++j) {
    if (fold) {
      const uint64_t m = size / 2;
      if (wid > 0) {
        // entry i of table k becomes src[i] + r (src[i + m] - src[i])
        const uint32_t lg = 63 - __clzll(m);
        const Fr rf = r_sh;
        for (uint64_t t = w; t < NT * m; t += nw) {
          const uint32_t k = (uint32_t)(t >> lg);
          const uint64_t i = t & (m - 1);
          const Fr* sp = pick<NT>(src, k);
          const Fr a0 = ldf(sp, i), a1 = ldf(sp, i + m);
          stf(pick<NT>(dst, k), i, fr_add(a0, fr_mul(rf, fr_sub(a1, a0))));
        }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < NT; ++k) src[k] = dst[k];
      size = m;
    }
    if (j == rounds) break;
    // evaluate: task u < size is the pair b = u mod half at t = 0 (u < half) or t = 2
    const uint64_t half = size / 2;
    Fr acc[2] = {fr_zero(), fr_zero()};
    if (wid > 0) {
      for (uint64_t u = w; u < size; u += nw) {
        const bool t2 = u >= half;
        const uint64_t b = t2 ? u - half : u;
        Fr x[NT];
#pragma unroll
        for (int k = 0; k < NT; ++k) {
          const Fr lo = ldf(src[k], b), hi = ldf(src[k], b + half);
          x[k] = t2 ? fr_sub(fr_double(hi), lo) : lo;
        }
        Fr v;
        if constexpr (NT == 3) v = fr_add(fr_mul(x[0], x[1]), x[2]);
        else v = fr_add(fr_mul_add2(x[0], x[1], x[2], x[3]), x[4]);
        if (t2) acc[1] = fr_add(acc[1], v);
        else acc[0] = fr_add(acc[0], v);
      }
    }
    // the claim wave takes the previous round's sums and challenge
    if (wid == 1 && j > 0) {
      pe0 = e_sh[0];
      pe2 = e_sh[1];
      pr = r_sh;
      pmsg = msg + 24 * (j - 1);
      pend = true;
    }
    if (size <= 64) {
      // Every task is in the first worker wave, one per lane: lanes [0, half)
      // hold the t = 0 terms and lanes [half, size) the t = 2 terms, so one
      // segmented sum over aligned blocks of `half` lanes (log2(half) DPP
      // steps) leaves e0 in lane half - 1 and e2 in lane size - 1.
      if (wid == 1) {
        Fr v = fr_add(acc[0], acc[1]);
        if (half >= 2) v = fr_add(v, dpp_fr<0xB1, 0xF>(v));   // quad_perm [1,0,3,2]
        if (half >= 4) v = fr_add(v, dpp_fr<0x4E, 0xF>(v));   // quad_perm [2,3,0,1]
        if (half >= 8) v = fr_add(v, dpp_fr<0x141, 0xF>(v));  // row_half_mirror
        if (half >= 16) v = fr_add(v, dpp_fr<0x140, 0xF>(v)); // row_mirror
        if (half >= 32) v = fr_add(v, dpp_fr<0x142, 0xA>(v)); // row_bcast15 into rows 1 and 3
        const uint32_t lane = threadIdx.x & 63;
        if (lane == half - 1) red1[0] = v;
        if (lane == size - 1) red1[1] = v;
      }
      __syncthreads();
      if (wid == 0) {
        acc[0] = red1[0];
        acc[1] = red1[1];
      }
    } else {
      block_sum_to_wave0<2>(acc);
    }
    if (wid == 0) {
      if (threadIdx.x == 0) {
        e_sh[0] = acc[0];
        e_sh[1] = acc[1];
      }
      lds_order();
      round_hash_wave<false>(state, e_sh, nullptr, 0);
      store_challenge(state, &r_sh, r_out + j);
    } else if (wid == 1 && pend) {
      claim = round_claim_wave(pr, pe0, fr_sub(claim, pe0), pe2, pmsg);
      pend = false;
    }
    __syncthreads();
    fold = true;
  }
  // the last round's claim move (the final fold has run)
  if (wid == 1) {
    if (rounds > 0) {
      pe0 = e_sh[0];
      pe2 = e_sh[1];
      pr = r_sh;
      pmsg = msg + 24 * (rounds - 1);
      pend = true;
    }
    if (pend) claim = round_claim_wave(pr, pe0, fr_sub(claim, pe0), pe2, pmsg);
    if (threadIdx.x == 64) {
      S->claim = claim;
      S->pending = 0;
    }
  }
  if (wid == 0) {
    const Fr v = opaque(ldf(src[0], 0));
    if (proof_value) finish_value_wave(state, v, final_out, proof_value);
    else if (threadIdx.x == 0) *final_out = v;
    sha_lanes_store(S->st, state);
  }
}

// ---- pipelined tail
// The round sums of round j + 1 are quadratics in the challenge r_j that folds
// level j (the tables after j folds) into level j + 1: for pair b of level
// j + 1 (2Q entries, pairs (b, b + Q)) and point t, each table's value is
// linear in r_j, equal at r_j = 0 and r_j = 1 to entries of level j (4Q
// entries): t = 0: L[b] and L[b + 2Q]; t = 2: 2 L[b + Q] - L[b] and
// 2 L[b + 3Q] - L[b + 2Q]. The term (products of pairs of tables plus the
// additive table) is then a quadratic q(r) fixed by q(0), q(1) and its leading
// coefficient (the product of the slopes); the sums over the pairs give
// e_t(r) = V0 + r (V1 - V0 - C2) + r^2 C2.

// Levels of a tail: at most 2^kTailMaxLog entries per table once evaluated,
// twice that before the pending fold, all in shared memory.
template <class Form>
struct TailLevel {
  Fr t[Form::NT][2u << kTailMaxLog];
};

// One table's value of a coefficient stream: s = 0: p(0), s = 1: p(1), s = 2: the slope.
__device__ __forceinline__ Fr tail_line(const Fr* L, uint32_t b, uint32_t Q, uint32_t s, bool t2) {
  Fr x0 = fr_zero(), x1 = fr_zero();
  if (s != 1) {
    const Fr a = opaque(L[b]);
    x0 = t2 ? fr_sub(fr_double(opaque(L[b + Q])), a) : a;
  }
  if (s != 0) {
    const Fr c = opaque(L[b + 2 * Q]);
    x1 = t2 ? fr_sub(fr_double(opaque(L[b + 3 * Q])), c) : c;
  }
  return s == 0 ? x0 : (s == 1 ? x1 : fr_sub(x1, x0));
}

// Coefficient s (q(0), q(1) or the leading one) summed over Q pairs by one
// wave, lanes 0..31 at t = 0 and lanes 32..63 at t = 2, to part[t][s]. With
// Direct the level needs no fold (the tail's first round when no challenge is
// pending; Q pairs of 2Q entries): q is constant, so s = 0 gives both values.
template <class Form, bool Direct>
__device__ __forceinline__ void tail_stream(const TailLevel<Form>& lv, uint32_t Q, uint32_t s, Fr (*part)[3]) {
  constexpr int NT = Form::NT;
  const uint32_t lane = threadIdx.x & 63;
  const bool t2 = lane >= 32;
  Fr v = fr_zero();
  for (uint32_t b = lane & 31; b < Q; b += 32) {
    Fr p[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      // the additive table has no slope product
      if (s == 2 && k == NT - 1) p[k] = fr_zero();
      else p[k] = tail_line(lv.t[k], b, Q, Direct ? 0 : s, t2);
    }
    if constexpr (NT == 3) v = fr_add(v, fr_add(fr_mul(p[0], p[1]), p[2]));
    else v = fr_add(v, fr_add(fr_mul_add2(p[0], p[1], p[2], p[3]), p[4]));
  }
  if (Q > 1) v = fr_add(v, dpp_fr<0xB1, 0xF>(v));    // quad_perm [1,0,3,2]
  if (Q > 2) v = fr_add(v, dpp_fr<0x4E, 0xF>(v));    // quad_perm [2,3,0,1]
  if (Q > 4) v = fr_add(v, dpp_fr<0x141, 0xF>(v));   // row_half_mirror
  if (Q > 8) v = fr_add(v, dpp_fr<0x140, 0xF>(v));   // row_mirror
  if (Q > 16) v = fr_add(v, dpp_fr<0x142, 0xA>(v));  // row_bcast15 into rows 1 and 3
  if ((lane & 31) == (Q > 16 ? 31 : 0)) {
    part[lane >> 5][s] = v;
    if (Direct) part[lane >> 5][1] = v;
  }
}

// The claim through a round with sums e0, e2 (e1 = claim - e0) and challenge r is
// g(r) = e0 + r X, X = A + r B, B = (e2 - 2 e1 + e0) / 2, A = e1 - e0 - B: X here,
// the second product in the tail's next half round.
__device__ __forceinline__ Fr tail_claim_x(const Fr& claim, const Fr& e0, const Fr& e2, const Fr& r) {
  const Fr e1 = fr_sub(claim, e0);
  const Fr B = fr_half(fr_add(fr_sub(e2, fr_double(e1)), e0));
  const Fr A = fr_sub(fr_sub(e1, e0), B);
  return fr_add(A, fr_mul(r, B));
}

// A round's message (e0, e1 = claim - e0, e2 in canonical form), lane k
// converting and storing element k.
__device__ __forceinline__ void tail_message(const Fr& claim, const Fr& e0, const Fr& e2, uint32_t* msg) {
  const uint32_t lane = threadIdx.x & 63;
  const Fr e1 = fr_sub(claim, e0);
  Fr x = e0;
#pragma unroll
  for (int k = 0; k < 8; ++k) x.v[k] = lane == 1 ? e1.v[k] : (lane == 2 ? e2.v[k] : x.v[k]);
  const Fr c = fr_from_mont(x);
  if (lane < 3) stf(reinterpret_cast<Fr*>(msg), lane, c);
}

// ST_TAIL_A / ST_TAIL_B, pipelined: the same rounds, messages, challenges and
// final values as body_tail, for levels of at most 2^kTailMaxLog entries, with
// the table work off the hash chain. Eight waves (two per SIMD, wave w on SIMD
// w mod 4), two workgroup barriers per round:
//  first half of round j   wave 0: e0, e2 of round j, the coefficient sums at
//                          r_{j-1}, one limb per lane (fr_row.hpp);
//                          wave 1: the claim through round j - 2 (second product);
//                          waves 2-7: level j - 1 folded into level j by r_{j-1};
//  second half             wave 0 hashes (e0, e2) into r_j, wave 4 writes the
//                          hash's schedule; waves 2, 3, 5: round j + 1's
//                          coefficient sums from level j; wave 1: the claim
//                          through round j - 1 (first product); wave 7: round
//                          j - 1's message.
// Round -1 is the grid round whose claim move is pending, if any. Measured with
// cycle stamps: a round of at most 32 pairs takes 8,600 cycles (three tables)
// against 14,300 with the sums evaluated in one lane (5,900 cycles instead of
// 1,900), the claim moved in one half (6,300) and the levels in device memory.
template <class Form>
__device__ __forceinline__ void body_tail_pipe(const Step& st, uint32_t, uint32_t) {
  constexpr int NT = Form::NT;
  __shared__ TailLevel<Form> lv;
  __shared__ Fr part[2][3];                        // coefficient sums (t; V0, V1, C2) of the next round
  __shared__ Fr r_sh[4], e_sh[4][2], claim_sh[4];  // by round mod 4; claim before the round
  __shared__ ShaHelper help;
  const Fr* rpending = P<const Fr*>(st, 2 * NT);
  DevState* S = P<DevState*>(st, 2 * NT + 1);
  Fr* r_out = P<Fr*>(st, 2 * NT + 2);
  uint32_t* msg = P<uint32_t*>(st, 2 * NT + 3);
  Fr* final_out = P<Fr*>(st, 2 * NT + 4);
  uint32_t* proof_value = P<uint32_t*>(st, 2 * NT + 5);
  const uint32_t wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint32_t size = (uint32_t)st.q[0], rounds = st.u[0];
  const bool pending = rpending != nullptr;
  // the folders in the order 2, 3, 5, 6, 7, 4 (wave 4 shares SIMD 0 with wave 0)
  const uint32_t ford = wid == 4 ? 5 : wid - 2 - (wid > 4);
  const uint32_t fw = ford * 64 + lane, nfw = 6 * 64;
  ShaLanes state;  // wave 0
  Fr claim;        // wave 1: the claim before round j - 1, X of its move
  Fr claim_x;
  const bool grid_pend = S->pending != 0;
  if (wid == 0) {
    state = sha_lanes_load(S->st);
    sha_init(sha_buf());
    if (lane == 0) {
      help.ready = 0;
      r_sh[3] = pending ? ldf(rpending, 0) : (grid_pend ? S->pend_r : fr_zero());
    }
  } else if (wid == 1) {
    claim = opaque(S->claim);
    if (lane == 0) {
      claim_sh[3] = claim;
      e_sh[3][0] = S->pend_e0;
      e_sh[3][1] = S->pend_e2;
    }
  }
#pragma unroll
  for (int k = 0; k < NT; ++k)
    for (uint32_t i = threadIdx.x; i < size; i += blockDim.x) lv.t[k][i] = ldf(P<const Fr*>(st, k), i);
  __syncthreads();
  // round 0's coefficients: from the unfolded tables (a pending fold) or directly
  if (rounds > 0) {
    if (pending) {
      if (wid == 2 || wid == 3 || wid == 5)
        tail_stream<Form, false>(lv, size / 4, wid == 2 ? 0 : (wid == 3 ? 1 : 2), part);
    } else if (wid == 2) {
      tail_stream<Form, true>(lv, size / 2, 0, part);
    } else if (wid == 3 && lane < 2) {
      part[lane][2] = fr_zero();
    }
  }
  __syncthreads();
  for (uint32_t j = 0; j < rounds; ++j) {
    const bool fold = pending || j > 0;
    const uint32_t m = 1u << (rounds - j);  // entries of level j
    const uint32_t q = (j + 3) & 3;         // slot of round j - 1
    if (wid == 0) {
      // round j's sums at r_{j-1}: rows 0 and 2 for t = 0, rows 1 and 3 for t = 2
      uint32_t r[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) r[k] = r_sh[q].v[k];
      const uint32_t t = (lane >> 4) & 1, i = lane & 15;
      uint32_t v0 = 0, v1 = 0, c2 = 0;
      if (i < 8) {
        v0 = part[t][0].v[i];
        v1 = part[t][1].v[i];
        c2 = part[t][2].v[i];
      }
      const uint32_t e = row_quadratic(r, v0, v1, c2);
      if (lane < 32 && i < 8) e_sh[j & 3][t].v[i] = e;
    } else if (wid == 1) {
      if (j > 0) {
        // the claim through round j - 2, to the one before round j - 1
        if (j > 1 || grid_pend) {
          const uint32_t q2 = (j + 2) & 3;
          claim = fr_add(opaque(e_sh[q2][0]), fr_mul(opaque(r_sh[q2]), claim_x));
        }
        if (lane == 0) claim_sh[q] = claim;
      }
    } else if (fold) {
      // level j - 1 into level j by r_{j-1}, in place
      const Fr rf = opaque(r_sh[q]);
      const uint32_t lg = rounds - j;
      for (uint32_t t = fw; t < NT * m; t += nfw) {
        Fr* L = lv.t[t >> lg];
        const uint32_t i = t & (m - 1);
        const Fr a0 = opaque(L[i]), a1 = opaque(L[i + m]);
        L[i] = fr_add(a0, fr_mul(rf, fr_sub(a1, a0)));
      }
    }
    __syncthreads();
    const uint32_t next = j + 1 < rounds ? m / 4 : 0;  // pairs of round j + 1
    if (wid == 0) {
      round_hash_wave<true>(state, e_sh[j & 3], &help, 3 * j);
      store_challenge(state, &r_sh[j & 3], r_out + j);
    } else if (wid == 4) {
      sha_help(round_word(e_sh[j & 3]), sha_buf(), &help, 3 * j);
    } else if (wid == 1) {
      if (j > 0 || grid_pend) claim_x = tail_claim_x(claim, opaque(e_sh[q][0]), opaque(e_sh[q][1]), opaque(r_sh[q]));
    } else if (wid == 7) {
      if (j > 0 || grid_pend)
        tail_message(opaque(claim_sh[q]), opaque(e_sh[q][0]), opaque(e_sh[q][1]), j > 0 ? msg + 24 * (j - 1) : S->pend_msg);
    } else if (next && (wid == 2 || wid == 3 || wid == 5)) {
      tail_stream<Form, false>(lv, next, wid == 2 ? 0 : (wid == 3 ? 1 : 2), part);
    }
    __syncthreads();
  }
  // the final fold (by r_{rounds-1}, or by the pending challenge when no round
  // is left), and the claim to the one before round rounds - 1
  const bool any_fold = pending || rounds > 0;
  const uint32_t ql = (rounds + 3) & 3;  // slot of the last round
  Fr v = fr_zero();                      // wave 0, lane k: the final value of table k
  if (wid == 0) {
    if (lane < NT) {
      const Fr* L = lv.t[lane];
      v = opaque(L[0]);
      if (any_fold) v = fr_add(v, fr_mul(opaque(r_sh[ql]), fr_sub(opaque(L[1]), v)));
    }
  } else if (wid == 1 && rounds > 0) {
    if (rounds > 1 || grid_pend) {
      const uint32_t q2 = (rounds + 2) & 3;
      claim = fr_add(opaque(e_sh[q2][0]), fr_mul(opaque(r_sh[q2]), claim_x));
    }
    if (lane == 0) claim_sh[ql] = claim;
  }
  __syncthreads();
  const bool last = rounds > 0 || grid_pend;  // a last round to move the claim through
  if (wid == 0) {
    if (any_fold && lane < NT) {
      Fr* dst = P<Fr*>(st, NT);
#pragma unroll
      for (int k = 1; k < NT; ++k)
        if (lane == (uint32_t)k) dst = P<Fr*>(st, NT + k);
      stf(dst, 0, v);
    }
    const Fr v0 = lane_fr(v, 0);
    if (proof_value) finish_value_wave(state, opaque(v0), final_out, proof_value);
    else if (lane == 0) *final_out = v0;
    sha_lanes_store(S->st, state);
  } else if (wid == 1 && last) {
    const Fr e0 = opaque(e_sh[ql][0]), r = opaque(r_sh[ql]);
    claim = fr_add(e0, fr_mul(r, tail_claim_x(claim, e0, opaque(e_sh[ql][1]), r)));
    if (lane == 0) {
      S->claim = claim;
      S->pending = 0;
    }
  } else if (wid == 7 && last) {
    tail_message(opaque(claim_sh[ql]), opaque(e_sh[ql][0]), opaque(e_sh[ql][1]),
                 rounds > 0 ? msg + 24 * (rounds - 1) : S->pend_msg);
  }
}

// ST_COPY_WEIGHTS: U[c] = Cu[c] EC[c], V[c] = Cv[c] EC[c]; SU, SV their sums
// (one workgroup). p0 Cu, p1 Cv, p2 EC, p3 U, p4 V, p5 S, q0 ncop.
__device__ __forceinline__ void body_copy_weights(const Step& st, uint32_t, uint32_t) {
  const Fr* Cu = P<const Fr*>(st, 0);
  const Fr* Cv = P<const Fr*>(st, 1);
  const Fr* EC = P<const Fr*>(st, 2);
  Fr* U = P<Fr*>(st, 3);
  Fr* V = P<Fr*>(st, 4);
  DevState* S = P<DevState*>(st, 5);
  Fr acc[2] = {fr_zero(), fr_zero()};
  for (uint64_t c = threadIdx.x; c < st.q[0]; c += kBlock) {
    const Fr ec = ldf(EC, c);
    const Fr u = fr_mul(ldf(Cu, c), ec), v = fr_mul(ldf(Cv, c), ec);
    stf(U, c, u);
    stf(V, c, v);
    acc[0] = fr_add(acc[0], u);
    acc[1] = fr_add(acc[1], v);
  }
  block_reduce<2>(acc);
  if (threadIdx.x == 0) {
    S->su = acc[0];
    S->sv = acc[1];
  }
}

// ST_P2_TABLES: phase-2 sub-circuit tables over y, the copy factors kept apart:
//   M[y,c] = U[c] Ma[y] + V[c] Mb[y],  A[y,c] = U[c] Aa[y] + V[c] Ab[y]
//   Ma[y] = sum_{MUL z: y_z=y} aU[z] EL[x_z] (Mb with bV; Aa, Ab over ADD gates)
//   Fa = vx Ma + Aa, Fb = vx Mb + Ab, Ka = vx Aa, Kb = vx Ab, Ks = SU Ka + SV Kb.
// Two adjacent threads per wire, one for the a tables and one for the b tables
// (a product per gate instead of two: 26 us for 2^12 wires with one thread, now 16).
// p0 yrow, p1 yent, p2 aU, p3 bV, p4 EL, p5 S, p6 Fa, p7 Fb, p8 Ka, p9 Kb, p10 Ks, q0 count.
__device__ __forceinline__ void body_p2_tables(const Step& st, uint32_t tile, uint32_t ntiles) {
  const uint32_t* __restrict__ yrow = P<const uint32_t*>(st, 0);
  const uint2* __restrict__ yent = P<const uint2*>(st, 1);
  const Fr* __restrict__ EL = P<const Fr*>(st, 4);
  const DevState* S = P<const DevState*>(st, 5);
  const bool b = threadIdx.x & 1;
  const Fr* __restrict__ weight = b ? P<const Fr*>(st, 3) : P<const Fr*>(st, 2);
  Fr* F = b ? P<Fr*>(st, 7) : P<Fr*>(st, 6);
  Fr* K = b ? P<Fr*>(st, 9) : P<Fr*>(st, 8);
  const Fr vx = opaque(S->vx), su = opaque(b ? S->sv : S->su);
  const uint64_t total = 2 * st.q[0];
  for (uint64_t t = GTID; t < total; t += GSTRIDE) {
    const uint64_t y = t >> 1;
    Fr m = fr_zero(), a = fr_zero();
    const uint32_t k1 = yrow[y + 1];
    for (uint32_t k = yrow[y]; k < k1; ++k) {
      const uint2 ent = yent[k];
      const Fr v = fr_mul(ldf(weight, ent.x), ldf(EL, ent.y & 0x7fffffffu));
      if (ent.y >> 31) m = fr_add(m, v);
      else a = fr_add(a, v);
    }
    const Fr ka = fr_mul(vx, a);
    stf(F, y, fr_add(fr_mul(vx, m), a));
    stf(K, y, ka);
    const Fr part = fr_mul(su, ka);
    const Fr ks = fr_add(part, shfl_xor_fr(part, 1));
    if (!b) stf(P<Fr*>(st, 10), y, ks);
  }
}

// ST_COPY_CONTRACT: row sums over the copies, P[y] = sum_c U[c] W[y,c],
// Q[y] = sum_c V[c] W[y,c]. A row of 2^n entries is handled by tpr = 2^u1 <= 256
// threads: enough of them for about 2^17 in all, but at least 32 (of a row of 32
// entries or more), since a thread's reduction and the sums over the threads
// cost as much as three entries (2^12 rows of 2^8 entries: 45 us with 256
// threads per row, 20 with 32).
// p0 W, p1 U, p2 V, p3 P, p4 Q, u0 n, u1 log2 of tpr, q0 rows.
__device__ __forceinline__ void body_copy_contract(const Step& st, uint32_t tile, uint32_t ntiles) {
  __shared__ Fr sw[2][kBlock / 64];
  const Fr* __restrict__ W = P<const Fr*>(st, 0);
  const Fr* __restrict__ U = P<const Fr*>(st, 1);
  const Fr* __restrict__ V = P<const Fr*>(st, 2);
  const uint32_t n = st.u[0];
  const uint64_t rows = st.q[0];
  const uint32_t tpr_log = st.u[1];
  const uint32_t tpr = 1u << tpr_log;
  const uint32_t lane = threadIdx.x & (tpr - 1);
  const uint64_t rows_per_tile = kBlock >> tpr_log;
  for (uint64_t base = (uint64_t)tile * rows_per_tile; base < rows; base += (uint64_t)ntiles * rows_per_tile) {
    const uint64_t row = base + (threadIdx.x >> tpr_log);
    Fr p = fr_zero(), q = fr_zero();
    if (row < rows) {
      // at most 16 unreduced products per accumulator between reductions
      const uint64_t ncop = 1ull << n;
      for (uint64_t c0 = lane; c0 < ncop; c0 += 16 * (uint64_t)tpr) {
        FrCols pw = frc_zero(), qw = frc_zero();
        const uint64_t c1 = c0 + 16 * (uint64_t)tpr < ncop ? c0 + 16 * (uint64_t)tpr : ncop;
        for (uint64_t c = c0; c < c1; c += tpr) {
          const Fr w = ldf(W, (row << n) | c);
          frc_mac(pw, ldf(U, c), w);
          frc_mac(qw, ldf(V, c), w);
        }
        p = fr_add(p, frw_reduce<16>(frc_wide(pw)));
        q = fr_add(q, frw_reduce<16>(frc_wide(qw)));
      }
    }
    for (uint32_t off = (tpr < 64 ? tpr : 64) / 2; off >= 1; off >>= 1) {
      p = fr_add(p, shfl_xor_fr(p, (int)off));
      q = fr_add(q, shfl_xor_fr(q, (int)off));
    }
    if (tpr > 64) {
      // the row's waves
      const uint32_t wid = threadIdx.x >> 6, nw = tpr / 64;
      __syncthreads();
      if ((threadIdx.x & 63) == 0) {
        sw[0][wid] = p;
        sw[1][wid] = q;
      }
      __syncthreads();
      if (lane == 0)
        for (uint32_t w = 1; w < nw; ++w) {
          p = fr_add(p, opaque(sw[0][wid + w]));
          q = fr_add(q, opaque(sw[1][wid + w]));
        }
    }
    if (lane == 0 && row < rows) {
      stf(P<Fr*>(st, 3), row, p);
      stf(P<Fr*>(st, 4), row, q);
    }
  }
}

// ST_LOCAL_CONTRACT: column sums over the sub-circuit variables, first stage:
// part[c * R + k] = sum_{y in chunk k} EqR[y] W[y,c] for R = u1 chunks of rows.
// Tile t = column block (t % xb) of 2^min(n, 6) columns and chunk (t / xb); the rows
// of a chunk are spread over the threads of a column, whose sums are added in the
// workgroup. (A thread per column left most of a workgroup idle with few copies,
// and left the second stage up to 512 additions in a row.)
// p0 W, p1 EqR, p2 part, u0 n, u1 R, q0 rows.
__device__ __forceinline__ void body_local_contract(const Step& st, uint32_t tile, uint32_t ntiles) {
  const Fr* __restrict__ W = P<const Fr*>(st, 0);
  const Fr* __restrict__ EqR = P<const Fr*>(st, 1);
  Fr* __restrict__ part = P<Fr*>(st, 2);
  const uint32_t n = st.u[0], R = st.u[1];
  const uint32_t clog = n < 6 ? n : 6, cols = 1u << clog, step = kBlock >> clog;
  const uint64_t rows = st.q[0], xb = 1ull << (n - clog), per = (rows + R - 1) / R;
  __shared__ Fr wave_sums[kBlock / 64][64];
  for (uint64_t t = tile; t < xb * R; t += ntiles) {
    const uint64_t c = (t % xb) * cols + (threadIdx.x & (cols - 1)), k = t / xb;
    const uint64_t y0 = k * per, y1 = y0 + per < rows ? y0 + per : rows;
    Fr acc = fr_zero();
    for (uint64_t ya = y0 + (threadIdx.x >> clog); ya < y1; ya += 16ull * step) {
      FrCols aw = frc_zero();
      for (uint64_t y = ya; y < y1 && y < ya + 16ull * step; y += step) frc_mac(aw, ldf(EqR, y), ldf(W, (y << n) | c));
      acc = fr_add(acc, frw_reduce<16>(frc_wide(aw)));
    }
    for (uint32_t off = 32; off >= cols; off >>= 1) acc = fr_add(acc, shfl_xor_fr(acc, off));
    __syncthreads();  // (the previous chunk's sums are read)
    wave_sums[threadIdx.x >> 6][threadIdx.x & 63] = acc;
    __syncthreads();
    if (threadIdx.x < cols) {
#pragma unroll
      for (int w = 1; w < kBlock / 64; ++w) acc = fr_add(acc, wave_sums[w][threadIdx.x]);
      stf(part, c * R + k, acc);
    }
  }
}

// ST_COPY_TABLES: the copy tables of phase 2. A column's R partials are summed
// by tpc = min(64, R) lanes of one wave:
// Wc[c] = sum_k part[c*R + k], Fc[c] = U[c] Fa~ + V[c] Fb~, Kc[c] = U[c] Ka~ + V[c] Kb~.
// p0 part, p1 U, p2 V, p3 fa_f, p4 fb_f, p5 S, p6 Wc, p7 Fc, p8 Kc, u0 R, q0 ncop.
__device__ __forceinline__ void body_copy_tables(const Step& st, uint32_t tile, uint32_t ntiles) {
  const Fr* __restrict__ part = P<const Fr*>(st, 0);
  const uint32_t R = st.u[0];
  const uint64_t ncop = st.q[0];
  // tpc lanes (at most a wave) per column, reduced with shuffles inside aligned lane groups
  const uint32_t rlog = 31 - __clz(R);
  const uint32_t tpc_log = rlog < 6 ? rlog : 6;
  const uint32_t tpc = 1u << tpc_log;
  const uint32_t lane = threadIdx.x & (tpc - 1);
  const uint64_t cols_per_tile = kBlock >> tpc_log;
  const DevState* S = P<const DevState*>(st, 5);
  const Fr fa = opaque(*P<const Fr*>(st, 3)), fb = opaque(*P<const Fr*>(st, 4));
  const Fr ka = opaque(S->ka_f), kb = opaque(S->kb_f);
  for (uint64_t base = (uint64_t)tile * cols_per_tile; base < ncop; base += (uint64_t)ntiles * cols_per_tile) {
    const uint64_t c = base + (threadIdx.x >> tpc_log);
    Fr w = fr_zero();
    if (c < ncop)
      for (uint32_t k = lane; k < R; k += tpc) w = fr_add(w, ldf(part, c * R + k));
    for (uint32_t off = tpc / 2; off >= 1; off >>= 1) w = fr_add(w, shfl_xor_fr(w, off));
    if (lane == 0 && c < ncop) {
      const Fr u = ldf(P<const Fr*>(st, 1), c), v = ldf(P<const Fr*>(st, 2), c);
      stf(P<Fr*>(st, 6), c, w);
      stf(P<Fr*>(st, 7), c, fr_mul_add2(u, fa, v, fb));
      stf(P<Fr*>(st, 8), c, fr_mul_add2(u, ka, v, kb));
    }
  }
}

// ST_LOCAL_VALUES: Ka~, Kb~ at the phase-2 sub-circuit point: dot products with
// EqR (one workgroup). p0 EqR, p1 Ka, p2 Kb, p3 S, q0 rows.
__device__ __forceinline__ void body_local_values(const Step& st, uint32_t tile, uint32_t ntiles) {
  const Fr* EqR = P<const Fr*>(st, 0);
  const Fr* Ka = P<const Fr*>(st, 1);
  const Fr* Kb = P<const Fr*>(st, 2);
  Fr acc[2] = {fr_zero(), fr_zero()};
  // lazy sums: at most 16 unreduced products per column accumulator
  const uint64_t stride = (uint64_t)ntiles * kBlock;
  for (uint64_t y0 = (uint64_t)tile * kBlock + threadIdx.x; y0 < st.q[0]; y0 += 16 * stride) {
    FrCols a = frc_zero(), b = frc_zero();
    const uint64_t y1 = y0 + 16 * stride < st.q[0] ? y0 + 16 * stride : st.q[0];
    for (uint64_t y = y0; y < y1; y += stride) {
      const Fr e = ldf(EqR, y);
      frc_mac(a, e, ldf(Ka, y));
      frc_mac(b, e, ldf(Kb, y));
    }
    acc[0] = fr_add(acc[0], frw_reduce<16>(frc_wide(a)));
    acc[1] = fr_add(acc[1], frw_reduce<16>(frc_wide(b)));
  }
  write_partial<2>(acc, P<Fr*>(st, 4), tile);
}
__device__ __forceinline__ void finish_local_values(const Step& st, uint32_t ntiles) {
  Fr tot[2];
  sum_partials<2>(P<const Fr*>(st, 4), ntiles, tot);
  if (threadIdx.x == 0) {
    DevState* S = P<DevState*>(st, 3);
    S->ka_f = tot[0];
    S->kb_f = tot[1];
  }
}

// ST_STATE_EXPORT / ST_STATE_IMPORT: transcript state bytes <-> device state.
// p0 S, p1 32-byte buffer.
__device__ __forceinline__ void body_state_export(const Step& st, uint32_t, uint32_t) {
  const DevState* S = P<const DevState*>(st, 0);
  uint8_t* out = P<uint8_t*>(st, 1);
  if (threadIdx.x < 8) {
    const uint32_t h = S->st[threadIdx.x];
    out[4 * threadIdx.x + 0] = (uint8_t)(h >> 24);
    out[4 * threadIdx.x + 1] = (uint8_t)(h >> 16);
    out[4 * threadIdx.x + 2] = (uint8_t)(h >> 8);
    out[4 * threadIdx.x + 3] = (uint8_t)h;
  }
}
__device__ __forceinline__ void body_state_import(const Step& st, uint32_t, uint32_t) {
  DevState* S = P<DevState*>(st, 0);
  const uint8_t* in = P<const uint8_t*>(st, 1);
  if (threadIdx.x < 8) {
    const uint8_t* b = in + 4 * threadIdx.x;
    S->st[threadIdx.x] = ((uint32_t)b[0] << 24) | ((uint32_t)b[1] << 16) | ((uint32_t)b[2] << 8) | b[3];
  }
  if (threadIdx.x == 0) {
    S->counter = 0;
    S->pending = 0;
  }
}

#undef GTID
#undef GSTRIDE

// Runs tile `tile` of a step; for reduction steps the last tile (by the
// counter in the proof's state) also runs the finisher. Used by the batch kernel.
__device__ __forceinline__ void run_step_tile(const Step& st, uint32_t tile, uint32_t ntiles) {
  uint32_t* counter = nullptr;
  switch (st.type) {
    case ST_WSUM: counter = &P<DevState*>(st, 4)->counter; break;
    case ST_P1_INIT_ROUND: counter = &P<DevState*>(st, 9)->counter; break;
    case ST_ROUND_A: counter = &P<DevState*>(st, RoundPtrs<3>::kS)->counter; break;
    case ST_ROUND_B: counter = &P<DevState*>(st, RoundPtrs<5>::kS)->counter; break;
    case ST_LOCAL_VALUES: counter = &P<DevState*>(st, 3)->counter; break;
    default: break;
  }
  switch (st.type) {
    case ST_TO_MONT: body_to_mont(st, tile, ntiles); break;
    case ST_FROM_MONT: body_from_mont(st, tile, ntiles); break;
    case ST_FORWARD: body_forward(st, tile, ntiles); break;
    case ST_DIGEST: body_digest(st, tile, ntiles); break;
    case ST_DIGEST_WAVE: body_digest_wave(st, tile, ntiles); break;
    case ST_TRANSCRIPT_BEGIN: body_transcript_begin(st, tile, ntiles); break;
    case ST_SQUEEZE: body_squeeze(st, tile, ntiles); break;
    case ST_LAYER_BEGIN: body_layer_begin(st, tile, ntiles); break;
    case ST_EQ: body_eq(st, tile, ntiles); break;
    case ST_WSUM:
      body_wsum(st, tile, ntiles);
      if (last_tile(counter, ntiles)) finish_wsum(st, ntiles);
      break;
    case ST_P1_INIT: body_p1_init(st, tile, ntiles); break;
    case ST_P1_INIT_ROUND:
      body_p1_init_round<false>(st, tile, ntiles);
      if (last_tile(counter, ntiles)) finish_p1_init_round<true>(st, ntiles);
      break;
    case ST_ROUND_A:
      body_round<FormA>(st, tile, ntiles);
      if (last_tile(counter, ntiles)) finish_round_step<FormA, true>(st, ntiles);
      break;
    case ST_ROUND_B:
      body_round<FormB>(st, tile, ntiles);
      if (last_tile(counter, ntiles)) finish_round_step<FormB, true>(st, ntiles);
      break;
    case ST_TAIL_A: body_tail<FormA>(st, tile, ntiles); break;
    case ST_TAIL_B: body_tail<FormB>(st, tile, ntiles); break;
    case ST_COPY_WEIGHTS: body_copy_weights(st, tile, ntiles); break;
    case ST_P2_TABLES: body_p2_tables(st, tile, ntiles); break;
    case ST_COPY_CONTRACT: body_copy_contract(st, tile, ntiles); break;
    case ST_LOCAL_CONTRACT: body_local_contract(st, tile, ntiles); break;
    case ST_COPY_TABLES: body_copy_tables(st, tile, ntiles); break;
    case ST_LOCAL_VALUES:
      body_local_values(st, tile, ntiles);
      if (last_tile(counter, ntiles)) finish_local_values(st, ntiles);
      break;
    case ST_STATE_EXPORT: body_state_export(st, tile, ntiles); break;
    case ST_STATE_IMPORT: body_state_import(st, tile, ntiles); break;
    default: break;
  }
}

}  // namespace gkr
