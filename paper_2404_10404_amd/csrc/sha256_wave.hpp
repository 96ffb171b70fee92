// One SHA-256 compression spread over the lanes of a wave (device code): the
// transcript's chain of hashes is serial, and a wave alone on its SIMD issues
// one instruction per 5 cycles (a dependent one per 8.5), so the compression's
// time is its instruction count. Written out per lane, a round takes 14
// instructions and a schedule word 10: 5,900 cycles per compression. Here:
//
//  - Rounds. Lanes with (lane & 8) == 0 hold e, f, g, h and the others a, b,
//    c, d, so one instruction sequence computes S1(e) + Ch(e,f,g) + .. and
//    S0(a) + Maj(a,b,c) + .. (rotation counts per lane; Maj(a,b,c) is
//    "a == b ? b : c", a choice like Ch). The a-lanes run two rounds behind
//    the e-lanes: e' = d + h + k + w + S1 + Ch needs d = a of three rounds
//    before, a' = e' - d + S0 + Maj needs the new e; with the lag of two both
//    operands sit in the other lane group's second register, one DPP add for
//    both. Nine instructions per round, 66 steps: 3,140 cycles measured with
//    the schedule given.
//  - Schedule. Lane i of a row of 16 holds word i; the next 16 words are
//    c + s1(lane - 2) + (lane - 7) iterated seven times (words 2i, 2i + 1 come
//    right at iteration i), 75 instructions per 16 words instead of 160. In
//    the same wave the whole compression takes 4,250 cycles; a second wave
//    that writes the schedule to shared memory while the first runs the
//    rounds takes its part off the chain.
#pragma once

#include "gkr_device.hpp"
#include "sha256.hpp"

namespace gkr {

// The chaining value: x[k] is h[4 + k] in lanes with (lane & 8) == 0, h[k] in the others.
struct ShaLanes {
  uint32_t x[4];
};

// Shared words of one wave's compressions (16-byte aligned).
struct ShaBuf {
  uint32_t wk[64];   // schedule words plus round constants
  uint32_t one[16];  // the a-lanes' constant term
  uint32_t msg[32];  // message words (big-endian values)
  uint32_t k[64];    // round constants
};

// Fills the constant parts (one wave, before its own use or a barrier).
__device__ __forceinline__ void sha_init(ShaBuf* buf) {
  const uint32_t lane = threadIdx.x & 63;
  buf->k[lane] = kSha256K[lane];
  if (lane < 16) buf->one[lane] = 1;
}

// A word in a register of its own: selections between two words of a struct
// go through it, or the compiler may select their addresses instead and put
// the struct in memory.
__device__ __forceinline__ uint32_t sha_reg(uint32_t x) {
  asm("" : "+v"(x));
  return x;
}
__device__ __forceinline__ uint32_t sha_sel(bool c, uint32_t a, uint32_t b) {
  a = sha_reg(a);
  b = sha_reg(b);
  return c ? a : b;
}

// The lane number, computed anew at each use: what follows from it (rotation
// counts, addresses) is not kept in registers through the code between hashes.
__device__ __forceinline__ uint32_t sha_lane() {
  uint32_t l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  return l;
}

// A DPP row shift of one word (lanes without a source read zero).
template <int Ctrl>
__device__ __forceinline__ uint32_t sha_dpp(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, Ctrl, 0xF, 0xF, true);
}

__device__ __forceinline__ uint32_t sha_s0(uint32_t y) { return xor3_32(rotr32(y, 7), rotr32(y, 18), y >> 3); }
__device__ __forceinline__ uint32_t sha_s1(uint32_t y) { return xor3_32(rotr32(y, 17), rotr32(y, 19), y >> 10); }

// Schedule words 16 g + 16 .. 16 g + 31 from 16 g .. 16 g + 15, word i in lane i mod 16.
__device__ __forceinline__ uint32_t sha_schedule(uint32_t w) {
  uint32_t c = w + sha_s0(sha_dpp<0x101>(w));  // row_shl:1 (lane 15 waits for the new word 0)
  c += sha_dpp<0x109>(w);                      // row_shl:9, words 9..15 for lanes 0..6
  c += sha_s1(sha_dpp<0x10E>(w));              // row_shl:14, words 14, 15 for lanes 0, 1
  c += sha_s0(sha_dpp<0x11F>(c));              // row_shr:15, the new word 0 for lane 15
  uint32_t v = c;
#pragma unroll
  for (int i = 0; i < 7; ++i) v = c + sha_dpp<0x117>(v) + sha_s1(sha_dpp<0x112>(v));  // row_shr:7, row_shr:2
  return v;
}

// One step of both lane groups: the new value replaces X3 (the roles then
// rotate). X1 was written a step ago at least, so its DPP read needs no wait.
#define GKR_SHA_STEP(X0, X1, X2, X3, WK)                                                \
  asm volatile(                                                                         \
      "v_xad_u32 %[q], %[x3], %[m], %[wk]\n\t"                                          \
      "v_bitop3_b32 %[mk], %[x0], %[x1], %[m] bitop3:0xd2\n\t"                          \
      "v_add_u32_dpp %[q], %[x1], %[q] row_ror:8 row_mask:0xf bank_mask:0xf\n\t"        \
      "v_alignbit_b32 %[t1], %[x0], %[x0], %[s1]\n\t"                                   \
      "v_alignbit_b32 %[t2], %[x0], %[x0], %[s2]\n\t"                                   \
      "v_alignbit_b32 %[t3], %[x0], %[x0], %[s3]\n\t"                                   \
      "v_bitop3_b32 %[mk], %[mk], %[x1], %[x2] bitop3:0xca\n\t"                         \
      "v_bitop3_b32 %[t1], %[t1], %[t2], %[t3] bitop3:0x96\n\t"                         \
      "v_add3_u32 %[x3], %[t1], %[mk], %[q]"                                            \
      : [x3] "+v"(X3), [q] "=&v"(q), [mk] "=&v"(mk), [t1] "=&v"(t1), [t2] "=&v"(t2),    \
        [t3] "=&v"(t3)                                                                  \
      : [x0] "v"(X0), [x1] "v"(X1), [x2] "v"(X2), [m] "v"(m), [wk] "v"(WK),             \
        [s1] "v"(s1), [s2] "v"(s2), [s3] "v"(s3))

__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }

// The waves' agreement on a schedule written by another wave: ready counts the
// 16-word groups written since the kernel began (groups 1..3 of each message).
struct ShaHelper {
  uint32_t ready;
};
// The count as a shared-memory (not flat) access: it keeps its order with the
// words' own shared-memory accesses.
typedef __attribute__((address_space(3))) volatile uint32_t LdsWord;

// The compression of the block whose word i is in lane i mod 16 of w, by the
// calling wave (64 active lanes). With Helped, groups 1..3 of the schedule
// come from another wave (sha_help), which counts them in help->ready from
// `base`; else this wave computes them.
template <bool Helped>
__device__ __forceinline__ ShaLanes sha_compress_wave(const ShaLanes& st, uint32_t w, ShaBuf* buf,
                                                      ShaHelper* help = nullptr, uint32_t base = 0) {
  const uint32_t lane = sha_lane();
  const bool at = (lane & 8) != 0;
  uint32_t q, mk, t1, t2, t3;
  // the a-lanes begin two steps early at (c, d) and take b, a in the first two steps
  uint32_t x0 = sha_sel(at, st.x[2], st.x[0]), x1 = sha_sel(at, st.x[3], st.x[1]), x2 = st.x[2], x3 = st.x[3];
  const uint32_t s1 = at ? 2 : 6, s2 = at ? 13 : 11, s3 = at ? 22 : 25, m = at ? ~0u : 0u;
  lds_order();
  if (lane < 16) buf->wk[lane] = w + buf->k[lane];
  lds_order();
  const U32x4* rd = reinterpret_cast<const U32x4*>(at ? buf->one : buf->wk);
  const uint32_t step = at ? 0 : 4;  // vectors per group
  U32x4 k0 = rd[0], k1 = rd[1], k2 = rd[2], k3 = rd[3];
  for (int g = 0; g < 4; ++g) {
    if (!Helped && g < 3) {
      w = sha_schedule(w);
      lds_order();
      if (lane < 16) buf->wk[16 * (g + 1) + lane] = w + buf->k[16 * (g + 1) + lane];
      lds_order();
    }
    const bool first = g == 0;
    GKR_SHA_STEP(x0, x1, x2, x3, k0.x);
    x3 = sha_sel(first && at, st.x[1], x3);
    GKR_SHA_STEP(x3, x0, x1, x2, k0.y);
    x2 = sha_sel(first && at, st.x[0], x2);
    GKR_SHA_STEP(x2, x3, x0, x1, k0.z);
    GKR_SHA_STEP(x1, x2, x3, x0, k0.w);
    GKR_SHA_STEP(x0, x1, x2, x3, k1.x);
    GKR_SHA_STEP(x3, x0, x1, x2, k1.y);
    GKR_SHA_STEP(x2, x3, x0, x1, k1.z);
    GKR_SHA_STEP(x1, x2, x3, x0, k1.w);
    GKR_SHA_STEP(x0, x1, x2, x3, k2.x);
    GKR_SHA_STEP(x3, x0, x1, x2, k2.y);
    GKR_SHA_STEP(x2, x3, x0, x1, k2.z);
    GKR_SHA_STEP(x1, x2, x3, x0, k2.w);
    GKR_SHA_STEP(x0, x1, x2, x3, k3.x);
    GKR_SHA_STEP(x3, x0, x1, x2, k3.y);
    GKR_SHA_STEP(x2, x3, x0, x1, k3.z);
    GKR_SHA_STEP(x1, x2, x3, x0, k3.w);
    if (g < 3) {
      if (Helped) {
        // the helper always writes its three groups, so this wait ends
        while ((int32_t)(*(LdsWord*)&help->ready - (base + g + 1)) < 0) {}
      }
      lds_order();
      rd += step;
      k0 = rd[0];
      k1 = rd[1];
      k2 = rd[2];
      k3 = rd[3];
    }
  }
  const uint32_t y2 = x2, y3 = x3;  // the e-lanes' last values
  const uint32_t one = 1;
  GKR_SHA_STEP(x0, x1, x2, x3, one);
  GKR_SHA_STEP(x3, x0, x1, x2, one);
  ShaLanes r;
  r.x[0] = st.x[0] + (at ? x2 : x0);
  r.x[1] = st.x[1] + (at ? x3 : x1);
  r.x[2] = st.x[2] + (at ? x0 : y2);
  r.x[3] = st.x[3] + (at ? x1 : y3);
  return r;
}
// The compression with its whole schedule (plus round constants) given in
// wk[0, 64), 16-byte aligned shared memory; one[0, 4) are ones.
__device__ __forceinline__ ShaLanes sha_compress_given(const ShaLanes& st, const uint32_t* wk, const uint32_t* one4) {
  const bool at = (sha_lane() & 8) != 0;
  uint32_t q, mk, t1, t2, t3;
  uint32_t x0 = sha_sel(at, st.x[2], st.x[0]), x1 = sha_sel(at, st.x[3], st.x[1]), x2 = st.x[2], x3 = st.x[3];
  const uint32_t s1 = at ? 2 : 6, s2 = at ? 13 : 11, s3 = at ? 22 : 25, m = at ? ~0u : 0u;
  const U32x4* rd = reinterpret_cast<const U32x4*>(at ? one4 : wk);
  const uint32_t step = at ? 0 : 1;
  U32x4 k0 = rd[0], k1 = rd[step];
  for (int g = 0; g < 16; g += 2) {
    const bool first = g == 0;
    GKR_SHA_STEP(x0, x1, x2, x3, k0.x);
    x3 = sha_sel(first && at, st.x[1], x3);
    GKR_SHA_STEP(x3, x0, x1, x2, k0.y);
    x2 = sha_sel(first && at, st.x[0], x2);
    GKR_SHA_STEP(x2, x3, x0, x1, k0.z);
    GKR_SHA_STEP(x1, x2, x3, x0, k0.w);
    rd += 2 * step;
    if (g < 14) k0 = rd[0];
    GKR_SHA_STEP(x0, x1, x2, x3, k1.x);
    GKR_SHA_STEP(x3, x0, x1, x2, k1.y);
    GKR_SHA_STEP(x2, x3, x0, x1, k1.z);
    GKR_SHA_STEP(x1, x2, x3, x0, k1.w);
    if (g < 14) k1 = rd[step];
  }
  const uint32_t y2 = x2, y3 = x3;
  const uint32_t one = 1;
  GKR_SHA_STEP(x0, x1, x2, x3, one);
  GKR_SHA_STEP(x3, x0, x1, x2, one);
  ShaLanes r;
  r.x[0] = st.x[0] + (at ? x2 : x0);
  r.x[1] = st.x[1] + (at ? x3 : x1);
  r.x[2] = st.x[2] + (at ? x0 : y2);
  r.x[3] = st.x[3] + (at ? x1 : y3);
  return r;
}
#undef GKR_SHA_STEP

// The helper's part (another wave of the workgroup): groups 1..3 of the
// schedule of the block in w, counted in help->ready up to base + 3.
__device__ __forceinline__ void sha_help(uint32_t w, ShaBuf* buf, ShaHelper* help,
                                         uint32_t base) {
  const uint32_t lane = sha_lane();
#pragma unroll
  for (int g = 1; g < 4; ++g) {
    w = sha_schedule(w);
    if (lane < 16) buf->wk[16 * g + lane] = w + buf->k[16 * g + lane];
    // one wave's shared-memory operations stay in order: the count follows the words
    lds_order();
    if (lane == 0) *(LdsWord*)&help->ready = base + g;
    lds_order();
  }
}

__device__ __forceinline__ ShaLanes sha_lanes_iv() {
  const Sha256State v = sha256_iv();
  const bool at = (sha_lane() & 8) != 0;
  ShaLanes s;
#pragma unroll
  for (int k = 0; k < 4; ++k) s.x[k] = sha_sel(at, v.h[k], v.h[4 + k]);
  return s;
}

// The chaining value from / to eight words in memory (global or shared).
__device__ __forceinline__ ShaLanes sha_lanes_load(const uint32_t* h) {
  const uint32_t o = (sha_lane() & 8) ? 0 : 4;
  ShaLanes s;
#pragma unroll
  for (int k = 0; k < 4; ++k) s.x[k] = h[o + k];
  return s;
}
__device__ __forceinline__ void sha_lanes_store(uint32_t* h, const ShaLanes& s) {
  const uint32_t lane = sha_lane();
  if (lane == 0 || lane == 8) {
    const uint32_t o = lane ? 0 : 4;
#pragma unroll
    for (int k = 0; k < 4; ++k) h[o + k] = s.x[k];
  }
}

// The candidate of the chaining value (little-endian digest bytes, 254 bits):
// this lane's four limbs, limbs 4..7 in lanes with (lane & 8) == 0, else 0..3.
__device__ __forceinline__ void sha_candidate_limbs(const ShaLanes& s, uint32_t (&v)[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = bswap32(s.x[k]);
  if (!(sha_lane() & 8)) v[3] &= 0x3fffffffu;
}

__device__ __forceinline__ Fr sha_candidate(const ShaLanes& s) {
  uint32_t v[4];
  sha_candidate_limbs(s, v);
  Fr r;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    r.v[k] = (uint32_t)__builtin_amdgcn_readlane((int)v[k], 8);
    r.v[4 + k] = (uint32_t)__builtin_amdgcn_readlane((int)v[k], 0);
  }
  return r;
}

// Whether the candidate is below p (the top limb decides but for one value in 2^30).
__device__ __forceinline__ bool sha_candidate_canonical(const ShaLanes& s) {
  const uint32_t top = bswap32((uint32_t)__builtin_amdgcn_readlane((int)s.x[3], 0)) & 0x3fffffffu;
  if (top != GKR_P7) return top < GKR_P7;
  return fr_is_canonical(sha_candidate(s));
}

// SHA-256 of the L-word message in buf->msg[0, L) (L <= 29), words beyond L
// of its blocks are padding, by the calling wave.
template <int L>
__device__ __forceinline__ ShaLanes sha_message_wave(ShaBuf* buf) {
  constexpr int B = (L + 3 + 15) / 16;
  const uint32_t li = sha_lane() & 15;
  lds_order();
  ShaLanes st = sha_lanes_iv();
  for (uint32_t b = 0; b < B; ++b) {
    const uint32_t i = 16 * b + li;
    const uint32_t v = buf->msg[i];
    const uint32_t w = i < L ? v : (i == L ? 0x80000000u : (i == 16 * B - 1 ? (uint32_t)(L * 32) : 0u));
    st = sha_compress_wave<false>(st, w, buf);
  }
  return st;
}

// state = SHA-256(state || "GKRC").
__device__ __forceinline__ void sha_rehash_wave(ShaLanes& st, ShaBuf* buf) {
  sha_lanes_store(buf->msg, st);
  if (sha_lane() == 1) buf->msg[8] = kTagChallenge;
  st = sha_message_wave<9>(buf);
}

// The state rehashed until it is a challenge (the candidate rule in gkr_bodies.hpp).
__device__ __forceinline__ void sha_accept_wave(ShaLanes& st, ShaBuf* buf) {
  for (int attempt = 0; attempt < 4096 && !sha_candidate_canonical(st); ++attempt) sha_rehash_wave(st, buf);
}

// A squeezed challenge, in every lane.
__device__ __forceinline__ Fr sha_squeeze_wave(ShaLanes& st, ShaBuf* buf) {
  sha_rehash_wave(st, buf);
  sha_accept_wave(st, buf);
  return sha_candidate(st);
}

// state = SHA-256(state || tag || eight words), the words from lanes 0..7.
__device__ __forceinline__ void sha_absorb_words_wave(ShaLanes& st, ShaBuf* buf, uint32_t tag,
                                                      uint32_t word) {
  const uint32_t lane = sha_lane();
  sha_lanes_store(buf->msg, st);
  if (lane == 1) buf->msg[8] = tag;
  if (lane < 8) buf->msg[9 + lane] = word;
  st = sha_message_wave<17>(buf);
}

// Limb k of a value that is the same in every lane, k = lane (lanes 0..7).
__device__ __forceinline__ uint32_t lane_limb(const Fr& a) {
  const uint32_t lane = sha_lane() & 7;
  uint32_t r = a.v[0];
#pragma unroll
  for (int k = 1; k < 8; ++k) r = sha_sel(lane == (uint32_t)k, a.v[k], r);
  return r;
}

}  // namespace gkr
