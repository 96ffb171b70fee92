// Field arithmetic with one limb per lane (device code), for the few products
// that sit on a chain of latencies: a Montgomery product in one lane is 272
// dependent multiply-add and carry instructions and takes 2,200 cycles in a
// wave that runs alone; with a limb per lane (each 16-lane row of the wave a
// product of its own, lanes 0..7 its limbs) a step of the product is one
// multiply-add for a_j b, one for m p and two lane moves: 800 cycles with the
// carries. Carries are resolved by carry lookahead on the wave's masks: with
// generate bits G and propagate bits P, the lanes that receive a carry are
// (P + 2 G) xor P.
#pragma once

#include "gkr_device.hpp"

namespace gkr {

// p's limb of this lane (0 in lanes 8..15 of a row).
__device__ __forceinline__ uint32_t row_p() {
  const uint32_t i = threadIdx.x & 15;
  uint32_t r = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) r = i == (uint32_t)k ? p_limb(k) : r;
  return r;
}

template <int Ctrl>
__device__ __forceinline__ uint32_t row_dpp(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, Ctrl, 0xF, 0xF, true);
}

// a b R^-1 mod p, below 2 p for a < p and b < 2^256, as limb sums below 2^34.
// a: the eight limbs in every lane of the row; b: this lane's limb (0 in lanes 8..15).
__device__ __forceinline__ uint64_t row_mul(const uint32_t (&a)[8], uint32_t b, uint32_t p) {
  uint32_t x = 0;
  uint64_t y = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint64_t u = (uint64_t)a[j] * b + x;
    const uint64_t z = (uint64_t)(uint32_t)u + y;  // y < 2^33
    const uint32_t m = row_dpp<0x150>((uint32_t)z) * GKR_NINV;  // row_newbcast:0
    const uint64_t v = (uint64_t)m * p + z;  // p's limbs are below 2^32 - 2^27: no overflow
    y = (u >> 32) + (v >> 32);
    x = row_dpp<0x101>((uint32_t)v);  // row_shl:1: lane 0's low word is zero and drops out
  }
  return y + x;
}

// The lanes that receive a carry, from the lanes that generate and propagate one.
__device__ __forceinline__ uint64_t row_carries(uint64_t gen, uint64_t prop) { return (prop + (gen << 1)) ^ prop; }

// Limb sums (carries into the next limb below 2^31, total below 2^256) as 32-bit limbs.
__device__ __forceinline__ uint32_t row_normalise(uint64_t s) {
  const uint32_t lo = (uint32_t)s, t = lo + row_dpp<0x111>((uint32_t)(s >> 32));  // row_shr:1
  const uint64_t c = row_carries(__ballot(t < lo), __ballot(t == ~0u));
  return t + (uint32_t)((c >> (threadIdx.x & 63)) & 1);
}

// t - p where t >= p, else t (t < 2^256, 32-bit limbs).
__device__ __forceinline__ uint32_t row_sub_p(uint32_t t, uint32_t p) {
  constexpr uint64_t kLimbs = 0x00ff00ff00ff00ffull;
  const uint64_t bor = row_carries(__ballot(t < p) & kLimbs, __ballot(t == p) & kLimbs);
  const uint64_t fits = ~bor & 0x0100010001000100ull;  // rows without a borrow out of limb 7
  const uint64_t rows = (fits << 8) - (fits >> 8);
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t d = t - p - (uint32_t)((bor >> lane) & 1);
  return (rows >> lane) & 1 ? d : t;
}

// The quadratic with values v0 at 0, v1 at 1 and leading coefficient c2, at r:
// v0 + r (v1 - v0 - c2 + r c2), reduced. This lane's limbs of v0, v1, c2 (all
// below p); r's limbs in every lane.
__device__ __forceinline__ uint32_t row_quadratic(const uint32_t (&r)[8], uint32_t v0, uint32_t v1, uint32_t c2) {
  const uint32_t i = threadIdx.x & 15, p = row_p();
  // v1 - v0 - c2 + 2 p, limb by limb: each limb but the top one borrows 4 from
  // the next, so it stays positive
  const int64_t two_p = 2 * (int64_t)p;
  const int64_t bias = i >= 8 ? 0 : (i < 7 ? (1ll << 34) : 0) - (i > 0 ? 4 : 0);
  const int64_t d = two_p + bias + (int64_t)v1 - (int64_t)v0 - (int64_t)c2;
  const uint32_t b = row_normalise(row_mul(r, c2, p) + (uint64_t)d);  // below 5 p < 2^256
  const uint32_t bb = i < 8 ? b : 0;
  const uint32_t e = row_normalise(row_mul(r, bb, p) + v0);  // below 3 p
  return row_sub_p(row_sub_p(e, p), p);
}

}  // namespace gkr
