// The integer arithmetic that ends a contraction on the matrix cores
// (gkr_contract.hip), for the device and for the host check of its bounds.
//
// A sum over 2^t terms is S = sum_k 2^(8k) E_k for k < 63, where E_k adds the
// products of at most 32 byte pairs per term: E_k <= 32 * 255^2 * 2^t < 2^(21 + t),
// and S < 2^(508 + t) for reduced operands. A layer has at most 2^30 entries and a
// contraction at least 2^8 rows, so t <= 22; the arithmetic holds up to t = 24.
#pragma once

#include "fr.hpp"

namespace gkr {

constexpr int kCcBands = 63;

// 2^508 mod p (plain form).
constexpr uint32_t kCcPow508[8] = {0x91e216dbu, 0xe7eaa887u, 0xe2ae14efu, 0xbbdd1653u,
                                   0x7e1479bcu, 0xd071bf6au, 0xb6a0ce61u, 0x1b59d92bu};

// acc[i] collects 32-bit words of weight 2^(32 i).
struct CcSum {
  uint64_t acc[18];
};

GKR_HD CcSum cc_sum_zero() {
  CcSum s;
#pragma unroll
  for (int i = 0; i < 18; ++i) s.acc[i] = 0;
  return s;
}

// S += 2^(8k) e, e < 2^45: the halves of e apart, as e << 24 can need 69 bits. A
// word receives four low halves, four carries and four high halves: below 2^40.
GKR_HD void cc_sum_band(CcSum& s, int k, uint64_t e) {
  const int sh = 8 * (k & 3);
  const uint64_t lo = (uint64_t)(uint32_t)e << sh, hi = (e >> 32) << sh;
  s.acc[k >> 2] += (uint32_t)lo;
  s.acc[(k >> 2) + 1] += (lo >> 32) + hi;
}

// S R^-1 mod p. The bits from 508 on, H < 2^(t + 4), are folded with 2^508 mod p
// (w508, plain form), which leaves less than 2^508 + 2^282 < 2 p^2.
GKR_HD Fr cc_sum_reduce(const CcSum& s, const uint32_t* w508) {
  uint32_t lim[17];
  uint64_t carry = 0;
#pragma unroll
  for (int i = 0; i < 17; ++i) {
    const uint64_t v = s.acc[i] + carry;
    lim[i] = (uint32_t)v;
    carry = v >> 32;
  }
  // S = H 2^508 + L  ==  L + H (2^508 mod p)
  const uint32_t H = (lim[15] >> 28) | (lim[16] << 4);
  lim[15] &= 0x0fffffffu;
  FrWide T;
  uint64_t c = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint64_t v = (uint64_t)lim[i] + (i < 8 ? (uint64_t)H * w508[i] : 0) + c;
    T.w[i] = (uint32_t)v;
    c = v >> 32;
  }
  return frw_reduce<4>(T);
}

}  // namespace gkr
