// Host check of the arithmetic that ends a matrix-core contraction: reads 2^508 mod
// p (8 limbs), then lines of 63 band sums, and prints the reduced value of each line
// as 64 hex digits. With an argument: prints the limbs of kCcPow508.
#include <cinttypes>
#include <cstdio>

#include "../../paper_2404_10404_amd/csrc/cc_sum.hpp"

using namespace gkr;

int main(int argc, char**) {
  if (argc > 1) {
    for (uint32_t x : kCcPow508) printf("%" PRIu32 "\n", x);
    return 0;
  }
  uint32_t w[8];
  for (int i = 0; i < 8; ++i)
    if (scanf("%" SCNu32, &w[i]) != 1) return 1;
  for (;;) {
    CcSum s = cc_sum_zero();
    for (int k = 0; k < kCcBands; ++k) {
      uint64_t e;
      if (scanf("%" SCNu64, &e) != 1) return k ? 1 : 0;
      cc_sum_band(s, k, e);
    }
    const Fr r = cc_sum_reduce(s, w);
    for (int k = 7; k >= 0; --k) printf("%08x", r.v[k]);
    printf("\n");
  }
}
