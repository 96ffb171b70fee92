// Rounds over tables too small to fill the chip, one product per thread
// (gkr_wide.hip; plain path only).
#pragma once

#include "gkr_internal.hpp"

namespace gkr {

// Largest number of pairs of a round that takes this form (three and five tables).
constexpr uint64_t kWideMaxHalfA = 1u << 13, kWideMaxHalfB = 1u << 13;
constexpr uint32_t kWidePairs = 32;  // pairs per workgroup

void launch_wide_step(const Step& st, hipStream_t s);

}  // namespace gkr
