// Rounds over tables too small to fill the chip, one product per thread
// (gkr_wide.hip; the lockstep kernel of a batch runs the same bodies).
#pragma once

#include "gkr_internal.hpp"

namespace gkr {

// Largest number of pairs (log2) of a round that takes this form.
constexpr uint32_t kWideMaxLogHalf = 13;
constexpr uint32_t kWidePairs = 32;  // pairs per workgroup

void launch_wide_step(const Step& st, hipStream_t s);

}  // namespace gkr
