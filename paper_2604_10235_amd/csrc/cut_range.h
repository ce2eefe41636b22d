// Range arithmetic of the counting rounds that look for the score of the last admitted token (select.hip).  Integers only,
// so that the same functions run on the host.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace codecomp {

constexpr int kCutBins = 2048;      // bins of one counting round

// Bins of 2^shift keys cut the range [lo, lo + width] into at most kCutBins.
__host__ __device__ inline int cut_shift(uint32_t width) { return width < (uint32_t)kCutBins ? 0 : 21 - __builtin_clz(width); }

// [lo, hi] becomes its bin `bin` (which holds a key, so it begins at hi or below).  The last bin may reach past hi, and next to
// the largest key past 2^32 too: its end is taken as a distance from lo, which cannot wrap.
__host__ __device__ inline void cut_narrow(uint32_t& lo, uint32_t& hi, uint32_t bin, int shift) {
  lo += bin << shift;
  const uint32_t width = hi - lo, last = (1u << shift) - 1u;
  hi = lo + (width < last ? width : last);
}

}  // namespace codecomp
