// Division by a number whose reciprocal the host has worked out (score_pass.h).  Integers and one float product, so that the
// same function runs on the host.
#pragma once
#include <hip/hip_runtime.h>

namespace codecomp {

// x / d for 0 <= x < 2^30, a quotient below 2^17 and inv = 1 / d in float: three roundings move the product by at most
// 2^17 * 3 * 2^-24 = 0.03, so its whole part is at most one off.  (The divisions that the compiler makes are 25 dependent scalar
// instructions each; seven of them stood before the first load of a pass's workgroup.)
__host__ __device__ __forceinline__ int divide(int x, int d, float inv) {
  const int q = (int)((float)x * inv), r = x - q * d;
  return r >= d ? q + 1 : r < 0 ? q - 1 : q;
}

}  // namespace codecomp
