// Device helpers shared by the fold's kernels (k_fold.hip, k_fold_ks.hip).
#pragma once
#include <type_traits>

#include "hfe_ntt_reg.h"

namespace hfe {
// f(std::bool_constant<z below 2^24>{}); f holds the rest of the kernel (a polynomial in registers that leaves two
// branches and goes on is spilled where they meet)
template <class F>
__device__ __forceinline__ void by_size(double zd, F f) {
  if (zd < 16777216.0)
    f(std::bool_constant<true>{});
  else
    f(std::bool_constant<false>{});
}

// The centered representative (exact: residues r > z / 2 become r - z) of a centered value of the transforms,
// whose magnitude may exceed z / 2 by the rounding of its quotient.
__device__ __forceinline__ double center_exact(double x, double zd) {
  const double r = residue_of_c(x, zd);
  return 2.0 * r > zd ? r - zd : r;
}

}  // namespace hfe
