// The fourth-order nuclear-matter sample kernel with every diagram's masks
// as compile-time constants (quartic regulator, polynomial label
// sums), fp64 (MBPT_FIXED_P 0) or fp32 (1): the build compiles the two in
// parallel.
#include "kernels_dev.hpp"

#if !defined(MBPT_FIXED_P)
#error "compile with -DMBPT_FIXED_P=<0|1>"
#endif

namespace mbpt {

template <>
hipError_t launch_o4_fixed<MBPT_FIXED_P>(const KArgs &a, int k0, int k1, int grid, int block,
                                         hipStream_t st) {
  constexpr int O = 4, Q = 4, P = MBPT_FIXED_P;
  const size_t lds = sample_lds_bytes(3 * (O + 1), a.phys.nb, block, lds_tables<Q, P>(),
                                        wave_words<O, Q, P, false>()) +
                     label_lds_bytes<O, Q, P, false>();
  hipLaunchKernelGGL((sample_order<O, Q, P, false, 2>), dim3(grid), dim3(block), lds, st, a, k0,
                     k1);
  return hipGetLastError();
}

}  // namespace mbpt
