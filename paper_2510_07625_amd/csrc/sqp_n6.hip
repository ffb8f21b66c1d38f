// Instantiations of the fused SQP kernel for n = 6 degrees of freedom (long solves:
// sqp_long.hip).
#include "gato_launch.hpp"
#include "gato_sqp.hpp"

namespace gato {

hipError_t launch_sqp_n6(int kpt, bool f64, int grid, const KArgs &a, hipStream_t s) {
  if (kpt == 4) return launch_sqp_n6_long(f64, grid, a, s);
  const dim3 g(grid), b(block_threads(6, kpt, a));
  switch (kpt * 2 + (f64 ? 1 : 0)) {
    case 2: hipLaunchKernelGGL((sqp_kernel<6, 1, float>), g, b, 0, s, a); break;
    case 3: hipLaunchKernelGGL((sqp_kernel<6, 1, double>), g, b, 0, s, a); break;
    case 4: hipLaunchKernelGGL((sqp_kernel<6, 2, float>), g, b, 0, s, a); break;
    case 5: hipLaunchKernelGGL((sqp_kernel<6, 2, double>), g, b, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace gato
