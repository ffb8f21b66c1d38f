// Instantiations of the fused SQP kernel for long solves of 6 and 7 degrees of
// freedom (four knots per lane group): on one workgroup, split, and for caller-given
// QP data. (A unit of their own for its loop alignment, see the build's flags.)
#include "gato_launch.hpp"
#include "gato_sqp.hpp"

namespace gato {

namespace {

template <int ND>
hipError_t launch(bool f64, int grid, const KArgs &a, hipStream_t s) {
  const dim3 g(grid), b(kBlock);
  if (!f64) hipLaunchKernelGGL((sqp_kernel<ND, 4, float>), g, b, 0, s, a);
  else if (a.mode == kModeKkt) hipLaunchKernelGGL(kkt_kernel<ND>, g, b, 0, s, a);
  else hipLaunchKernelGGL((sqp_kernel<ND, 4, double>), g, b, 0, s, a);
  return hipGetLastError();
}

// Split solves: a cooperative launch, so that the parts of a solve are resident
// together.
template <int ND>
hipError_t launch_split(bool f64, int grid, const KArgs &a, hipStream_t s) {
  const void *f = f64 ? reinterpret_cast<const void *>(&sqp_kernel<ND, 4, double, false, true>)
                      : reinterpret_cast<const void *>(&sqp_kernel<ND, 4, float, false, true>);
  const hipError_t e = cooperative_fits(f, grid);
  if (e != hipSuccess) return e;
  KArgs arg = a;
  void *args[] = {&arg};
  return hipLaunchCooperativeKernel(f, dim3(grid), dim3(kBlock), args, 0, s);
}

}  // namespace

hipError_t launch_sqp_n6_long(bool f64, int grid, const KArgs &a, hipStream_t s) { return launch<6>(f64, grid, a, s); }
hipError_t launch_sqp_n7_long(bool f64, int grid, const KArgs &a, hipStream_t s) { return launch<7>(f64, grid, a, s); }
hipError_t launch_sqp_n6_split(int grid, bool f64, const KArgs &a, hipStream_t s) {
  return launch_split<6>(f64, grid, a, s);
}
hipError_t launch_sqp_n7_split(int grid, bool f64, const KArgs &a, hipStream_t s) {
  return launch_split<7>(f64, grid, a, s);
}

}  // namespace gato
