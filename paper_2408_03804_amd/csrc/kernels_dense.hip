// The pass kernels instantiated with the folded dense DFT on the matrix cores, for axis lengths
// without a compiled radix schedule.  A translation unit of its own so that it compiles beside
// kernels.hip; the launchers there route dense plans here.
#include "pass_kernels.h"

namespace fh {

hipError_t launch_xinv_dense(int cons, const XInvArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  return dispatch_xinv<kDense>(cons, a, grid, sm, s);
}
hipError_t launch_mid_dense(int dir, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  return dispatch_mid<kDense>(dir, rows, a, grid, sm, s);
}
hipError_t launch_outer_dense(int mode, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  return outer_cg_mode(mode) ? dispatch_outer_cg<kDense>(mode, a, grid, sm, s) : dispatch_outer<kDense>(mode, rows, a, grid, sm, s);
}
hipError_t set_smem_limits_dense(const Geom& g, size_t bytes) {
  hipError_t e = xinv_limits<kDense>(g, bytes);
  if (e == hipSuccess) e = mid_limits<kDense>(bytes);
  if (e == hipSuccess) e = outer_limits<kDense>(g, bytes);
  if (e == hipSuccess) e = outer_cg_limits<kDense>(g, bytes);
  return e;
}

}  // namespace fh
