// The inverse x pass and the y passes with the run-time radix stages (any axis length; the lengths
// with compiled schedules among them).
#include "pass_kernels.h"

namespace fh {

hipError_t launch_xinv_radix(int cons, const XInvArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  return dispatch_xinv<0>(cons, a, grid, sm, s);
}
hipError_t launch_mid_radix(int dir, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  return dispatch_mid<0>(dir, rows, a, grid, sm, s);
}
hipError_t set_smem_limits_radix(const Geom& g, size_t bytes) {
  hipError_t e = xinv_limits<0>(g, bytes);
  return e == hipSuccess ? mid_limits<0>(bytes) : e;
}

}  // namespace fh
