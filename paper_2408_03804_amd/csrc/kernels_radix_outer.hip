// The outer pass (projection, plain transforms) with the run-time radix stages.
#include "pass_kernels.h"

namespace fh {

hipError_t launch_outer_radix(int mode, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  return dispatch_outer<0>(mode, rows, a, grid, sm, s);
}
hipError_t set_smem_limits_radix_outer(const Geom& g, size_t bytes) { return outer_limits<0>(g, bytes); }

}  // namespace fh
