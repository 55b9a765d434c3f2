// The outer passes of the CG on displacements with the run-time radix stages.
#include "pass_kernels.h"

namespace fh {

hipError_t launch_outer_cg_radix(int mode, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  return dispatch_outer_cg<0>(mode, a, grid, sm, s);
}
hipError_t set_smem_limits_radix_cg(const Geom& g, size_t bytes) { return outer_cg_limits<0>(g, bytes); }

}  // namespace fh
