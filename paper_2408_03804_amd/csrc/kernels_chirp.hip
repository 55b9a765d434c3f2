// The pass kernels instantiated with the chirp-z (Bluestein) FFT, for axes whose plan carries a
// convolution length m > 0 (lengths with large prime factors).  A translation unit of its own so
// that it compiles beside kernels.hip; the launchers there route chirp-z plans here.
#include "pass_kernels.h"

namespace fh {

hipError_t launch_xinv_chirp(int cons, const XInvArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  return dispatch_xinv<kChirp>(cons, a, grid, sm, s);
}
hipError_t launch_mid_chirp(int dir, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  return dispatch_mid<kChirp>(dir, rows, a, grid, sm, s);
}
hipError_t launch_outer_chirp(int mode, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  return outer_cg_mode(mode) ? dispatch_outer_cg<kChirp>(mode, a, grid, sm, s) : dispatch_outer<kChirp>(mode, rows, a, grid, sm, s);
}
hipError_t set_smem_limits_chirp(const Geom& g, size_t bytes) {
  hipError_t e = xinv_limits<kChirp>(g, bytes);
  if (e == hipSuccess) e = mid_limits<kChirp>(bytes);
  if (e == hipSuccess) e = outer_limits<kChirp>(g, bytes);
  if (e == hipSuccess) e = outer_cg_limits<kChirp>(g, bytes);
  return e;
}

}  // namespace fh
