// The x passes of one constitutive law, for every FFT variant.  They hold the law's arithmetic and
// every producer, so each law is a translation unit of its own (they compile
// beside one another); a unit defines FH_XPASS (its function's name) and FH_XPASS_LAWS(X), a list
// X(matcode, MAT, NDIM).
#include "pass_kernels.h"

namespace fh {

namespace {

template <int MAT, int NDIM, int NF>
hipError_t xfwd_one(int prod, const XFwdArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  if constexpr (NDIM == 3) {
    if (prod == PROD_XOP || prod == PROD_XOP_STORED) {
      if (prod == PROD_XOP) hipLaunchKernelGGL((k_xop<0, MAT, 3, NF>), grid, dim3(kThreads), sm, s, a);
      else hipLaunchKernelGGL((k_xop<1, MAT, 3, NF>), grid, dim3(kThreads), sm, s, a);
      return hipGetLastError();
    }
  }
  switch (prod) {
    case PROD_IDENT: hipLaunchKernelGGL((k_xfwd<PROD_IDENT, MAT, NDIM, NF>), grid, dim3(kThreads), sm, s, a); break;
    case PROD_STRESS: hipLaunchKernelGGL((k_xfwd<PROD_STRESS, MAT, NDIM, NF>), grid, dim3(kThreads), sm, s, a); break;
    case PROD_CGOP: hipLaunchKernelGGL((k_xfwd<PROD_CGOP, MAT, NDIM, NF>), grid, dim3(kThreads), sm, s, a); break;
    case PROD_TRHS: hipLaunchKernelGGL((k_xfwd<PROD_TRHS, MAT, NDIM, NF>), grid, dim3(kThreads), sm, s, a); break;
    case PROD_CGOP_STORED:
      hipLaunchKernelGGL((k_xfwd<PROD_CGOP_STORED, MAT, NDIM, NF>), grid, dim3(kThreads), sm, s, a);
      break;
    case PROD_ADJ: hipLaunchKernelGGL((k_xfwd<PROD_ADJ, MAT, NDIM, NF>), grid, dim3(kThreads), sm, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// 3D axes of a length with its own CG-loop kernels
template <int MAT, int NF>
hipError_t xfwd_fixed(int prod, const XFwdArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  if constexpr (stored_len_kernels(variant_len(NF), !finite_mat(MAT))) {
    if (prod == PROD_XOP_STORED) {
      hipLaunchKernelGGL((k_xop<1, MAT, 3, NF>), grid, dim3(kThreads), sm, s, a);
      return hipGetLastError();
    }
  }
  if (prod == PROD_XOP) hipLaunchKernelGGL((k_xop<0, MAT, 3, NF>), grid, dim3(kThreads), sm, s, a);
  else if (prod == PROD_CGOP) hipLaunchKernelGGL((k_xfwd<PROD_CGOP, MAT, 3, NF>), grid, dim3(kThreads), sm, s, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int MAT, int NDIM>
hipError_t xfwd_nf(int nf, int prod, const XFwdArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  switch (nf) {
    case 0: return xfwd_one<MAT, NDIM, 0>(prod, a, grid, sm, s);
    case kChirp: return xfwd_one<MAT, NDIM, kChirp>(prod, a, grid, sm, s);
    case kDense: return xfwd_one<MAT, NDIM, kDense>(prod, a, grid, sm, s);
    default: break;
  }
  if constexpr (NDIM == 3) {
    switch (nf) {
      case 128: return xfwd_fixed<MAT, 128>(prod, a, grid, sm, s);
      case kStaged + 96: return xfwd_fixed<MAT, kStaged + 96>(prod, a, grid, sm, s);
      case kStaged + 64: return xfwd_fixed<MAT, kStaged + 64>(prod, a, grid, sm, s);
      case kStaged + 48: return xfwd_fixed<MAT, kStaged + 48>(prod, a, grid, sm, s);
      case kStaged + 32: return xfwd_fixed<MAT, kStaged + 32>(prod, a, grid, sm, s);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

template <int MAT, int NDIM, int NF>
hipError_t limits_one(size_t bytes) {
  hipError_t e = hipSuccess;
  for (const void* fn : {reinterpret_cast<const void*>(k_xfwd<PROD_IDENT, MAT, NDIM, NF>),
                         reinterpret_cast<const void*>(k_xfwd<PROD_STRESS, MAT, NDIM, NF>),
                         reinterpret_cast<const void*>(k_xfwd<PROD_CGOP, MAT, NDIM, NF>),
                         reinterpret_cast<const void*>(k_xfwd<PROD_TRHS, MAT, NDIM, NF>),
                         reinterpret_cast<const void*>(k_xfwd<PROD_CGOP_STORED, MAT, NDIM, NF>),
                         reinterpret_cast<const void*>(k_xfwd<PROD_ADJ, MAT, NDIM, NF>)})
    if (e == hipSuccess) e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if constexpr (NDIM == 3) {
    for (const void* fn : {reinterpret_cast<const void*>(k_xop<0, MAT, 3, NF>),
                           reinterpret_cast<const void*>(k_xop<1, MAT, 3, NF>)})
      if (e == hipSuccess) e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  }
  return e;
}

template <int MAT, int NF>
hipError_t stored_limit(size_t bytes) {
  if constexpr (stored_len_kernels(variant_len(NF), !finite_mat(MAT))) return raise_limit(k_xop<1, MAT, 3, NF>, bytes);
  return hipSuccess;
}

template <int MAT, int NDIM>
hipError_t limits_all(size_t bytes) {
  hipError_t e = limits_one<MAT, NDIM, 0>(bytes);
  if (e == hipSuccess) e = limits_one<MAT, NDIM, kChirp>(bytes);
  if (e == hipSuccess) e = limits_one<MAT, NDIM, kDense>(bytes);
  if constexpr (NDIM == 3) {
    for (const void* fn : {reinterpret_cast<const void*>(k_xfwd<PROD_CGOP, MAT, 3, 128>),
                           reinterpret_cast<const void*>(k_xfwd<PROD_CGOP, MAT, 3, kStaged + 96>),
                           reinterpret_cast<const void*>(k_xfwd<PROD_CGOP, MAT, 3, kStaged + 64>),
                           reinterpret_cast<const void*>(k_xfwd<PROD_CGOP, MAT, 3, kStaged + 48>),
                           reinterpret_cast<const void*>(k_xfwd<PROD_CGOP, MAT, 3, kStaged + 32>),
                           reinterpret_cast<const void*>(k_xop<0, MAT, 3, 128>),
                           reinterpret_cast<const void*>(k_xop<0, MAT, 3, kStaged + 96>),
                           reinterpret_cast<const void*>(k_xop<0, MAT, 3, kStaged + 64>),
                           reinterpret_cast<const void*>(k_xop<0, MAT, 3, kStaged + 48>),
                           reinterpret_cast<const void*>(k_xop<0, MAT, 3, kStaged + 32>)})
      if (e == hipSuccess) e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) e = stored_limit<MAT, 128>(bytes);
    if (e == hipSuccess) e = stored_limit<MAT, kStaged + 96>(bytes);
    if (e == hipSuccess) e = stored_limit<MAT, kStaged + 64>(bytes);
    if (e == hipSuccess) e = stored_limit<MAT, kStaged + 48>(bytes);
    if (e == hipSuccess) e = stored_limit<MAT, kStaged + 32>(bytes);
  }
  return e;
}

}  // namespace

#define FH_CAT2(a, b) a##b
#define FH_CAT(a, b) FH_CAT2(a, b)

// launch with FFT variant nf (a template value of k_xfwd)
hipError_t FH_XPASS(int nf, int prod, int mat, const XFwdArgs& a, dim3 grid, size_t sm, hipStream_t s) {
#define FH_X(code, MAT, NDIM) \
  if (mat == code) return xfwd_nf<MAT, NDIM>(nf, prod, a, grid, sm, s);
  FH_XPASS_LAWS(FH_X)
#undef FH_X
  return hipErrorInvalidValue;
}

hipError_t FH_CAT(FH_XPASS, _limits)(int mat, size_t bytes) {
#define FH_X(code, MAT, NDIM) \
  if (mat == code) return limits_all<MAT, NDIM>(bytes);
  FH_XPASS_LAWS(FH_X)
#undef FH_X
  return hipErrorInvalidValue;
}

}  // namespace fh
