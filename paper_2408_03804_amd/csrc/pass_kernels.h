// The pass kernels of the Fourier-Galerkin Newton-CG solve for gfx950 (FP64), as templates:
// kernels.hip instantiates them with the direct FFT stages (and the kernels specialised for
// 128-point axes), kernels_fixed.hip for 96-, 64-, 48- and 32-point axes, kernels_chirp.hip with
// the chirp-z transform.
//
// One CG iteration (section 3 equilibrium operator, section 3.2 incremental
// stress, Appendix A linear solve) is five passes over the data:
//
//   xfwd   per voxel: x += alpha_prev p, p = r + beta p, tau = K(F) : p by dual
//          numbers, partial <p, tau>; real-to-complex FFT of tau along x
//   mid    complex FFT along y of the half spectrum            (3D only)
//   outer  FFT along the outer axis, G-hat(xi) : tau-hat on each wavevector,
//          inverse FFT along the outer axis
//   mid    inverse FFT along y                                 (3D only)
//   xinv   complex-to-real FFT along x, r -= alpha q, partial <r, r>
//
// (the CG on strain fields, in 2D and for CG tolerances below kDisplacementTol) or, in 3D at the
// tolerances in everyday use, the CG on displacements:
//
//   outer  x += alpha_prev p, p = r + beta p per wavevector, the strain of p, inverse FFT along z
//   mid    inverse FFT along y
//   x      complex-to-real FFT along x, tau = K(F) : p by dual numbers, partial <p, tau>,
//          real-to-complex FFT along x, in place
//   mid    FFT along y (one block sums <p, tau>, alpha)
//   outer  FFT along z, u of tau, r -= alpha u, partial <r, r>
//
// A compatible strain is the (symmetrised, for small strain) gradient of a displacement, so on each
// wavevector xi the CG vectors x, r and p are three complex numbers u instead of 9 (small strain: 6)
// real ones per voxel:
//   finite strain  A-hat_ij = u_i xi_j
//   small strain   A-hat_ij = (u_i xi_j + u_j xi_i) / 2
// (the factor i of the gradient is part of u).  The projection of a field tau is the u of
//   finite   u = tau-hat xi / |xi|^2
//   small    u = 2 t / |xi|^2 - (xi . t) xi / |xi|^4,  t = tau-hat xi
// and its squared norm, by Parseval, (1/N) sum w |xi|^2 |u|^2 (small: w (|xi|^2 |u|^2 + |xi . u|^2) / 2)
// over the half spectrum, w = 2 except on the planes kx = 0 and kx = nx/2.  These are the iterates of
// the CG on the strains in exact arithmetic; at 128^3 (finite strain) an iteration moves 731 B per
// voxel instead of 1064 B.  In floating point the strain fields also carry an incompatible rounding
// part that no iteration reduces; where rounding decides the iteration count (badly conditioned cells) the
// counts of the two differ by one to four per cent (kDisplacementTol, with the measurements).
// The spectra of real fields on the planes kx = 0 and kx = nx/2 are Hermitian in the other axes.  A
// part of r that is not (rounding of the transforms) would vanish on the way through real space and
// so never be reduced; the forward passes of the CG on displacements therefore keep that symmetry
// exactly: the y pass averages each value with the conjugate of its mirror
// image, and the outer pass of a mirrored ky runs on the conjugate sequence, so that both
// compute the same numbers.
//
// Both add a one-block reduction that turns the partial sums into beta on the device.  <p, q> is taken
// as <p, K:p>: p lies in the range of the projection G (it is built from projected residuals) and G is
// self-adjoint, so <p, G(K:p)> = <G p, K:p> = <p, K:p> in exact arithmetic; q is therefore never
// stored.  On strain fields the update x += alpha p of iteration k is applied by the xfwd pass of
// iteration k+1, which reads p anyway (k_cg_finish applies the last one).
#pragma once

#include "common.h"
#include "fft_lds.h"
#include "kernels.h"
#include "materials.h"

namespace fh {

// matcode = 2 * material + (ndim - 2); 8, 9: Neo-Hookean, J2 under plane stress (2D)
#define FH_DISPATCH_MAT(matcode, MACRO) \
  switch (matcode) {                    \
    case 0: MACRO(MAT_LE, 2); break;    \
    case 1: MACRO(MAT_LE, 3); break;    \
    case 2: MACRO(MAT_NH, 2); break;    \
    case 3: MACRO(MAT_NH, 3); break;    \
    case 4: MACRO(MAT_STVK, 2); break;  \
    case 5: MACRO(MAT_STVK, 3); break;  \
    case 6: MACRO(MAT_J2, 2); break;    \
    case 7: MACRO(MAT_J2, 3); break;    \
    case 8: MACRO(MAT_NH_PS, 2); break; \
    case 9: MACRO(MAT_J2_PS, 2); break; \
    default: return hipErrorInvalidValue; \
  }

// Parameters (and for J2 the plastic history) of voxel v.
template <int MAT, int NDIM>
__device__ __forceinline__ void load_local(const MatParams& m, long long v, Local& L) {
  const int ph = m.phase[v];
  const double* row = m.table + (long long)m.tstride * ph;
  L.lam = row[0];
  L.mu = row[1];
  if (m.scale != nullptr) {
    const double s = m.scale[v];
    L.lam *= s;
    L.mu *= s;
  }
  if constexpr (j2_mat(MAT)) {
    constexpr int C = MatTraits<MAT, NDIM>::C;
    L.sy = row[2];
    L.H = row[3];
#pragma unroll
    for (int k = 0; k <= C; ++k) L.hist[k] = m.hist[k * m.hN + v];
  }
}

__device__ __forceinline__ int ceil_div(int a, int b) { return (a + b - 1) / b; }

// FFT variant of a pass kernel (template parameter NF):
//   0              any length with direct stages, with the register staging or the ping-pong
//                  buffer the host chose;
//   kChirp         the chirp-z transform (plans with m > 0; kernels_chirp.hip);
//   L, 0 < L < kStaged   length L only, one butterfly per thread per stage (the launchers check
//                  fixed_one_ok): only that length's code and a butterfly's registers;
//   kStaged + L    length L only (a compiled schedule), register staging of up to kInplaceElems
//                  elements per thread (the host chose in-place stages; kernels_fixed.hip).
// The generic kernels hold every compiled schedule, and their registers follow the longest one;
// the length-specific kernels hold one.  The buffers hold lds_len(pl) rows per sequence.
constexpr int kChirp = -1;
constexpr int kDense = -2;  // the folded dense DFT (plans with dense set; kernels_dense.hip)
constexpr int kStaged = 1 << 12;
template <int D, int NF>
__device__ __forceinline__ void pass_fft(double2* A, double2* Bf, int nseq, const AxisPlan& pl, int inplace) {
  if constexpr (NF > kStaged) fixed_stages<NF - kStaged, D, 0, 1>(A, nseq, make_fastdiv((unsigned)nseq), pl.tw);
  else if constexpr (NF > 0) fft_fixed_one<NF, D>(A, nseq, pl.tw);
  else if constexpr (NF == kChirp) fft_chirp<D>(A, Bf, nseq, pl, inplace);
  else if constexpr (NF == kDense) fft_dense<D>(A, Bf, nseq, pl, inplace);
  else fft_lds_any<D>(A, Bf, nseq, pl, inplace);
}

// Streaming access for the CG vectors and the linearisation point: each is touched once
// per CG iteration, so keeping them out of the caches leaves room for the half spectrum
// that the FFT passes hand to each other.
__device__ __forceinline__ double ld_stream(const double* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ void st_stream(double* p, double v) { __builtin_nontemporal_store(v, p); }

// nt: past the caches (wave-uniform)
__device__ __forceinline__ double2 ld_vec(const double2* p, bool nt) {
  if (!nt) return *p;
  typedef double v2d __attribute__((ext_vector_type(2)));
  const v2d v = __builtin_nontemporal_load(reinterpret_cast<const v2d*>(p));
  return make_double2(v.x, v.y);
}
__device__ __forceinline__ void st_vec(double2* p, double2 v, bool nt) {
  if (!nt) {
    *p = v;
    return;
  }
  typedef double v2d __attribute__((ext_vector_type(2)));
  __builtin_nontemporal_store(v2d{v.x, v.y}, reinterpret_cast<v2d*>(p));
}

// Sum of x[tid], x[tid + kThreads], x[tid + 2 kThreads], ... (i < n) in that order, with up to S of
// the thread's loads in flight together; bitwise the strided loop's sum.
template <int S, int BD>
__device__ __forceinline__ double strided_sum(const double* __restrict__ x, int n) {
  double acc = 0.0;
  for (int base = 0; base < n; base += S * BD) {
    double v[S];
#pragma unroll
    for (int e = 0; e < S; ++e) {
      const int i = base + (int)threadIdx.x + e * BD;
      v[e] = i < n ? x[i] : 0.0;
    }
#pragma unroll
    for (int e = 0; e < S; ++e) acc += v[e];
  }
  return acc;
}

// Gather n complex entries into LDS: dst[t] = src(t), t < n.  Each thread issues up to S global loads
// before its first LDS write, so that S of its loads are in flight together (in a plain
// load-then-write loop each load waits for the previous one).  The loads are unconditional, at a
// clamped index: a load under a condition is waited for before the next one is issued.
template <int S, typename Src>
__device__ __forceinline__ void gather_staged(double2* dst, int n, Src src) {
  for (int base = 0; base < n; base += S * kThreads) {
    double2 v[S];
#pragma unroll
    for (int e = 0; e < S; ++e) v[e] = src(min(base + (int)threadIdx.x + e * kThreads, n - 1));
#pragma unroll
    for (int e = 0; e < S; ++e) {
      const int t = base + (int)threadIdx.x + e * kThreads;
      if (t < n) dst[t] = v[e];
    }
  }
}

// ============================================================================
// CG scalar bookkeeping from a reduced sum (fixed-order two-stage sums)
// ============================================================================
template <int WHAT>
__device__ __forceinline__ void cg_finalize(CgState& S, double s) {
  if (WHAT == RED_SRC) {
    S.src2 = s;
  } else if (WHAT == RED_RHS) {
    S.rr0 = s;
    S.rr = s;
    S.iters = 0;
    S.first = 1;
    S.beta = 0.0;
    if (!finite_bits(s)) S.status = CG_BREAKDOWN;
    else if (sqrt(s) <= 1e-13 * sqrt(S.src2)) S.status = CG_ZERO_RHS;
    else if (sqrt(s) <= S.tol * sqrt(s)) S.status = CG_CONVERGED;
    else if (S.max_iters <= 0) S.status = CG_MAXIT;
    else S.status = CG_RUNNING;
  } else if (WHAT == RED_PQ) {
    // runs inside the outer pass, whose other blocks read the status: a breakdown is only
    // flagged here and becomes the status at the <r, r> step
    S.pq = s;
    if (!(finite_bits(s) && s > 0.0)) S.pq_fail = 1;
    else S.alpha = S.rr / s;
  } else {  // RED_RR
    if (S.pq_fail) {
      S.status = CG_BREAKDOWN;
      return;
    }
    S.beta = s / S.rr;
    S.rr = s;
    S.iters += 1;
    S.first = 0;
    if (!finite_bits(s)) S.status = CG_BREAKDOWN;
    else if (sqrt(s) <= S.tol * sqrt(S.rr0)) S.status = CG_CONVERGED;
    else if (S.iters >= S.max_iters) S.status = CG_MAXIT;
  }
}

// ============================================================================
// x-axis forward pass
// ============================================================================
template <int PROD, int MAT, int NDIM, int NF = 0>
__global__ void __launch_bounds__(kThreads) k_xfwd(XFwdArgs a) {
  constexpr int C = MatTraits<MAT, NDIM>::C;
  constexpr bool CGOP = (PROD == PROD_CGOP || PROD == PROD_CGOP_STORED);
  const int b = a.active ? a.active[blockIdx.y] : (int)blockIdx.y;
  if (CGOP) {
    if (a.st[b].status != CG_RUNNING) return;
  }
  const Geom& g = a.g;
  // cell of this right-hand side and its load index within the cell
  MatParams mat = a.mat;
  int lb = b;
  if (a.per_inst > 0) {
    const int cell = b / a.per_inst;
    lb = b - cell * a.per_inst;
    mat.phase += (long long)cell * g.N;
    mat.table += (long long)cell * 2 * kMaxPhase;
  }
  const int nx = g.nx;
  const int rows = g.ny * g.nz;
  const int row0 = blockIdx.x * a.R;
  const int nr = min(a.R, rows - row0);
  const int nseq = C * nr;
  const int P = (nseq + 1) >> 1;
  extern __shared__ double2 smem[];
  double2* A = smem;
  // CG operator: strain staged by phase A (after the FFT buffers)
  const int nv = nr * nx;
  double* E = reinterpret_cast<double*>(smem + (size_t)(a.inplace ? 1 : 2) * g.lx * P);
  double2* Bf = smem + (size_t)g.lx * P;  // ping-pong partner (unused in place)
  __shared__ double red[kThreads / 64];

  double beta = 0.0, alpha_prev = 0.0;
  int first = 1;
  if (CGOP) {
    beta = a.st[b].beta;
    alpha_prev = a.st[b].alpha;
    first = a.st[b].first;
  }
  const long long N = g.N;
  double acc = 0.0;
  int bad = 0;

  // LDS slot of component j of row r at column x (two real rows per complex sequence)
  auto slot = [&](int j, int r, int x) -> double* {
    const int qr = j * nr + r;
    return reinterpret_cast<double*>(&A[x * P + (qr >> 1)]) + (qr & 1);
  };

  if (CGOP) {
    // phase A: every global load of the voxel in flight together.
    //   x += alpha_prev p_old ; p = r + beta p_old   (p staged in the FFT slots)
    //   strain staged for phase B
    for (int t = threadIdx.x; t < nv; t += blockDim.x) {
      const int r = t / nx;
      const int x = t - r * nx;
      const long long vox = (long long)(row0 + r) * nx + x;
      if (PROD == PROD_CGOP && MAT != MAT_LE) {
#pragma unroll
        for (int j = 0; j < C; ++j) E[j * nv + t] = ld_stream(a.F + j * N + vox);
      }
      if (!j2_mat(MAT)) {
        Local L;
        load_local<MAT, NDIM>(mat, vox, L);  // brings the phase id and table line into cache
        (void)L;
      }
      // r, p and x are distinct buffers: every load is issued before the first store (without the
      // restrict qualifiers the compiler must order each component's loads after the previous
      // component's stores, one memory round trip per component)
      const double* __restrict__ rin = a.in + (long long)b * C * N + vox;
      double* __restrict__ pio = a.p + (long long)b * C * N + vox;
      double* __restrict__ xio = a.x + (long long)b * C * N + vox;
      double rv[C], pv[C], xv[C];
#pragma unroll
      for (int j = 0; j < C; ++j) rv[j] = ld_stream(rin + j * N);
      if (!first) {
#pragma unroll
        for (int j = 0; j < C; ++j) {
          pv[j] = ld_stream(pio + j * N);
          xv[j] = ld_stream(xio + j * N);
        }
      }
#pragma unroll
      for (int j = 0; j < C; ++j) {
        double pj = rv[j];
        if (!first) {
          st_stream(xio + j * N, xv[j] + alpha_prev * pv[j]);
          pj = rv[j] + beta * pv[j];
        }
        st_stream(pio + j * N, pj);
        *slot(j, r, x) = pj;
      }
    }
  }

  // phase B (or the only phase): per-voxel producer, result into the LDS slots
#pragma unroll 1
  for (int t = threadIdx.x; t < nr * nx; t += blockDim.x) {
    const int r = t / nx;
    const int x = t - r * nx;
    const long long vox = (long long)(row0 + r) * nx + x;
    double v[C];
    if (PROD == PROD_IDENT) {
#pragma unroll
      for (int j = 0; j < C; ++j) v[j] = a.in[((long long)b * C + j) * N + vox];
    } else {
      Local L;
      double e[C];
      // the linear elastic energy is quadratic: K does not depend on the strain,
      // so the tangent passes do not read it
      // (lam, mu) are re-read here (cache hits): staging them in LDS as well
      // raises the register count of the fused kernel by a third
      load_local<MAT, NDIM>(mat, vox, L);
      if (CGOP) {
#pragma unroll
        for (int j = 0; j < C; ++j) e[j] = (PROD == PROD_CGOP && MAT != MAT_LE) ? E[j * nv + t] : 0.0;
      } else {
        const bool need_e = (PROD == PROD_STRESS) || (PROD == PROD_ADJ) || (MAT != MAT_LE);
#pragma unroll
        for (int j = 0; j < C; ++j) e[j] = need_e ? a.F[j * N + vox] : 0.0;
      }
      if (PROD == PROD_STRESS) {
        if (finite_mat(MAT)) {
          const double J = det_packed<NDIM>(e);
          if (!(finite_bits(J) && J > 0.0)) bad = 1;
        }
        stress_ad<MAT, NDIM>(e, L, v);
#pragma unroll
        for (int j = 0; j < C; ++j) {
          acc += v[j] * v[j];
          if (!finite_bits(v[j])) bad = 1;
        }
      } else if (PROD == PROD_ADJ) {
        // objective gradient with respect to the strain: g = w_e P + K : W
        double P[C], W[C];
#pragma unroll
        for (int j = 0; j < C; ++j) W[j] = a.unit[j];
        stress_and_jvp_ad<MAT, NDIM>(e, W, L, P, v);
#pragma unroll
        for (int j = 0; j < C; ++j) {
          v[j] += a.w_energy * P[j];
          acc += v[j] * v[j];
        }
      } else if (PROD == PROD_TRHS) {
        double de[C];
#pragma unroll
        for (int j = 0; j < C; ++j) de[j] = (j == lb) ? a.unit[lb] : 0.0;
        tangent_jvp_ad<MAT, NDIM>(e, de, L, v);
#pragma unroll
        for (int j = 0; j < C; ++j) acc += v[j] * v[j];
      } else {  // CG operator: v = K : p with p from phase A
        double pv[C];
#pragma unroll
        for (int j = 0; j < C; ++j) pv[j] = *slot(j, r, x);
        if (PROD == PROD_CGOP) {
          tangent_jvp_ad<MAT, NDIM>(e, pv, L, v);
        } else {
          // stored symmetric tangent, upper triangle row by row
#pragma unroll
          for (int i = 0; i < C; ++i) v[i] = 0.0;
          int idx = 0;
#pragma unroll
          for (int i = 0; i < C; ++i) {
#pragma unroll
            for (int j = i; j < C; ++j) {
              const double k = a.Kst[(long long)idx * N + vox];
              v[i] += k * pv[j];
              if (j != i) v[j] += k * pv[i];
              ++idx;
            }
          }
        }
#pragma unroll
        for (int j = 0; j < C; ++j) acc += pv[j] * v[j];
      }
    }
#pragma unroll
    for (int j = 0; j < C; ++j) *slot(j, r, x) = v[j];
  }
  if (nseq & 1) {
    for (int x = threadIdx.x; x < nx; x += blockDim.x) A[x * P + P - 1].y = 0.0;
  }
  if (PROD == PROD_STRESS && bad) a.st[b].domain = 1;
  __syncthreads();

  pass_fft<-1, NF>(A, Bf, P, a.px, a.inplace);
  const double2* res = A;

  // separate the two real rows packed in each complex sequence
  const int nxh = g.nxh;
  const FastDiv fdh = make_fastdiv((unsigned)nxh);
  for (int t = threadIdx.x; t < P * nxh; t += blockDim.x) {
    const int q = (int)fdiv((unsigned)t, fdh);
    const int k = t - q * nxh;
    const double2 zk = res[k * P + q];
    const double2 zm = res[(k == 0 ? 0 : nx - k) * P + q];
    const int qa = 2 * q;
    const int ja = qa / nr;
    const int ra = qa - ja * nr;
    a.spec[((long long)b * C + ja) * g.Nh + (long long)(row0 + ra) * g.nxp + k] =
        make_double2(0.5 * (zk.x + zm.x), 0.5 * (zk.y - zm.y));
    if (qa + 1 < nseq) {
      const int jb = (qa + 1) / nr;
      const int rb = (qa + 1) - jb * nr;
      a.spec[((long long)b * C + jb) * g.Nh + (long long)(row0 + rb) * g.nxp + k] =
          make_double2(0.5 * (zk.y + zm.y), 0.5 * (zm.x - zk.x));
    }
  }

  if (PROD != PROD_IDENT) {
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) a.partials[(long long)b * a.nblocks + blockIdx.x] = s;
  }
}

// ============================================================================
// x-axis inverse pass
// ============================================================================
template <int CONS, int C, int NF = 0>
// 4 waves per SIMD (at most 128 VGPRs): measured 5 % faster at 128^3 than the unconstrained 166
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(NF == kDense ? 3 : 4, 8))) k_xinv(XInvArgs a) {
  const int b = a.active ? a.active[blockIdx.y] : (int)blockIdx.y;
  if (CONS == CONS_CGUPD) {
    if (a.st[b].status != CG_RUNNING) return;
  }
  const Geom& g = a.g;
  const int nx = g.nx;
  const int nxh = g.nxh;
  const int rows = g.ny * g.nz;
  const int row0 = blockIdx.x * a.R;
  const int nr = min(a.R, rows - row0);
  const int nseq = C * nr;
  const int P = (nseq + 1) >> 1;
  extern __shared__ double2 smem[];
  double2* A = smem;
  double2* H = smem + (size_t)g.lx * P;  // loaded half rows, then the ping-pong partner
  __shared__ double red[kThreads / 64];
  const long long N = g.N;

  // the residual of this thread's voxel is loaded before the transform so that
  // its latency hides behind the FFT (one voxel per thread)
  const bool pre = (CONS == CONS_CGUPD) && (nr * nx <= (int)blockDim.x);
  double rpre[C];
  if (pre && (int)threadIdx.x < nr * nx) {
    const int r = threadIdx.x / nx;
    const int x = threadIdx.x - r * nx;
    const long long vox = (long long)(row0 + r) * nx + x;
#pragma unroll
    for (int j = 0; j < C; ++j) rpre[j] = ld_stream(a.r + ((long long)b * C + j) * N + vox);
  }

  const FastDiv fdh = make_fastdiv((unsigned)nxh);
  const FastDiv fdp = make_fastdiv((unsigned)P);
  const int hcnt = nseq * nxh;
  for (int base = 0; base < hcnt; base += 8 * kThreads) {
    double2 v[8];
    int di[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int t = min(base + (int)threadIdx.x + e * kThreads, hcnt - 1);
      const int qr = (int)fdiv((unsigned)t, fdh);
      const int k = t - qr * nxh;
      const int j = qr / nr;
      const int r = qr - j * nr;
      di[e] = k * nseq + qr;
      v[e] = a.spec[((long long)b * C + j) * g.Nh + (long long)(row0 + r) * g.nxp + k];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (base + (int)threadIdx.x + e * kThreads < hcnt) H[di[e]] = v[e];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < P * nx; t += blockDim.x) {
    const int k = (int)fdiv((unsigned)t, fdp);
    const int q = t - k * P;
    const int qa = 2 * q;
    const bool hb = qa + 1 < nseq;
    double2 z;
    if (k < nxh) {
      double2 ha = H[k * nseq + qa];
      double2 hv = hb ? H[k * nseq + qa + 1] : make_double2(0.0, 0.0);
      if (k == 0 || 2 * k == nx) {
        ha.y = 0.0;
        hv.y = 0.0;
      }
      z = make_double2(ha.x - hv.y, ha.y + hv.x);
    } else {
      const int m = nx - k;
      const double2 ha = H[m * nseq + qa];
      const double2 hv = hb ? H[m * nseq + qa + 1] : make_double2(0.0, 0.0);
      z = make_double2(ha.x + hv.y, hv.x - ha.y);
    }
    A[k * P + q] = z;
  }
  __syncthreads();

  pass_fft<1, NF>(A, H, P, a.px, a.inplace);
  const double2* res = A;

  double alpha = 0.0;
  if (CONS == CONS_CGUPD) alpha = a.st[b].alpha;
  double acc = 0.0;
  for (int t = threadIdx.x; t < nr * nx; t += blockDim.x) {
    const int r = t / nx;
    const int x = t - r * nx;
    const long long vox = (long long)(row0 + r) * nx + x;
    // the residual's components are all loaded before the first store (restrict: no component's
    // store has to wait for the next one's load)
    double* __restrict__ rio = a.r + (long long)b * C * N + vox;
    double rv[C];
    if (CONS == CONS_CGUPD) {
#pragma unroll
      for (int j = 0; j < C; ++j) rv[j] = pre ? rpre[j] : ld_stream(rio + j * N);
    }
#pragma unroll
    for (int j = 0; j < C; ++j) {
      const int qr = j * nr + r;
      const double* d = reinterpret_cast<const double*>(&res[x * P + (qr >> 1)]);
      const double u = d[qr & 1] * a.scale;
      const long long idx = ((long long)b * C + j) * N + vox;
      if (CONS == CONS_IDENT) {
        a.out[idx] = u;
      } else if (CONS == CONS_RHS) {
        a.r[idx] = -u;
        a.x[idx] = 0.0;
        acc += u * u;
      } else {
        const double rn = rv[j] - alpha * u;
        st_stream(rio + j * N, rn);
        acc += rn * rn;
      }
    }
  }
  if (CONS != CONS_IDENT) {
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) a.partials[(long long)b * a.nblocks + blockIdx.x] = s;
  }
}

// ============================================================================
// x-axis pass of the CG on displacements
// ============================================================================
// The C real rows (component j of line r) of a block are packed two per complex sequence: real row
// qr = j * nr + r is the real (even qr) or imaginary part of sequence qr / 2, so that its entry x is the
// double 2 P x + qr of A: component j of a voxel always sits nr doubles behind component j - 1.
__device__ __forceinline__ double* x_slot(double2* A, int P, int nr, int j, int r, int x) {
  const int qr = j * nr + r;
  return reinterpret_cast<double*>(&A[x * P + (qr >> 1)]) + (qr & 1);
}

// Axis length of FFT variant NF if it has one compiled in, else 0.
constexpr int variant_len(int nf) { return nf > kStaged ? nf - kStaged : nf > 0 ? nf : 0; }

// Half spectra of the block's real rows into packed full spectra in LDS (k and nx - k from one load
// pair), and back.  NX: the axis length if known at compile time.  From 94 points on a wavefront
// takes whole sequences (its sequence index is scalar, lanes run along k), three of them in flight:
// the index arithmetic of flattened loops was a good part of the x pass's instructions.
template <int NX>
__device__ __forceinline__ void load_rows(double2* A, const double2* spec, const Geom& g, int nseq, int nr, int row0) {
  const int P = (nseq + 1) >> 1;
  const int nx = NX > 0 ? NX : g.nx, nxh = nx / 2 + 1;
  const FastDiv fdr = make_fastdiv((unsigned)nr);
  auto row = [&](int qr) {
    const int j = (int)fdiv((unsigned)qr, fdr);
    return spec + j * g.Nh + (long long)(row0 + qr - j * nr) * g.nxp;
  };
  auto put = [&](int q, int k, double2 ha, double2 hb) {
    if (2 * q + 1 == nseq) hb = make_double2(0.0, 0.0);
    if (k == 0 || 2 * k == nx) {
      A[k * P + q] = make_double2(ha.x, hb.x);
    } else {
      A[k * P + q] = make_double2(ha.x - hb.y, ha.y + hb.x);
      A[(nx - k) * P + q] = make_double2(ha.x + hb.y, hb.x - ha.y);
    }
  };
  constexpr int S = 3;
  if (nxh >= 48) {
    constexpr int W = kThreads / 64;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    for (int k0 = 0; k0 < nxh; k0 += 64) {
      const int kc = min(k0 + lane, nxh - 1);
      for (int q0 = wave; q0 < P; q0 += S * W) {
        double2 ha[S], hb[S];
#pragma unroll
        for (int e = 0; e < S; ++e) {
          const int q = min(q0 + e * W, P - 1);
          ha[e] = row(2 * q)[kc];
          hb[e] = row(min(2 * q + 1, nseq - 1))[kc];
        }
#pragma unroll
        for (int e = 0; e < S; ++e)
          if (q0 + e * W < P && k0 + lane < nxh) put(q0 + e * W, k0 + lane, ha[e], hb[e]);
      }
    }
  } else {
    const FastDiv fdh = make_fastdiv((unsigned)nxh);
    const int cnt = P * nxh;
    for (int base = 0; base < cnt; base += S * kThreads) {
      double2 ha[S], hb[S];
#pragma unroll
      for (int e = 0; e < S; ++e) {
        const int t = min(base + (int)threadIdx.x + e * kThreads, cnt - 1);
        const int q = NX > 0 ? t / (NX / 2 + 1) : (int)fdiv((unsigned)t, fdh);
        const int k = t - q * nxh;
        ha[e] = row(2 * q)[k];
        hb[e] = row(min(2 * q + 1, nseq - 1))[k];
      }
#pragma unroll
      for (int e = 0; e < S; ++e) {
        const int t = base + (int)threadIdx.x + e * kThreads;
        const int q = NX > 0 ? t / (NX / 2 + 1) : (int)fdiv((unsigned)t, fdh);
        if (t < cnt) put(q, t - q * nxh, ha[e], hb[e]);
      }
    }
  }
}

// Separate the two real rows packed in each transformed sequence and store their half spectra.
template <int NX>
__device__ __forceinline__ void store_rows(const double2* A, double2* spec, const Geom& g, int nseq, int nr, int row0) {
  const int P = (nseq + 1) >> 1;
  const int nx = NX > 0 ? NX : g.nx, nxh = nx / 2 + 1;
  const FastDiv fdr = make_fastdiv((unsigned)nr);
  auto put = [&](int q, int k) {
    const double2 zk = A[k * P + q];
    const double2 zm = A[(k == 0 ? 0 : nx - k) * P + q];
    const int ja = (int)fdiv((unsigned)(2 * q), fdr);
    (spec + ja * g.Nh + (long long)(row0 + 2 * q - ja * nr) * g.nxp)[k] =
        make_double2(0.5 * (zk.x + zm.x), 0.5 * (zk.y - zm.y));
    if (2 * q + 1 < nseq) {
      const int jb = (int)fdiv((unsigned)(2 * q + 1), fdr);
      (spec + jb * g.Nh + (long long)(row0 + 2 * q + 1 - jb * nr) * g.nxp)[k] =
          make_double2(0.5 * (zk.y + zm.y), 0.5 * (zm.x - zk.x));
    }
  };
  if (nxh >= 48) {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    for (int q = wave; q < P; q += kThreads / 64)
      for (int k = threadIdx.x & 63; k < nxh; k += 64) put(q, k);
  } else {
    const FastDiv fdh = make_fastdiv((unsigned)nxh);
    for (int t = threadIdx.x; t < P * nxh; t += blockDim.x) {
      const int q = NX > 0 ? t / (NX / 2 + 1) : (int)fdiv((unsigned)t, fdh);
      put(q, t - q * nxh);
    }
  }
}

// Material of right-hand side b of a multi-cell batch (its cell's phase map and table) and the load
// index within the cell.
__device__ __forceinline__ MatParams cell_material(const XFwdArgs& a, int b, int* load) {
  MatParams mat = a.mat;
  *load = b;
  if (a.per_inst > 0) {
    const int cell = b / a.per_inst;
    *load = b - cell * a.per_inst;
    mat.phase += (long long)cell * a.g.N;
    mat.table += (long long)cell * 2 * kMaxPhase;
  }
  return mat;
}

// K : p of one voxel from the stored symmetric tangent (upper triangle row by row)
template <int C>
__device__ __forceinline__ void stored_apply(const double* Kst, long long N, long long vox, const double* pv, double* v) {
#pragma unroll
  for (int i = 0; i < C; ++i) v[i] = 0.0;
  int idx = 0;
#pragma unroll
  for (int i = 0; i < C; ++i) {
#pragma unroll
    for (int j = i; j < C; ++j) {
      const double k = Kst[(long long)idx * N + vox];
      v[i] += k * pv[j];
      if (j != i) v[j] += k * pv[i];
      ++idx;
    }
  }
}

// The x pass of a CG iteration: inverse transform of the strain of p, K : p per voxel (dual numbers,
// or the stored tangent), partial <p, K:p>, forward transform, in place in the spectrum.
// It reads and writes the half spectrum and reads the linearisation point: 219 B per voxel at 128^3,
// c = 9, which a copy takes 107 us for; measured 123 us (149 us while its index arithmetic was a third
// of its 1376 instructions per voxel), in place of the forward and the inverse x pass of the CG on
// strain fields, 184 and 92 us.  The strain of this thread's voxel is loaded beside the spectrum when a
// block has one voxel per thread, so that it is there when the inverse transform is done.
template <int STORED, int MAT, int NDIM, int NF = 0>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(NF > 0 ? 4 : 2, 8))) k_xop(XFwdArgs a) {
  constexpr int C = MatTraits<MAT, NDIM>::C;
  constexpr bool NEED_E = !STORED && MAT != MAT_LE;
  constexpr int NX = variant_len(NF);
  const int b = a.active ? a.active[blockIdx.y] : (int)blockIdx.y;
  if (a.st[b].status != CG_RUNNING) return;
  const Geom& g = a.g;
  int lb;
  const MatParams mat = cell_material(a, b, &lb);
  const int nx = NX > 0 ? NX : g.nx;
  const int row0 = blockIdx.x * a.R;
  const int nr = min(a.R, g.ny * g.nz - row0);
  const int nseq = C * nr;
  const int P = (nseq + 1) >> 1;
  extern __shared__ double2 smem[];
  double2* A = smem;
  double2* Bf = smem + (size_t)g.lx * P;  // ping-pong partner (unused in place)
  __shared__ double red[kThreads / 64];
  const long long N = g.N;
  double2* spec = a.spec + (long long)b * C * g.Nh;

  const bool pre = nr * nx <= (int)blockDim.x;
  double epre[C];
  if (NEED_E && pre && (int)threadIdx.x < nr * nx) {
#pragma unroll
    for (int j = 0; j < C; ++j) epre[j] = ld_stream(a.F + j * N + (long long)row0 * nx + threadIdx.x);
  }
  load_rows<NX>(A, spec, g, nseq, nr, row0);
  __syncthreads();
  pass_fft<1, NF>(A, Bf, P, a.px, a.inplace);

  double acc = 0.0;
  const FastDiv fdx = make_fastdiv((unsigned)nx);
  // Both arms of the branches on `even` give the same address.  They are there for the registers: one
  // unconditional access each, from the voxel's first slot, makes the compiler keep the C addresses across the law
  // and spill 11 registers instead of 3 (Neo-Hookean 128^3: 156 us against 126; St. Venant-Kirchhoff 96^3:
  // 86 against 69; forming the addresses again for the stores: 174 and 83).
  const bool even = (nr & 1) == 0;
#pragma unroll 1
  for (int t = threadIdx.x; t < nr * nx; t += blockDim.x) {
    const int r = NX > 0 ? t / (NX > 0 ? NX : 1) : (int)fdiv((unsigned)t, fdx);
    const int x = t - r * nx;
    const long long vox = (long long)row0 * nx + t;
    double* slot = x_slot(A, P, nr, 0, r, x);
    double pv[C], v[C];
#pragma unroll
    for (int j = 0; j < C; ++j) pv[j] = (even ? slot[j * nr] : *x_slot(A, P, nr, j, r, x)) * a.scale;
    if (STORED) {
      stored_apply<C>(a.Kst, N, vox, pv, v);
    } else {
      Local L;
      double e[C];
      load_local<MAT, NDIM>(mat, vox, L);
#pragma unroll
      for (int j = 0; j < C; ++j) e[j] = !NEED_E ? 0.0 : pre ? epre[j] : ld_stream(a.F + j * N + vox);
      tangent_jvp_ad<MAT, NDIM>(e, pv, L, v);
    }
#pragma unroll
    for (int j = 0; j < C; ++j) {
      acc += pv[j] * v[j];
      if (even) slot[j * nr] = v[j];
      else *x_slot(A, P, nr, j, r, x) = v[j];
    }
  }
  if (nseq & 1) {
    for (int x = threadIdx.x; x < nx; x += blockDim.x) A[x * P + P - 1].y = 0.0;
  }
  __syncthreads();
  pass_fft<-1, NF>(A, Bf, P, a.px, a.inplace);
  store_rows<NX>(A, spec, g, nseq, nr, row0);
  const double s = block_sum(acc, red);
  if (threadIdx.x == 0) a.partials[(long long)b * a.nblocks + blockIdx.x] = s;
}

// One block of a launch sums <p, K:p> of its right-hand side and sets alpha, for the next launch
// (every thread of the block calls it; no block of this launch reads what it writes).
__device__ __forceinline__ void reduce_alpha(const AxisArgs& a, int b) {
  __shared__ double red[kThreads / 64];
  const double s = block_sum(strided_sum<8, kThreads>(a.pq_partials + (long long)b * a.pq_nblocks, a.pq_nblocks), red);
  if (threadIdx.x == 0) cg_finalize<RED_PQ>(a.pq_st[b], s);
}

// kx on a plane whose spectrum mirrors itself
__device__ __forceinline__ bool mirror_plane(int kx, int nx) { return kx == 0 || 2 * kx == nx; }
// Row y of sequence q of the transform of a real sequence, averaged with the conjugate of its mirror
// image (D[y * nseq + q], rows 0..n-1).
__device__ __forceinline__ double2 hermitian(const double2* D, int y, int q, int nseq, int n) {
  const double2 v = D[y * nseq + q];
  const double2 m = D[(y == 0 ? 0 : n - y) * nseq + q];
  return make_double2(0.5 * (v.x + m.x), 0.5 * (v.y - m.y));
}

// ============================================================================
// y-axis pass (3D): complex FFT of the half spectrum along y, in place
// ============================================================================
// A block transforms the tw bins kx0.. of ZB consecutive z planes (contiguous in memory when
// the tile spans the whole row); sequence q = zz * tw + s, element y at A[y * nseq + q].
template <int DIR, int NF = 0>
__global__ void __launch_bounds__(kThreads) k_mid(AxisArgs a) {
  const Geom& g = a.g;
  const int vb = blockIdx.z / g.c;
  const int comp = blockIdx.z - vb * g.c;
  const int b = a.active ? a.active[vb] : vb;
  if (a.st != nullptr && a.st[b].status != CG_RUNNING) return;
  if (DIR < 0 && a.pq_st != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && comp == 0) reduce_alpha(a, b);
  const int kx0 = blockIdx.x * a.TX;
  const int tw = kx_tile_width(g.nxh, a.TX, blockIdx.x);
  const int ny = g.ny;
  const int z0 = blockIdx.y * a.ZB;
  const int nseq = min(a.ZB, g.nz - z0) * tw;
  extern __shared__ double2 smem[];
  double2* A = smem;
  double2* Bf = smem + (size_t)g.lm * nseq;
  const long long base = ((long long)b * g.c + comp) * g.Nh + (long long)z0 * ny * g.nxp + kx0;
  const FastDiv fdq = make_fastdiv((unsigned)nseq);
  const FastDiv fdt = make_fastdiv((unsigned)tw);
  gather_staged<8>(A, ny * nseq, [&](int t) {
    const int y = (int)fdiv((unsigned)t, fdq);
    const int q = t - y * nseq;
    const int zz = (int)fdiv((unsigned)q, fdt);
    const int s = q - zz * tw;
    return a.spec[base + (long long)(zz * ny + y) * g.nxp + s];
  });
  __syncthreads();
  pass_fft<DIR, NF>(A, Bf, nseq, a.pl, a.inplace);
  for (int t = threadIdx.x; t < ny * nseq; t += blockDim.x) {
    const int y = (int)fdiv((unsigned)t, fdq);
    const int q = t - y * nseq;
    const int zz = (int)fdiv((unsigned)q, fdt);
    const int s = q - zz * tw;
    a.spec[base + (long long)(zz * ny + y) * g.nxp + s] =
        (DIR < 0 && a.mirror && mirror_plane(kx0 + s, g.nx)) ? hermitian(A, y, q, nseq, ny) : A[t];
  }
}

// Consecutive blocks are dealt round-robin to the 8 XCDs, each with its own L2.  Re-index the
// grid so that the blocks one XCD receives are consecutive in (x, y, z): neighbouring kx tiles of
// a spectrum row, which share 128-byte lines when a tile is not a whole number of lines, then run
// on the same XCD close in time and meet in its L2.  For any number of blocks: left in the hardware's order
// where it is no multiple of 8, the passes with one-bin tiles paid for it in every line (outer passes of the
// CG on displacements, small strain 32 x 36 x 32, 612 blocks: 11.3 + 14.6 us, now 9.0 + 10.4, with 544 blocks
// at 32^3 8.6 + 9.6; 36^3, 684 blocks, 13.3 + 16.2, now 10.5 + 12.0).
__device__ __forceinline__ void xcd_blocks(unsigned* bx, unsigned* by, unsigned* bz) {
  const unsigned l2 = xcd_order(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z),
                                gridDim.x * gridDim.y * gridDim.z);
  *bx = l2 % gridDim.x;
  *by = (l2 / gridDim.x) % gridDim.y;
  *bz = l2 / (gridDim.x * gridDim.y);
}

// ============================================================================
// outer-axis pass with the projection G-hat (section 3)
// ============================================================================
__device__ __forceinline__ double signed_freq(int k, int n, double scale) {
  if (2 * k < n) return k * scale;
  if (2 * k == n) return 0.0;  // Nyquist: zero wavevector component
  return (k - n) * scale;
}

// finite strain: A -> (A n) (x) n on row-major d x d tensors
template <int D>
__device__ __forceinline__ void project_finite(double2* v, const double* nv) {
  double2 an[D];
#pragma unroll
  for (int i = 0; i < D; ++i) {
    an[i] = make_double2(0.0, 0.0);
#pragma unroll
    for (int j = 0; j < D; ++j) {
      an[i].x += v[i * D + j].x * nv[j];
      an[i].y += v[i * D + j].y * nv[j];
    }
  }
#pragma unroll
  for (int i = 0; i < D; ++i)
#pragma unroll
    for (int j = 0; j < D; ++j) v[i * D + j] = make_double2(an[i].x * nv[j], an[i].y * nv[j]);
}

// small strain, Mandel packed: A -> n (x) (A n) + (A n) (x) n - (n.A.n) n (x) n
template <int D>
__device__ __forceinline__ void project_small(double2* v, const double* nv) {
  const double r2 = 1.41421356237309504880;
  const double h2 = 0.70710678118654752440;
  double2 T[D][D];
  if (D == 3) {
    T[0][0] = v[0]; T[1][1] = v[1]; T[2][2] = v[2];
    T[1][2] = T[2][1] = make_double2(h2 * v[3].x, h2 * v[3].y);
    T[0][2] = T[2][0] = make_double2(h2 * v[4].x, h2 * v[4].y);
    T[0][1] = T[1][0] = make_double2(h2 * v[5].x, h2 * v[5].y);
  } else {
    T[0][0] = v[0]; T[1][1] = v[1];
    T[0][1] = T[1][0] = make_double2(h2 * v[2].x, h2 * v[2].y);
  }
  double2 an[D];
#pragma unroll
  for (int i = 0; i < D; ++i) {
    an[i] = make_double2(0.0, 0.0);
#pragma unroll
    for (int j = 0; j < D; ++j) {
      an[i].x += T[i][j].x * nv[j];
      an[i].y += T[i][j].y * nv[j];
    }
  }
  double2 s = make_double2(0.0, 0.0);
#pragma unroll
  for (int i = 0; i < D; ++i) {
    s.x += nv[i] * an[i].x;
    s.y += nv[i] * an[i].y;
  }
  auto o = [&](int i, int j) {
    return make_double2(an[i].x * nv[j] + nv[i] * an[j].x - s.x * nv[i] * nv[j],
                        an[i].y * nv[j] + nv[i] * an[j].y - s.y * nv[i] * nv[j]);
  };
  if (D == 3) {
    v[0] = o(0, 0); v[1] = o(1, 1); v[2] = o(2, 2);
    double2 t;
    t = o(1, 2); v[3] = make_double2(r2 * t.x, r2 * t.y);
    t = o(0, 2); v[4] = make_double2(r2 * t.x, r2 * t.y);
    t = o(0, 1); v[5] = make_double2(r2 * t.x, r2 * t.y);
  } else {
    v[0] = o(0, 0); v[1] = o(1, 1);
    const double2 t = o(0, 1);
    v[2] = make_double2(r2 * t.x, r2 * t.y);
  }
}

// Finite strain projects each row of F on its own ((A n)_i n_j involves only
// row i), so a block transforms the NDIM components of one row; small strain
// couples all C Mandel components.  LDS layout: element o of sequence (jj, s)
// at D[o * nseq + jj * tw + s], nseq = G * tw, one FFT call for all of them.
template <int MODE, int SMALL, int NDIM, int NF = 0>
// uncapped: a 5-wave cap spilled 87 VGPRs in the small-strain projection (256-cell job 2 % slower)
__global__ void __launch_bounds__(kThreads) k_outer(AxisArgs a) {
  constexpr int C = SMALL ? (NDIM == 3 ? 6 : 3) : (NDIM == 3 ? 9 : 4);
  constexpr int G = SMALL ? C : NDIM;
  constexpr int NGRP = C / G;
  const Geom& g = a.g;
  unsigned bx, by, bz;
  xcd_blocks(&bx, &by, &bz);
  const int vb = bz / NGRP;
  const int grp = bz - vb * NGRP;
  const int b = a.active ? a.active[vb] : vb;
  if (a.st != nullptr && a.st[b].status != CG_RUNNING) return;
  if (MODE == OUTER_PROJECT && a.pq_st != nullptr && bx == 0 && by == 0 && grp == 0) {
    // <p, K:p> and alpha of right-hand side b, summed in a fixed order; nothing in this
    // pass reads them (the inverse x pass does)
    __shared__ double red[kThreads / 64];
    const double s = block_sum(strided_sum<8, kThreads>(a.pq_partials + (long long)b * a.pq_nblocks, a.pq_nblocks), red);
    if (threadIdx.x == 0) cg_finalize<RED_PQ>(a.pq_st[b], s);
  }
  const int kx0 = bx * a.TX;
  const int tw = kx_tile_width(g.nxh, a.TX, (int)bx);
  const int mid = by;
  const int n = g.n_outer;
  const int nseq = G * tw;
  const int cnt = n * nseq;
  extern __shared__ double2 smem[];
  double2* D = smem;
  double2* pong = smem + (size_t)g.lo * nseq;
  const long long ostride = (long long)g.n_mid * g.nxp;
  const long long base0 = (long long)mid * g.nxp + kx0;
  const long long cbase = ((long long)b * C + grp * G) * g.Nh;

  const FastDiv fdq = make_fastdiv((unsigned)nseq);
  const FastDiv fdt = make_fastdiv((unsigned)tw);
  for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
    const int o = (int)fdiv((unsigned)t, fdq);
    const int rem = t - o * nseq;
    const int jj = (int)fdiv((unsigned)rem, fdt);
    const int s = rem - jj * tw;
    D[t] = a.spec[cbase + (long long)jj * g.Nh + base0 + o * ostride + s];
  }
  __syncthreads();

  if (MODE != OUTER_INV) pass_fft<-1, NF>(D, pong, nseq, a.pl, a.inplace);

  if (MODE == OUTER_PROJECT) {
    for (int t = threadIdx.x; t < n * tw; t += blockDim.x) {
      const int o = (int)fdiv((unsigned)t, fdt);
      const int s = t - o * tw;
      double xi[NDIM];
      xi[0] = signed_freq(kx0 + s, g.nx, g.ks[0]);
      if (NDIM == 3) {
        xi[1] = signed_freq(mid, g.ny, g.ks[1]);
        xi[NDIM - 1] = signed_freq(o, g.nz, g.ks[2]);
      } else {
        xi[1] = signed_freq(o, g.ny, g.ks[1]);
      }
      double nrm2 = 0.0;
#pragma unroll
      for (int i = 0; i < NDIM; ++i) nrm2 += xi[i] * xi[i];
      double2 v[G];
      const int e0 = o * nseq + s;
      if (nrm2 > 0.0) {
        const double inv = 1.0 / sqrt(nrm2);
        double nv[NDIM];
#pragma unroll
        for (int i = 0; i < NDIM; ++i) nv[i] = xi[i] * inv;
#pragma unroll
        for (int jj = 0; jj < G; ++jj) v[jj] = D[e0 + jj * tw];
        if (SMALL) {
          project_small<NDIM>(v, nv);
        } else {
          // one row of F: (sum_j A_j n_j) n
          double2 an = make_double2(0.0, 0.0);
#pragma unroll
          for (int jj = 0; jj < G; ++jj) {
            an.x += v[jj].x * nv[jj];
            an.y += v[jj].y * nv[jj];
          }
#pragma unroll
          for (int jj = 0; jj < G; ++jj) v[jj] = make_double2(an.x * nv[jj], an.y * nv[jj]);
        }
      } else {
#pragma unroll
        for (int jj = 0; jj < G; ++jj) v[jj] = make_double2(0.0, 0.0);
      }
#pragma unroll
      for (int jj = 0; jj < G; ++jj) D[e0 + jj * tw] = v[jj];
    }
    __syncthreads();
  }

  if (MODE != OUTER_FWD) pass_fft<+1, NF>(D, pong, nseq, a.pl, a.inplace);

  for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
    const int o = (int)fdiv((unsigned)t, fdq);
    const int rem = t - o * nseq;
    const int jj = (int)fdiv((unsigned)rem, fdt);
    const int s = rem - jj * tw;
    a.spec[cbase + (long long)jj * g.Nh + base0 + o * ostride + s] = D[t];
  }
}

// ============================================================================
// finite strain, 3D: the projection chain row by row
// ============================================================================
// G-hat maps a row a_i = (a_i0, a_i1, a_i2) of A-hat to s_i xi with s_i = (a_i . xi) / |xi|^2
// ((A n) (x) n with n = xi / |xi|).  xi_x depends only on kx and xi_y only on ky, so both factors
// commute with the transforms along the other axes: the forward y pass already combines
// v_i = xi_x a_i0 + xi_y a_i1 (w_i = a_i2 stays), the outer pass reads two components per row,
// forms s_i = (v_i + xi_z w_i) / |xi|^2 and writes back s_i and xi_z s_i, and the inverse y pass
// expands them to xi_x s_i, xi_y s_i, xi_z s_i.  The y and outer passes then move 15 + 12 + 15
// instead of 18 + 18 + 18 component transfers per wavevector, and the outer pass transforms
// 2 instead of 3 columns per row.  Slots: (i,0) carries v_i / s_i, (i,2) carries w_i / xi_z s_i.

// y pass of row i = blockIdx.z mod 3 over a tile of TX bins and ZB planes, one component tile in
// LDS at a time (the LDS and occupancy of a plain y pass); what the next phase combines is held in
// registers, at most kFrowHeld elements per thread (the host keeps ny * TX * ZB <= kFrowHeld * 256).
// Element y of sequence q = zz * tw + s at A[y * nseq + q]; thread t owns elements t + e * 256.
//   DIR = -1: Y a_i0 -> held = xi_x Y a_i0;  Y a_i1 -> slot (i,0) = held + xi_y Y a_i1;
//             Y a_i2 -> slot (i,2)
//   DIR = +1: slot (i,0) = u -> held = xi_y u, Y^-1 u -> slot (i,0) = xi_x Y^-1 u;
//             Y^-1 held -> slot (i,1);  slot (i,2) = w -> Y^-1 w -> slot (i,2)

template <int DIR, int NF>
// 4 waves per SIMD (at most 128 VGPRs; 157 unconstrained): measured 15 % faster at 128^3
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(NF == kDense ? 3 : 4, 8))) k_mid_frow(AxisArgs a) {
  const Geom& g = a.g;
  unsigned bx, by, bz;
  xcd_blocks(&bx, &by, &bz);
  const int vb = bz / 3;
  const int row = bz - vb * 3;
  const int b = a.active ? a.active[vb] : vb;
  if (a.st != nullptr && a.st[b].status != CG_RUNNING) return;
  if (DIR < 0 && a.pq_st != nullptr && bx == 0 && by == 0 && row == 0) reduce_alpha(a, b);
  const int kx0 = bx * a.TX;
  const int tw = kx_tile_width(g.nxh, a.TX, bx);
  const int ny = g.ny;
  const int z0 = by * a.ZB;
  const int nseq = min(a.ZB, g.nz - z0) * tw;
  const int cnt = ny * nseq;
  extern __shared__ double2 smem[];
  double2* A = smem;
  double2* Bf = smem + (size_t)g.lm * nseq;
  const long long cbase = ((long long)b * 9 + row * 3) * g.Nh + (long long)z0 * ny * g.nxp + kx0;
  const FastDiv fdq = make_fastdiv((unsigned)nseq);
  const FastDiv fdt = make_fastdiv((unsigned)tw);
  // global offset (within a component) and wavevector components of element t
  auto where = [&](int t, long long* off, double* xx, double* xy) {
    const int y = (int)fdiv((unsigned)t, fdq);
    const int q = t - y * nseq;
    const int zz = (int)fdiv((unsigned)q, fdt);
    const int sx = q - zz * tw;
    *off = (long long)(zz * ny + y) * g.nxp + sx;
    *xx = signed_freq(kx0 + sx, g.nx, g.ks[0]);
    *xy = signed_freq(y, ny, g.ks[1]);
  };
  // transformed entry t; on a mirror plane (xi_x = 0) made Hermitian
  auto value = [&](int t, double xx) {
    if (DIR > 0 || !a.mirror || xx != 0.0) return A[t];
    const int y = (int)fdiv((unsigned)t, fdq);
    return hermitian(A, y, t - y * nseq, nseq, ny);
  };
  auto load = [&](int slot) {
    for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
      long long off;
      double xx, xy;
      where(t, &off, &xx, &xy);
      A[t] = a.spec[cbase + slot * g.Nh + off];
    }
  };
  auto store = [&](int slot) {
    for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
      long long off;
      double xx, xy;
      where(t, &off, &xx, &xy);
      a.spec[cbase + slot * g.Nh + off] = value(t, xx);
    }
  };
  double2 held[kFrowHeld];
  if (DIR < 0) {
    load(0);
    __syncthreads();
    pass_fft<-1, NF>(A, Bf, nseq, a.pl, a.inplace);
#pragma unroll
    for (int e = 0; e < kFrowHeld; ++e) {
      const int t = threadIdx.x + e * blockDim.x;
      if (t < cnt) {
        long long off;
        double xx, xy;
        where(t, &off, &xx, &xy);
        held[e] = make_double2(xx * A[t].x, xx * A[t].y);
      }
    }
    __syncthreads();
    load(1);
    __syncthreads();
    pass_fft<-1, NF>(A, Bf, nseq, a.pl, a.inplace);
#pragma unroll
    for (int e = 0; e < kFrowHeld; ++e) {
      const int t = threadIdx.x + e * blockDim.x;
      if (t < cnt) {
        long long off;
        double xx, xy;
        where(t, &off, &xx, &xy);
        const double2 v = value(t, xx);
        a.spec[cbase + off] = make_double2(held[e].x + xy * v.x, held[e].y + xy * v.y);
      }
    }
    __syncthreads();
    load(2);
    __syncthreads();
    pass_fft<-1, NF>(A, Bf, nseq, a.pl, a.inplace);
    store(2);
  } else {
#pragma unroll
    for (int e = 0; e < kFrowHeld; ++e) {
      const int t = threadIdx.x + e * blockDim.x;
      if (t < cnt) {
        long long off;
        double xx, xy;
        where(t, &off, &xx, &xy);
        const double2 u = a.spec[cbase + off];
        A[t] = u;
        held[e] = make_double2(xy * u.x, xy * u.y);
      }
    }
    __syncthreads();
    pass_fft<1, NF>(A, Bf, nseq, a.pl, a.inplace);
    for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
      long long off;
      double xx, xy;
      where(t, &off, &xx, &xy);
      a.spec[cbase + off] = make_double2(xx * A[t].x, xx * A[t].y);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kFrowHeld; ++e) {
      const int t = threadIdx.x + e * blockDim.x;
      if (t < cnt) A[t] = held[e];
    }
    __syncthreads();
    pass_fft<1, NF>(A, Bf, nseq, a.pl, a.inplace);
    store(1);
    __syncthreads();
    load(2);
    __syncthreads();
    pass_fft<1, NF>(A, Bf, nseq, a.pl, a.inplace);
    store(2);
  }
}

// Outer (z) pass of the row-wise projection: row i = blockIdx.z mod 3 (after the XCD-aware
// re-indexing), slots (i,0) = v and (i,2) = w of TX bins at one ky.  LDS: element o of sequence
// (jj, s) at D[o * 2 tw + jj * tw + s].
template <int NF>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(NF == kDense ? 3 : 5, 8))) k_outer_frow(AxisArgs a) {
  const Geom& g = a.g;
  unsigned bx, by, bz;
  xcd_blocks(&bx, &by, &bz);
  const int vb = bz / 3;
  const int row = bz - vb * 3;
  const int b = a.active ? a.active[vb] : vb;
  if (a.st != nullptr && a.st[b].status != CG_RUNNING) return;
  if (a.pq_st != nullptr && bx == 0 && by == 0 && row == 0) {
    // <p, K:p> and alpha of right-hand side b, summed in a fixed order (read by the inverse x pass)
    __shared__ double red[kThreads / 64];
    const double sum = block_sum(strided_sum<8, kThreads>(a.pq_partials + (long long)b * a.pq_nblocks, a.pq_nblocks), red);
    if (threadIdx.x == 0) cg_finalize<RED_PQ>(a.pq_st[b], sum);
  }
  const int kx0 = bx * a.TX;
  const int tw = kx_tile_width(g.nxh, a.TX, (int)bx);
  const int mid = by;
  const int n = g.nz;
  const int nseq = 2 * tw;
  const int cnt = n * nseq;
  extern __shared__ double2 smem[];
  double2* D = smem;
  double2* pong = smem + (size_t)g.lo * nseq;
  const long long ostride = (long long)g.ny * g.nxp;
  const long long cbase = ((long long)b * 9 + row * 3) * g.Nh + (long long)mid * g.nxp + kx0;
  const FastDiv fdq = make_fastdiv((unsigned)nseq);
  const FastDiv fdt = make_fastdiv((unsigned)tw);
  for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
    const int o = (int)fdiv((unsigned)t, fdq);
    const int rem = t - o * nseq;
    const int jj = (int)fdiv((unsigned)rem, fdt);
    const int sx = rem - jj * tw;
    D[t] = a.spec[cbase + 2 * jj * g.Nh + o * ostride + sx];
  }
  __syncthreads();
  pass_fft<-1, NF>(D, pong, nseq, a.pl, a.inplace);
  const double xy = signed_freq(mid, g.ny, g.ks[1]);
  for (int t = threadIdx.x; t < n * tw; t += blockDim.x) {
    const int o = (int)fdiv((unsigned)t, fdt);
    const int sx = t - o * tw;
    const double xx = signed_freq(kx0 + sx, g.nx, g.ks[0]);
    const double xz = signed_freq(o, n, g.ks[2]);
    const double nrm2 = xx * xx + xy * xy + xz * xz;
    const int e0 = o * nseq + sx;
    double2 sv = make_double2(0.0, 0.0);
    if (nrm2 > 0.0) {
      const double inv = 1.0 / nrm2;
      const double2 v = D[e0];
      const double2 w = D[e0 + tw];
      sv = make_double2((v.x + xz * w.x) * inv, (v.y + xz * w.y) * inv);
    }
    D[e0] = sv;
    D[e0 + tw] = make_double2(xz * sv.x, xz * sv.y);
  }
  __syncthreads();
  pass_fft<1, NF>(D, pong, nseq, a.pl, a.inplace);
  for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
    const int o = (int)fdiv((unsigned)t, fdq);
    const int rem = t - o * nseq;
    const int jj = (int)fdiv((unsigned)rem, fdt);
    const int sx = rem - jj * tw;
    a.spec[cbase + 2 * jj * g.Nh + o * ostride + sx] = D[t];
  }
}

// ============================================================================
// outer-axis passes of the CG on displacements (3D)
// ============================================================================
// Bins (kx0 + s, ky, kz) of a block: TX bins of kx at one ky along the whole outer axis.
// LDS: element o of sequence (jj, s) at D[o * nseq + jj * tw + s].
// Finite strain: a block takes one row i of F, whose spectrum arrives (and leaves) as two sequences
// per bin: v_i = xi_x a_i0 + xi_y a_i1 and w_i = a_i2 in the slots (i,0) and (i,2) of the row-wise
// y pass.  Small strain: all six components.
// Bound by HBM, the CG's vector updates being done here on one component per row of F (128^3: forward
// 96 B per voxel, 53 us; inverse 168 B, 73 us); the projection pass on strain fields (96 B, 51 us)
// leaves them to the x passes, on nine components each.  Small strain, 6 right-hand sides at 64^3: 18
// and 26 us.
template <int SMALL>
struct OuterTile {
  static constexpr int NDIM = 3;
  static constexpr int C = SMALL ? 6 : 9;
  static constexpr int G = SMALL ? C : 2;         // sequences per bin
  static constexpr int NGRP = SMALL ? 1 : NDIM;   // blocks per bin tile
  static constexpr int DU = SMALL ? NDIM : 1;     // displacement components per block
  int b, grp, kx0, tw, ky, n, nseq, part;
  long long ostride, spec0, u0;
  FastDiv fdq, fdt;

  __device__ __forceinline__ OuterTile(const AxisArgs& a) {
    const Geom& g = a.g;
    unsigned bx, by, bz;
    xcd_blocks(&bx, &by, &bz);
    const int vb = bz / NGRP;
    grp = bz - vb * NGRP;
    b = a.active ? a.active[vb] : vb;
    kx0 = bx * a.TX;
    tw = kx_tile_width(g.nxh, a.TX, (int)bx);
    ky = by;
    n = g.n_outer;
    nseq = G * tw;
    part = bx + gridDim.x * (by + gridDim.y * grp);
    ostride = (long long)g.n_mid * g.nxp;
    const long long base = (long long)ky * g.nxp + kx0;
    spec0 = ((long long)b * C + (SMALL ? 0 : grp * NDIM)) * g.Nh + base;
    u0 = ((long long)b * NDIM + grp) * g.Nh + base;
    fdq = make_fastdiv((unsigned)nseq);
    fdt = make_fastdiv((unsigned)tw);
  }
  // spectrum offset of LDS entry t, its sequence jj and bin s
  __device__ __forceinline__ long long spec_at(const Geom& g, int t, int* jj, int* s) const {
    const int o = (int)fdiv((unsigned)t, fdq);
    const int rem = t - o * nseq;
    *jj = (int)fdiv((unsigned)rem, fdt);
    *s = rem - *jj * tw;
    const int slot = SMALL ? *jj : 2 * *jj;
    return spec0 + slot * g.Nh + o * ostride + *s;
  }
  // bin t of the block's n * tw: outer index o, bin s, displacement offset, wavevector
  __device__ __forceinline__ void bin(const Geom& g, int t, int* po, int* ps, long long* uo, double* xi) const {
    const int o = (int)fdiv((unsigned)t, fdt);
    const int s = t - o * tw;
    *po = o;
    *ps = s;
    *uo = u0 + o * ostride + s;
    xi[0] = signed_freq(kx0 + s, g.nx, g.ks[0]);
    xi[1] = signed_freq(ky, g.ny, g.ks[1]);
    xi[2] = signed_freq(o, g.nz, g.ks[2]);
  }
};

// Forward: outer-axis FFT of tau-hat, its displacement u, r -= alpha u (a.mode OUTER_CGFWD), or
// r = -u (OUTER_RHS); partial <r, r>.  Reads the spectrum once and reads and writes r.
template <int SMALL, int NF>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(NF > 0 && !SMALL ? 5 : 2, 8))) k_ofwd(AxisArgs a) {
  typedef OuterTile<SMALL> Tile;
  constexpr int NDIM = 3, G = Tile::G, DU = Tile::DU;
  const Geom& g = a.g;
  const Tile T(a);
  const bool cg = a.mode == OUTER_CGFWD;
  if (cg && a.st[T.b].status != CG_RUNNING) return;
  extern __shared__ double2 smem[];
  double2* D = smem;
  double2* pong = smem + (size_t)g.lo * T.nseq;
  __shared__ double red[kThreads / 64];
  const double alpha = cg ? a.st[T.b].alpha : 0.0;
  const int cnt = T.n * T.nseq;
  // a mirror plane's sequence at ky is the conjugate of the one at ny - ky (minus it for v, which
  // carries xi_y): beyond ny / 2 the latter is transformed and the result mirrored below
  const bool mirror = 2 * T.ky > g.ny;
  gather_staged<4>(D, cnt, [&](int t) {
    int jj, s;
    double2 v = a.spec[T.spec_at(g, t, &jj, &s)];
    if (mirror && mirror_plane(T.kx0 + s, g.nx)) v = (!SMALL && jj == 0) ? make_double2(-v.x, v.y) : make_double2(v.x, -v.y);
    return v;
  });
  __syncthreads();
  pass_fft<-1, NF>(D, pong, T.nseq, a.pl, a.inplace);
  double acc = 0.0;
  for (int t = threadIdx.x; t < T.n * T.tw; t += blockDim.x) {
    int o, s;
    long long uo;
    double xi[NDIM];
    T.bin(g, t, &o, &s, &uo, xi);
    const bool edge = mirror_plane(T.kx0 + s, g.nx);
    const bool flip = mirror && edge;              // take the mirror image of row n - o
    const bool self = edge && !flip && (T.ky == 0 || 2 * T.ky == g.ny);
    const int row = flip && o > 0 ? T.n - o : o;
    if (flip) {
#pragma unroll
      for (int i = 0; i < NDIM; ++i) xi[i] = -xi[i];
    }
    auto value = [&](int jj) {
      return self ? hermitian(D, row, jj * T.tw + s, T.nseq, T.n) : D[row * T.nseq + jj * T.tw + s];
    };
    double2 r[DU];
#pragma unroll
    for (int i = 0; i < DU; ++i) r[i] = cg ? ld_vec(a.ru + uo + i * g.Nh, a.stream) : make_double2(0.0, 0.0);
    double n2 = 0.0;
#pragma unroll
    for (int i = 0; i < NDIM; ++i) n2 += xi[i] * xi[i];
    double2 u[DU];
#pragma unroll
    for (int i = 0; i < DU; ++i) u[i] = make_double2(0.0, 0.0);
    if (n2 > 0.0) {
      const double inv = 1.0 / n2;
      if constexpr (SMALL) {
        const double h2 = 0.70710678118654752440;
        double2 v[G];
#pragma unroll
        for (int j = 0; j < G; ++j) v[j] = value(j);
        double2 t3[NDIM];
        t3[0] = make_double2(v[0].x * xi[0] + h2 * (v[5].x * xi[1] + v[4].x * xi[2]), v[0].y * xi[0] + h2 * (v[5].y * xi[1] + v[4].y * xi[2]));
        t3[1] = make_double2(v[1].x * xi[1] + h2 * (v[5].x * xi[0] + v[3].x * xi[2]), v[1].y * xi[1] + h2 * (v[5].y * xi[0] + v[3].y * xi[2]));
        t3[2] = make_double2(v[2].x * xi[2] + h2 * (v[4].x * xi[0] + v[3].x * xi[1]), v[2].y * xi[2] + h2 * (v[4].y * xi[0] + v[3].y * xi[1]));
        double2 d = make_double2(0.0, 0.0);
#pragma unroll
        for (int i = 0; i < NDIM; ++i) {
          d.x += xi[i] * t3[i].x;
          d.y += xi[i] * t3[i].y;
        }
        d = cscale(d, inv);
#pragma unroll
        for (int i = 0; i < NDIM; ++i)
          u[i] = make_double2((2.0 * t3[i].x - d.x * xi[i]) * inv, (2.0 * t3[i].y - d.y * xi[i]) * inv);
      } else {
        const double2 v = value(0);
        const double2 w = value(1);
        u[0] = make_double2((v.x + xi[2] * w.x) * inv, (v.y + xi[2] * w.y) * inv);
      }
    }
    if (flip) {  // u at -xi is -conj of u at xi
#pragma unroll
      for (int i = 0; i < DU; ++i) u[i].x = -u[i].x;
    }
    double nrm = 0.0;
    double2 d = make_double2(0.0, 0.0);
#pragma unroll
    for (int i = 0; i < DU; ++i) {
      if (cg) r[i] = make_double2(r[i].x - alpha * u[i].x, r[i].y - alpha * u[i].y);
      else r[i] = make_double2(-u[i].x, -u[i].y);
      st_vec(a.ru + uo + i * g.Nh, r[i], a.stream);
      nrm += n2 * (r[i].x * r[i].x + r[i].y * r[i].y);
      if (SMALL) {
        d.x += xi[i] * r[i].x;
        d.y += xi[i] * r[i].y;
      }
    }
    if (SMALL) nrm = 0.5 * (nrm + d.x * d.x + d.y * d.y);
    acc += edge ? nrm : 2.0 * nrm;
  }
  const double sum = block_sum(acc, red);
  if (threadIdx.x == 0) a.rr_partials[(long long)T.b * a.rr_nblocks + T.part] = sum * a.inv_n;
}

// Inverse: a displacement per bin, its strain in the form the inverse passes take, inverse outer-axis
// FFT.  a.mode OUTER_CGINV: x += alpha p, p = r + beta p, the strain of p (first iteration: x = 0, p = r);
// OUTER_SOLUTION: the strain of x + alpha p (zero if no iteration was done); OUTER_RESIDUAL: of r.
template <int SMALL, int NF>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(NF > 0 && !SMALL ? 5 : 2, 8))) k_oinv(AxisArgs a) {
  typedef OuterTile<SMALL> Tile;
  constexpr int NDIM = 3, G = Tile::G, DU = Tile::DU;
  const Geom& g = a.g;
  const Tile T(a);
  const CgState& S = a.st[T.b];
  if (a.mode == OUTER_CGINV && S.status != CG_RUNNING) return;
  const double alpha = S.alpha, beta = S.beta;
  const bool first = S.first;
  // the last update of x is still to be made for a solve that stopped after an iteration
  const bool some = S.iters >= 1;
  const bool last = some && (S.status == CG_CONVERGED || S.status == CG_MAXIT);
  extern __shared__ double2 smem[];
  double2* D = smem;
  double2* pong = smem + (size_t)g.lo * T.nseq;
  for (int t = threadIdx.x; t < T.n * T.tw; t += blockDim.x) {
    int o, s;
    long long uo;
    double xi[NDIM];
    T.bin(g, t, &o, &s, &uo, xi);
    const int e0 = o * T.nseq + s;
    double2 u[DU];
    if (a.mode == OUTER_CGINV) {
      double2 po[DU], xo[DU];
#pragma unroll
      for (int i = 0; i < DU; ++i) {
        u[i] = ld_vec(a.ru + uo + i * g.Nh, a.stream);
        if (!first) {
          po[i] = ld_vec(a.pu + uo + i * g.Nh, a.stream);
          xo[i] = ld_vec(a.xu + uo + i * g.Nh, a.stream);
        }
      }
#pragma unroll
      for (int i = 0; i < DU; ++i) {
        double2 x = make_double2(0.0, 0.0);
        if (!first) {
          x = make_double2(xo[i].x + alpha * po[i].x, xo[i].y + alpha * po[i].y);
          u[i] = make_double2(u[i].x + beta * po[i].x, u[i].y + beta * po[i].y);
        }
        st_vec(a.xu + uo + i * g.Nh, x, a.stream);
        st_vec(a.pu + uo + i * g.Nh, u[i], a.stream);
      }
    } else {
#pragma unroll
      for (int i = 0; i < DU; ++i) {
        u[i] = make_double2(0.0, 0.0);
        if (a.mode == OUTER_RESIDUAL) {
          u[i] = a.ru[uo + i * g.Nh];
        } else if (some) {
          u[i] = a.xu[uo + i * g.Nh];
          if (last) {
            const double2 p = a.pu[uo + i * g.Nh];
            u[i] = make_double2(u[i].x + alpha * p.x, u[i].y + alpha * p.y);
          }
        }
      }
    }
    if constexpr (SMALL) {
      const double h2 = 0.70710678118654752440;
      double2 v[G];
#pragma unroll
      for (int i = 0; i < NDIM; ++i) v[i] = cscale(u[i], xi[i]);
      // sqrt(2) times half the symmetrised product
      auto shear = [&](int i, int j) {
        return make_double2(h2 * (u[i].x * xi[j] + u[j].x * xi[i]), h2 * (u[i].y * xi[j] + u[j].y * xi[i]));
      };
      v[3] = shear(1, 2);
      v[4] = shear(0, 2);
      v[5] = shear(0, 1);
#pragma unroll
      for (int j = 0; j < G; ++j) D[e0 + j * T.tw] = v[j];
    } else {
      // the inverse y pass multiplies by xi_x and xi_y
      D[e0] = u[0];
      D[e0 + T.tw] = cscale(u[0], xi[2]);
    }
  }
  __syncthreads();
  pass_fft<+1, NF>(D, pong, T.nseq, a.pl, a.inplace);
  const int cnt = T.n * T.nseq;
  for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
    int jj, s;
    a.spec[T.spec_at(g, t, &jj, &s)] = D[t];
  }
}

// ============================================================================
// launches of the pass kernels with FFT variant NF (grid and LDS bytes from the caller)
// ============================================================================
template <int NF>
hipError_t dispatch_xinv(int cons, const XInvArgs& a, dim3 grid, size_t sm, hipStream_t s) {
#define FH_L(CC)                                                                                              \
  switch (cons) {                                                                                             \
    case CONS_IDENT: hipLaunchKernelGGL((k_xinv<CONS_IDENT, CC, NF>), grid, dim3(kThreads), sm, s, a); break; \
    case CONS_RHS: hipLaunchKernelGGL((k_xinv<CONS_RHS, CC, NF>), grid, dim3(kThreads), sm, s, a); break;     \
    case CONS_CGUPD: hipLaunchKernelGGL((k_xinv<CONS_CGUPD, CC, NF>), grid, dim3(kThreads), sm, s, a); break; \
    default: return hipErrorInvalidValue;                                                                     \
  }
  switch (a.g.c) {
    case 3: FH_L(3); break;
    case 4: FH_L(4); break;
    case 6: FH_L(6); break;
    case 9: FH_L(9); break;
    default: return hipErrorInvalidValue;
  }
#undef FH_L
  return hipGetLastError();
}

// rows: the row-wise finite-strain y pass of the projection chain
template <int NF>
hipError_t dispatch_mid(int dir, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  if (rows) {
    if (dir < 0) hipLaunchKernelGGL((k_mid_frow<-1, NF>), grid, dim3(kThreads), sm, s, a);
    else hipLaunchKernelGGL((k_mid_frow<1, NF>), grid, dim3(kThreads), sm, s, a);
  } else {
    if (dir < 0) hipLaunchKernelGGL((k_mid<-1, NF>), grid, dim3(kThreads), sm, s, a);
    else hipLaunchKernelGGL((k_mid<1, NF>), grid, dim3(kThreads), sm, s, a);
  }
  return hipGetLastError();
}

// the outer passes of the CG on displacements
template <int NF, int SMALL>
hipError_t dispatch_outer_cg(bool inverse, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  if (inverse) hipLaunchKernelGGL((k_oinv<SMALL, NF>), grid, dim3(kThreads), sm, s, a);
  else hipLaunchKernelGGL((k_ofwd<SMALL, NF>), grid, dim3(kThreads), sm, s, a);
  return hipGetLastError();
}

template <int NF>
hipError_t dispatch_outer_cg(int mode, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  const bool inv = mode != OUTER_CGFWD && mode != OUTER_RHS;
  return a.g.small ? dispatch_outer_cg<NF, 1>(inv, a, grid, sm, s) : dispatch_outer_cg<NF, 0>(inv, a, grid, sm, s);
}

// rows: the row-wise finite-strain projection (3D)
template <int NF>
hipError_t dispatch_outer(int mode, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s) {
  if (rows) {
    hipLaunchKernelGGL((k_outer_frow<NF>), grid, dim3(kThreads), sm, s, a);
    return hipGetLastError();
  }
#define FH_L(SM, D)                                                                                                  \
  switch (mode) {                                                                                                    \
    case OUTER_PROJECT: hipLaunchKernelGGL((k_outer<OUTER_PROJECT, SM, D, NF>), grid, dim3(kThreads), sm, s, a); break; \
    case OUTER_FWD: hipLaunchKernelGGL((k_outer<OUTER_FWD, SM, D, NF>), grid, dim3(kThreads), sm, s, a); break;         \
    case OUTER_INV: hipLaunchKernelGGL((k_outer<OUTER_INV, SM, D, NF>), grid, dim3(kThreads), sm, s, a); break;         \
    default: return hipErrorInvalidValue;                                                                            \
  }
  if (a.g.small) {
    if (a.g.ndim == 3) { FH_L(1, 3) } else { FH_L(1, 2) }
  } else {
    if (a.g.ndim == 3) { FH_L(0, 3) } else { FH_L(0, 2) }
  }
#undef FH_L
  return hipGetLastError();
}

// Dynamic-LDS limits of the pass kernels of variant NF that a grid of this kind launches (the x passes
// with a law: xpass_law.h).
template <typename Fn>
hipError_t raise_limit(Fn* fn, size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}
template <int NF, int SMALL>
hipError_t outer_cg_limits(size_t bytes) {
  hipError_t e = raise_limit(k_ofwd<SMALL, NF>, bytes);
  return e == hipSuccess ? raise_limit(k_oinv<SMALL, NF>, bytes) : e;
}
template <int NF>
hipError_t outer_cg_limits(const Geom& g, size_t bytes) {
  return g.small ? outer_cg_limits<NF, 1>(bytes) : outer_cg_limits<NF, 0>(bytes);
}
template <int NF, int SMALL, int NDIM>
hipError_t outer_limits(size_t bytes) {
  hipError_t e = raise_limit(k_outer<OUTER_PROJECT, SMALL, NDIM, NF>, bytes);
  if (e == hipSuccess) e = raise_limit(k_outer<OUTER_FWD, SMALL, NDIM, NF>, bytes);
  if (e == hipSuccess) e = raise_limit(k_outer<OUTER_INV, SMALL, NDIM, NF>, bytes);
  return e;
}
template <int NF>
hipError_t outer_limits(const Geom& g, size_t bytes) {
  hipError_t e = raise_limit(k_outer_frow<NF>, bytes);
  if (e != hipSuccess) return e;
  if (g.small) return g.ndim == 3 ? outer_limits<NF, 1, 3>(bytes) : outer_limits<NF, 1, 2>(bytes);
  return g.ndim == 3 ? outer_limits<NF, 0, 3>(bytes) : outer_limits<NF, 0, 2>(bytes);
}
template <int NF>
hipError_t mid_limits(size_t bytes) {
  hipError_t e = raise_limit(k_mid<-1, NF>, bytes);
  if (e == hipSuccess) e = raise_limit(k_mid<1, NF>, bytes);
  if (e == hipSuccess) e = raise_limit(k_mid_frow<-1, NF>, bytes);
  if (e == hipSuccess) e = raise_limit(k_mid_frow<1, NF>, bytes);
  return e;
}
template <int NF, int C>
hipError_t xinv_limits(size_t bytes) {
  hipError_t e = raise_limit(k_xinv<CONS_IDENT, C, NF>, bytes);
  if (e == hipSuccess) e = raise_limit(k_xinv<CONS_RHS, C, NF>, bytes);
  if (e == hipSuccess) e = raise_limit(k_xinv<CONS_CGUPD, C, NF>, bytes);
  return e;
}
template <int NF>
hipError_t xinv_limits(const Geom& g, size_t bytes) {
  switch (g.c) {
    case 3: return xinv_limits<NF, 3>(bytes);
    case 4: return xinv_limits<NF, 4>(bytes);
    case 6: return xinv_limits<NF, 6>(bytes);
    case 9: return xinv_limits<NF, 9>(bytes);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fh
