// Kernel launchers used by the host driver (all enqueue on the given stream).
#pragma once

#include "common.h"

namespace fh {

// PROD_CGOP*: the forward x pass of the CG on strain fields; PROD_XOP*: the x pass of the CG on displacements
enum Producer {
  PROD_IDENT = 0, PROD_STRESS = 1, PROD_CGOP = 2, PROD_TRHS = 3, PROD_CGOP_STORED = 4, PROD_ADJ = 5,
  PROD_XOP = 6, PROD_XOP_STORED = 7
};
enum Consumer { CONS_IDENT = 0, CONS_RHS = 1, CONS_CGUPD = 2 };
// projection and plain transforms; CG on displacements: the iteration's forward and inverse passes,
// the right-hand side, the expansion of the solution or of the residual
enum OuterMode {
  OUTER_PROJECT = 0, OUTER_FWD = 1, OUTER_INV = 2, OUTER_CGFWD = 3, OUTER_RHS = 4, OUTER_CGINV = 5,
  OUTER_SOLUTION = 6, OUTER_RESIDUAL = 7
};
inline bool outer_cg_mode(int mode) { return mode >= OUTER_CGFWD; }
// 3D grids with a CG tolerance from here on run the CG on displacements (pass_kernels.h).  Where the two forms
// take the same iterations it is the faster one at any tolerance: 33^3, 64^3 and 128^3, contrast 10 and 20,
// linear elastic, Neo-Hookean, St. Venant-Kirchhoff and J2, at 1e-10 to 1e-13 the counts are equal or one
// apart (64^3 tangent at contrast 100: equal) and a Neo-Hookean solve takes 22.4 ms against 23.1 at 33^3 (1e-10),
// 34.3 / 48.4 at 64^3 and 168.8 / 203.4 at 128^3 (both 1e-12).  Where rounding decides the counts they are not
// those of the textbook CG on strains: 6 x 5 x 7 with densities from 0.05, cubed, 152 / 154 iterations at 1e-11,
// 164 / 168 at 1e-12, 177 / 184 at 1e-13; 16^3 with densities from 0.01 21556 / 21025 at 1e-12; and a tolerance
// beyond rounding (16^3, 1e-16) is met by its recursive residual where the strain fields' stagnates.  Callers
// that ask for less than 1e-11 compare with the textbook iteration and keep it.
// There is no such form in 2D, which has no y pass to save traffic in and whose iterations cost their launches.
constexpr double kDisplacementTol = 1e-11;
enum Reduce { RED_SRC = 0, RED_RHS = 1, RED_PQ = 2, RED_RR = 3 };

// x-axis forward pass: per-voxel producer, then real-to-complex FFT along x.
struct XFwdArgs {
  Geom g;
  AxisPlan px;
  int R;                 // rows (y,z lines) per block
  int nblocks;           // blocks per right-hand side
  int inplace;           // FFT stages staged through registers (one LDS buffer)
  const double* in;      // IDENT: field [B][c][N]; CGOP: residual r [B][c][N]
  double* p;             // CGOP: search direction, updated in place
  double* x;             // CGOP: CG solution, receives the previous iteration's alpha p
  const double* F;       // linearisation point / strain [c][N]
  const double* Kst;     // stored tangent [c(c+1)/2][N]
  double2* spec;         // [B][c][Nh]
  MatParams mat;          // cell 0; cell i has its phase map at phase + i N, its table at table + i 2 kMaxPhase
  int per_inst;          // right-hand sides per cell of a multi-cell batch (0: one cell, every b uses cell 0)
  const int* active;     // nullable: right-hand side of launch index blockIdx.y (the running ones)
  CgState* st;           // per right-hand side
  double* partials;      // [B][nblocks]
  double unit[kMaxC];    // TRHS: load l of a cell is unit[l] * e_l in the packed basis; ADJ: packed W
  double w_energy;       // ADJ: weight of the energy in the objective
  double scale;          // XOP: 1 / N of the inverse transform
};

// x-axis inverse pass: complex-to-real FFT along x, then per-voxel consumer.
struct XInvArgs {
  Geom g;
  AxisPlan px;
  int R;
  int nblocks;
  int inplace;
  const double2* spec;
  double* out;           // IDENT output [B][c][N]
  double* x;             // RHS: CG solution [B][c][N], set to zero
  double* r;             // CG residual [B][c][N]
  const int* active;     // nullable: right-hand side of launch index blockIdx.y
  CgState* st;
  double* partials;
  double scale;          // 1 / N
};

// y (3D) or outer-axis pass over the half spectrum.
struct AxisArgs {
  Geom g;
  AxisPlan pl;
  int TX;                // kx bins per block
  int ZB;                // y pass: consecutive z planes per block (1 for the other passes)
  int inplace;
  int proj;              // y pass inside the projection chain (finite strain 3D: the row-wise
                         // y passes that carry two components per row to the outer pass)
  double2* spec;
  const CgState* st;     // nullable: skip right-hand sides whose CG is not running
  const int* active;     // nullable: right-hand side of each launch-index group
  // nullable: the x pass's <p, K:p> block partials; one block per right-hand side of the pass sums them
  // and sets alpha, in place of a separate reduction launch (the outer pass of the CG on strain fields,
  // the forward y pass of the CG on displacements)
  CgState* pq_st;
  const double* pq_partials;
  int pq_nblocks;
  // CG on displacements.  mirror: forward y pass, keep the mirror planes Hermitian.  Outer passes: mode
  // (launch_outer sets it), the CG vectors [B][d][Nh], and the <r, r> block partials [B][rr_nblocks]
  int mirror;
  int mode;
  double2 *xu, *ru, *pu;
  double* rr_partials;
  int rr_nblocks;
  double inv_n;          // 1 / N
  int stream;            // the CG vectors pass the caches by
};

// dynamic LDS bytes of each pass; `inplace` drops the ping-pong buffer
size_t xfwd_smem(const Geom& g, int R, int inplace);
size_t xinv_smem(const Geom& g, int R, int inplace);
size_t xop_smem(const Geom& g, int R, int inplace);  // x pass of the CG on displacements
// y pass; proj != 0: the projection chain's y pass (three tiles per block for finite strain 3D)
size_t mid_smem(const Geom& g, int TX, int inplace, int ZB = 1, int proj = 0);
// sequences of one FFT call of a y-pass block of TX bins and ZB planes
int mid_sequences(const Geom& g, int TX, int ZB, int proj);
// the row-wise finite-strain y pass holds kFrowHeld elements per thread: ny * TX * ZB must fit
constexpr int kFrowHeld = 8;
bool mid_fits(const Geom& g, int TX, int ZB, int proj);
// z planes per y-pass block for a tile of TX bins: 1 unless the tile spans the whole stored row,
// then as many as fit 32 KiB of LDS while the pass keeps about 512 blocks over B right-hand sides
int mid_planes(const Geom& g, const AxisPlan& pl, int TX, int inplace, long long B, int proj = 0);
// outer pass: LDS bytes, components per block and blocks per right-hand side along z of the
// grid, for the projection (mode OUTER_PROJECT) or a plain transform (OUTER_FWD / OUTER_INV)
size_t outer_smem(const Geom& g, int TX, int inplace, int mode = OUTER_PROJECT);
int outer_group(const Geom& g, int mode = OUTER_PROJECT);
int outer_groups_per_rhs(const Geom& g, int mode = OUTER_PROJECT);
// register staging possible for an outer-pass block of TX bins (widest tile)
bool outer_inplace_ok(const Geom& g, const AxisPlan& pl, int TX, int mode = OUTER_PROJECT);
// true if the y pass of the projection chain uses the row-wise finite-strain kernels
inline bool finite_rows(const Geom& g) { return !g.small && g.ndim == 3; }
// true if an in-place transform of nseq sequences of this plan fits the register staging
bool inplace_ok(const AxisPlan& pl, int nseq);

// FFT plan of an axis of length n: the direct stages, or the chirp-z form with its convolution
// length when the direct stages' prime lengths other than 2, 3 and 5 sum to more than chirp_above
// (0: never); table pointers left null.  False if n has no factorisation within kMaxStages stages.
bool make_plan(int n, AxisPlan* pl, int chirp_above);
// chirp_above of axis `axis` (0: x) of length n.  Measured per pass (us per CG iteration, direct stages / chirp-z;
// the outer pass, both directions, and the x or y passes together) on n x n grids and on one long axis over
// 64 x 64.  The chirp-z form's cost is that of its length m, the direct stages' grows with the prime.
// Outer axis, 270: 2D 257 48 / 55, 311 55 / 46; 3D finite strain 257 348 / 485, 311 512 / 470, 433 939 / 727,
// small strain 311 542 / 508.  (Two lengths between are not in line, for m has five radix stages there or two
// blocks no longer fit a CU: 337 559 / 628 and 586 / 941, 401 710 / 772 and 832 / 1129.)
// x and y, up to 400 points (m <= 800), 300 in 3D finite strain: x 257 500 / 628, 311 672 / 609, 337 888 / 717,
// 379 1002 / 651, y 257 626 / 665, 311 774 / 677, 379 1067 / 761; 360 elsewhere: small strain x 311 425 / 453,
// 337 457 / 518, 379 575 / 498, y 337 504 / 568, 379 580 / 515, 2D x 337 88 / 94, 379 97 / 88.
// Longer ones, whose buffers leave fewer blocks on a CU, 410: finite strain x 401 1076 / 1490, y 401 1229 / 1141,
// 433 1495 / 1093; small strain x 401 657 / 644, 433 750 / 607, y 401 681 / 806, 433 807 / 780; 2D 401 102 / 107,
// 433 108 / 103.
constexpr int kChirpOuter = 270;
constexpr int kChirpRowsFinite = 300;
constexpr int kChirpRowsShort = 360;
constexpr int kChirpRows = 410;
inline int chirp_limit(int n, int ndim, int axis, bool small) {
  if (axis == ndim - 1) return kChirpOuter;
  return n > 400 ? kChirpRows : ndim == 3 && !small ? kChirpRowsFinite : kChirpRowsShort;
}
// true if axis `axis` (0: x), of length n, of a grid of ndim dimensions and `voxels` points runs the folded
// dense DFT: lengths without a compiled schedule from 17 (below, one row tile would be mostly padding) to
// kDenseMax points, beyond kDenseAll only with a large prime factor.  Measured against the radix and direct
// prime stages, us per CG iteration (finite strain): 33^3 80 against 97, 57^3 114 / 161, 91^3 298 / 402,
// 119^3 616 / 864, 119^2 54 / 56; but 143^2 (11 x 13) 68 / 58, 221^2 80 / 63, 143^3 1638 / 1545, as its cost
// per element grows with n.  The line beyond kDenseAll is on the sum of the primes above 5.  2D: 120; even at
// a prime of 151, 178^2 (89) 75 / 68.  3D: 85; one long axis over 96 x 96, us per iteration of the stages over
// the dense DFT's, small strain x, y, outer axis and finite strain the same: 161 (7 x 23) 0.91 0.82 1.00, 0.92
// 0.91 1.01; 164 (41) 0.86 0.76 0.92, 0.86 0.87 0.95; 201 (67) 1.10 0.97 0.99, 0.88 1.10 0.94; 237 (79) 1.12
// 1.03 1.02, 0.97 1.19 1.19; 178 (89) 1.30 1.05 1.10, 1.06 1.32 1.10; 254 (127) 1.30 1.19 1.17, 1.15 1.41
// 1.33.  (Over 24 x 24, where a pass is latency, the stages gain below the line too: 0.83 to 1.06 at 41 to 79,
// the finite-strain y axis 0.6.)
// Lengths with no prime factor above 5 have cheap radix stages (two to four).  Their chain of LDS round
// trips is the longer one where a pass is latency (2D: 36^2 to 125^2 49 / 55 to 60 / 65; 3D up to 30 points:
// 30^3 71 / 119, 24 cells of 20^3 to 30^3 even), but the dense DFT has more to compute where the card is
// full.  In 3D
// - beyond kDenseSmooth points they run the stages (finite strain 72^3 203 / 180, 100^3 418 / 350, 125^3
//   656 / 520; small strain 72^3 178 / 128, 108^3 449 / 280), except for the finite-strain y passes, three
//   transforms in a row per block, of at most kDenseFewVoxels (16 x 72 x 16 77 / 84, 16 x 125 x 16 86 / 97,
//   32 x 125 x 32 112 / 116; 64 x 72 x 64 135 / 130);
// - in small strain the y axis (whose passes are plain copies through the transform) runs the stages from 36
//   points on (16 x 36 x 16 66 / 64, 24 cells of it 367 / 321, 23 cells of 32 x 40 x 32 1223 / 1010), and
//   40 = 8 x 5 points, two stages, on any axis (40^3 82 / 77, 15 cells of it 1341 / 1024);
// - the others keep the dense DFT (finite strain 36^3 86 / 110, 60^3 115 / 136; small strain, x passes 36^3
//   13 / 19, 50^3 17 / 23).
// The cells of a batch run what one cell of their size runs.
constexpr int kDenseAll = 128;
constexpr int kDenseMax = 256;
constexpr int kDenseSmooth = 64;
constexpr long long kDenseFewVoxels = 1 << 17;
// by default: whether any grid of that many dimensions runs it on an axis of that length
bool dense_len(int n, int ndim, int axis = 1, bool small = false, long long voxels = 0);
size_t dense_elems(int n);  // entries of its operand-fragment table
// LDS rows per sequence of the x, mid and outer transforms of the plans pl[0..ndim-1]
void set_lds_lens(Geom* g, const AxisPlan* pl);
// the stages of length n (radices 16/8/4/2/3/5 and remaining primes); false if more than kMaxStages
bool factorize(int n, int* radix, int* nst);
// complex entries of an axis plan's device tables: twiddles of lds_len, then chirp (n) and filter (m)
// of a chirp-z axis, or the operand fragments of a dense axis
size_t plan_table_elems(const AxisPlan& pl);
// entries from one axis's tables to the next one's where a grid's axes share a buffer (whole 256 bytes)
inline size_t plan_table_stride(const AxisPlan& pl) { return (plan_table_elems(pl) + 15) / 16 * 16; }
// Set the table pointers of the plan pl into `base` (plan_table_elems entries, device memory) and make the
// tables that the caller's twiddles (exp(-2 pi i j / L), already there) do not cover: a chirp-z plan's, a
// dense plan's fragments.  all: pl is a grid's three axes (n = 0: none), plan_table_stride entries each,
// and the twiddles are made too (by sincospi of reduced arguments; a dense axis gets none, its
// transform reads the fragments alone): one launch for all axes, beside one for each chirp-z axis.
hipError_t launch_plan_tables(AxisPlan* pl, double2* base, hipStream_t s, bool all);

hipError_t launch_xfwd(int prod, int mat, const XFwdArgs& a, int B, hipStream_t s);
hipError_t launch_xinv(int cons, const XInvArgs& a, int B, hipStream_t s);
hipError_t launch_mid(int dir, const AxisArgs& a, int B, hipStream_t s);
hipError_t launch_outer(int mode, const AxisArgs& a, int B, hipStream_t s);
// B blocks; block i reduces right-hand side active[i] (active nullable: i)
hipError_t launch_cg_reduce(int what, CgState* st, const double* partials, int nblocks, int B, hipStream_t s,
                            const int* active = nullptr);
// x += alpha p for every right-hand side whose CG stopped after at least one full iteration
hipError_t launch_cg_finish(double* x, const double* p, const CgState* st, const Geom& g, int B, hipStream_t s);

// Newton-level and post-processing kernels.
hipError_t launch_init_reference(double* F, const Geom& g, hipStream_t s);
hipError_t launch_shift(double* F, const double* delta, const Geom& g, hipStream_t s);
hipError_t launch_update(double* F, const double* x, double* partials, int nblocks, const Geom& g,
                         hipStream_t s);
hipError_t launch_homogenize(int mat, const double* F, MatParams m, double* partials, int nblocks,
                             const Geom& g, CgState* st, hipStream_t s);
hipError_t launch_tangent_matrix(int mat, const double* F, const double* X, const double* unit, MatParams m,
                                 double* partials, int nblocks, const Geom& g, hipStream_t s);
hipError_t launch_reduce_slots(const double* partials, int nslots, int nblocks, double* out, hipStream_t s);
hipError_t launch_store_tangent(int mat, const double* F, MatParams m, double* Kst, const Geom& g,
                                hipStream_t s);
hipError_t launch_expand(const double* packed, double* full, const Geom& g, hipStream_t s);
hipError_t launch_pack(const double* full, double* packed, const Geom& g, hipStream_t s);
hipError_t launch_stress_field(int mat, const double* F, MatParams m, double* full_out, double* energy_out,
                               const Geom& g, hipStream_t s);
hipError_t launch_simp_scale(const double* density, double p, double* scale, long long N, hipStream_t s);
hipError_t launch_check_phase(const uint8_t* phase, long long N, int nphase, int* flag, hipStream_t s);
hipError_t launch_debug_constitutive(int mat, const double* e, const double* de, double* P, double* KdE,
                                     double* psi, MatParams m, const Geom& g, hipStream_t s);
// dJ/drho_v = p / (N rho_v) [ w_e psi_v + (W + x_v) : P_v ]  (adjoint density gradient)
hipError_t launch_simp_gradient(int mat, const double* F, const double* x, MatParams m, const double* density,
                                double p, const double* W, double w_energy, double* grad, const Geom& g,
                                hipStream_t s);
// J2 plasticity: commit the history at the converged strain F (in place), and the
// cumulative plastic strain of the state at F
hipError_t launch_j2_commit(int mat, const double* F, MatParams m, double* hist, const Geom& g, hipStream_t s);
hipError_t launch_j2_plastic(int mat, const double* F, MatParams m, double* out, const Geom& g, hipStream_t s);
hipError_t set_smem_limits(const Geom& g, int mat, size_t bytes);
// x passes of one law with FFT variant nf (pass_fft in pass_kernels.h); dynamic-LDS limits
#define FH_XPASS_DECL(name)                                                                                  \
  hipError_t name(int nf, int prod, int mat, const XFwdArgs& a, dim3 grid, size_t sm, hipStream_t s); \
  hipError_t name##_limits(int mat, size_t bytes);
FH_XPASS_DECL(xpass_le)
FH_XPASS_DECL(xpass_nh)
FH_XPASS_DECL(xpass_stvk)
FH_XPASS_DECL(xpass_j2)
FH_XPASS_DECL(xpass_ps)
#undef FH_XPASS_DECL
// the pass kernels with run-time radix stages (kernels_radix*.hip)
hipError_t launch_xinv_radix(int cons, const XInvArgs& a, dim3 grid, size_t sm, hipStream_t s);
hipError_t launch_mid_radix(int dir, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s);
hipError_t launch_outer_radix(int mode, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s);
hipError_t launch_outer_cg_radix(int mode, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s);
hipError_t set_smem_limits_radix(const Geom& g, size_t bytes);
hipError_t set_smem_limits_radix_outer(const Geom& g, size_t bytes);
hipError_t set_smem_limits_radix_cg(const Geom& g, size_t bytes);
// the pass kernels with the chirp-z transform (kernels_chirp.hip), for plans with m > 0
hipError_t launch_xinv_chirp(int cons, const XInvArgs& a, dim3 grid, size_t sm, hipStream_t s);
hipError_t launch_mid_chirp(int dir, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s);
hipError_t launch_outer_chirp(int mode, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s);
hipError_t set_smem_limits_chirp(const Geom& g, size_t bytes);
// the pass kernels with the folded dense DFT (kernels_dense.hip), for plans with dense set
hipError_t launch_xinv_dense(int cons, const XInvArgs& a, dim3 grid, size_t sm, hipStream_t s);
hipError_t launch_mid_dense(int dir, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s);
hipError_t launch_outer_dense(int mode, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s);
hipError_t set_smem_limits_dense(const Geom& g, size_t bytes);
// the CG-loop pass kernels for single axis lengths with compiled schedules (kernels_fixed.hip):
// lengths that have them; each launcher sets *done when it launched (else the caller launches the
// generic kernel)
bool fixed_len_kernels(int n);
// of those (and 128), lengths whose x pass of the CG on displacements has its own kernel with the stored
// tangent too.  That pass holds both transforms: on the run-time radix stages 32^3 ran slower than on strain
// fields, whose inverse pass has its own kernels (J2, us per solve, strain fields / run-time stages / own
// kernel: 32^3 5513 / 5612 / 5459, 64^3 12424 / 10041 / 9633).  Nine components and 96 points spill in four
// waves: 96^3 Neo-Hookean 102.7 ms on the run-time stages, 105.0 with a kernel of its own; 128^3 192.5 / 190.7.
constexpr bool stored_len_kernels(int n, bool small) { return small || n <= 64; }
hipError_t launch_xinv_fixed(int cons, const XInvArgs& a, dim3 grid, size_t sm, hipStream_t s, bool* done);
hipError_t launch_mid_fixed(int dir, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s, bool* done);
hipError_t launch_outer_fixed(int mode, bool rows, const AxisArgs& a, dim3 grid, size_t sm, hipStream_t s, bool* done);
hipError_t set_smem_limits_fixed(const Geom& g, size_t bytes);

// Scratch of the allocation-free projection: a file-scope device array of this many bytes per
// device (noalloc_scratch.hip); its address on the current device.
constexpr size_t kNoAllocScratchBytes = 64ull << 20;
hipError_t noalloc_scratch_address(void** out);

}  // namespace fh
