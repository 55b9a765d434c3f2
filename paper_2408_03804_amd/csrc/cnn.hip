// Voxel-CNN stiffness surrogate on the gfx950 matrix cores.
//
// Every layer is a bf16 x bf16 -> fp32 GEMM on gfx950 MFMA 16x16x32 tiles:
//   conv forward      pre[m][co]   = col[m][k] . W[co][k]            (col = periodic stride-2 im2col)
//   conv weight grad  dW[co][k]    = sum_m dpre[m][co] col[m][k]      (split over m, fixed-order sum)
//   conv input grad   dcol[m][k]   = sum_co dpre[m][co] W[co][k], gathered back to the voxels
// col and dcol are never stored where the channels are multiples of 8: the tile loaders gather their
// operands from the previous block's activations, the phase map or dpre (implicit GEMM).  Bias and gelu
// (their derivative in the input gradient) are applied to the accumulators.
//   dense layers      the same three products with m = sample
// around small element-wise kernels (pooling, loss, Adam).  All sums that
// cross blocks go through partial buffers reduced in a fixed order, so a training step is
// bitwise reproducible.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "fft_homog.h"
#include "fft_homog_cnn.h"

namespace cnn {

typedef uint16_t bf16;
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kT = 256;
constexpr int BM = 64, BN = 64, BK = 128;  // GEMM tile
constexpr int kMaxSplits = 1024;
constexpr int kColRows = 256;  // rows per block of the bias-gradient column sums

// fp32 -> bf16, round to nearest even (NaN stays NaN)
__host__ __device__ inline bf16 to_bf16(float f) {
  uint32_t u;
  memcpy(&u, &f, 4);
  if ((u & 0x7f800000u) == 0x7f800000u) return (bf16)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16)(u >> 16);
}
__device__ inline float from_bf16(bf16 b) { return __uint_as_float((uint32_t)b << 16); }

__device__ inline float gelu(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ inline float gelu_grad(float x) {
  return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * 0.39894228040143268f * expf(-0.5f * x * x);
}

// quotient by d of r < 2^31 (magic = ceil(2^(31 + s) / d), 2^s >= d: exact over that range)
struct Div {
  uint32_t d, magic, s;
};
Div make_div(int d) {
  Div f{(uint32_t)d, 0, 0};
  while ((1u << f.s) < f.d) ++f.s;
  f.magic = (uint32_t)(((1ull << (31 + f.s)) + f.d - 1) / f.d);
  return f;
}
__device__ inline uint32_t quot(uint32_t r, const Div& f) { return __umulhi(r << 1, f.magic) >> f.s; }

// ---------------------------------------------------------------------------
// GEMM: C[z][m][n] = sum_{k in split z} A(m,k) B(n,k)
// ---------------------------------------------------------------------------
// Implicit im2col operand of a conv block: element (row, k) of col, row = ((b m + oz) m + oy) m + ox
// over the m^3 outputs of each sample, k = t Ci + ci with tap t = 9 tz + 3 ty + tx < 27, is
// src[b, (2 oz + tz - 1) mod n, (2 oy + ty - 1) mod n, (2 ox + tx - 1) mod n, ci]  (n = 2 m), and
// zero for k >= 27 Ci.  Ci % 8 == 0, so 8 consecutive k share a tap (one 16-byte load).
struct ConvOperand {
  const bf16* src;  // [b][z][y][x][Ci] activations of the previous block
  int n, Ci;
  Div m, ci;
};

// operands of k_gemm: from memory, contiguous along k or along rows; the im2col operand, k along its
// columns (forward) or along its rows (weight gradient); block 1's 27 taps as bits, k along rows
enum Operand { OP_K, OP_ROW, OP_COL, OP_COLT, OP_BITS };
constexpr bool along_k(int op) { return op == OP_K || op == OP_COL; }

struct GemmArgs {
  int M, N, K, kchunk;
  const bf16* A;
  long long sam, sak;
  const bf16* B;
  long long sbn, sbk;
  float* C;               // product, or with bias: product + bias (nullable)
  const float* bias;
  bf16* act;              // bf16(gelu(C)) (nullable)
  ConvOperand cv;         // the implicit operand (A for OP_COL, B for OP_COLT)
  const uint8_t* bits;    // OP_BITS: 4 bytes per output row
};

// periodic input coordinate of output coordinate o and tap component t (0..2)
__device__ inline int tap_coord(int o, int t, int n) {
  int i = 2 * o + t - 1;
  if (i < 0) i += n;
  if (i >= n) i -= n;
  return i;
}

// output row -> (sample, oz, oy, ox); rows are below 2^31 (max_batch m^3 outputs per block)
struct Row {
  uint32_t b;
  int z, y, x;
};
__device__ inline Row row_of(uint32_t r, const Div& m) {
  Row w;
  uint32_t q = quot(r, m);
  w.x = (int)(r - q * m.d);
  r = q;
  q = quot(r, m);
  w.y = (int)(r - q * m.d);
  r = q;
  w.b = quot(r, m);
  w.z = (int)(r - w.b * m.d);
  return w;
}
// Addresses of the im2col operand without a wrap per coordinate: an output's centre tap, and a tap's offset
// from it.  Only tap component 0 of output coordinate 0 leaves the cell, by -1: it gets the axis length
// back (both masks set).  The divisions and wraps of every entry were most of the loaders' instructions.
struct OutputRef {
  const bf16* p;
  int fz, fy, fx;  // -1 where the output coordinate is 0
};
__device__ inline OutputRef output_ref(const ConvOperand& c, uint32_t row) {
  const Row w = row_of(row, c.m);
  OutputRef r;
  r.p = c.src + (((w.b * (long long)c.n + 2 * w.z) * c.n + 2 * w.y) * c.n + 2 * w.x) * c.Ci;
  r.fz = w.z == 0 ? -1 : 0;
  r.fy = w.y == 0 ? -1 : 0;
  r.fx = w.x == 0 ? -1 : 0;
  return r;
}
struct TapOffset {
  int off, wz, wy, wx;  // a cell's activations are at most 2^28 entries
};
__device__ inline TapOffset tap_offset(const ConvOperand& c, int tap, int ci) {
  const int tz = tap / 9, ty = (tap / 3) % 3, tx = tap % 3;
  TapOffset t;
  t.off = (((tz - 1) * c.n + ty - 1) * c.n + tx - 1) * c.Ci + ci;
  t.wx = tx == 0 ? c.n * c.Ci : 0;
  t.wy = ty == 0 ? c.n * c.n * c.Ci : 0;
  t.wz = tz == 0 ? c.n * c.n * c.n * c.Ci : 0;
  return t;
}
__device__ inline uint4 conv_gather(const OutputRef& r, const TapOffset& t) {
  return *reinterpret_cast<const uint4*>(r.p + (t.off + (r.fz & t.wz) + (r.fy & t.wy) + (r.fx & t.wx)));
}

// Tiles of 64 rows x BK in LDS, in 16-byte groups of 8 k: group g of row r at g ^ (r ^ r / 8) mod 8.
// So neither the reads of the MFMA operands (16 rows at one g), nor the 16-byte stores along k, nor
// the 4-byte stores of an operand that is contiguous along rows (8 rows of 8, two k each) meet in a bank.
__device__ inline int tile_at(int r, int g) { return r * BK + ((g ^ ((r ^ (r >> 3)) & 7)) << 3); }

// This thread's p-th (of 4) 8 entries of a tile: along k, row t / 16 + 16 p at group t mod 16; along
// rows, 8 (t mod 8) .. + 7 at k = 2 (t / 8 + 32 (p / 2)) + p mod 2 (so that it holds pairs of k).
__device__ inline int chunk_row(bool kc, int p) { return kc ? ((int)threadIdx.x >> 4) + 16 * p : ((int)threadIdx.x & 7) * 8; }
__device__ inline int chunk_k(bool kc, int p) {
  return kc ? ((int)threadIdx.x & 15) * 8 : 2 * (((int)threadIdx.x >> 3) + 32 * (p >> 1)) + (p & 1);
}

// Four chunks of an operand in memory, zero outside [0, nrows) x [.., kend).  VEC: every chunk inside is
// 16 aligned bytes.  Loads are then unconditional, from a clamped address, and chunks outside are cleared
// when they are stored (ok): a load under a condition is waited for where its branch ends, not where its
// value is used, which left nothing in flight during the products.  Else every chunk decides for itself:
// 16 bytes where it is whole and aligned, entry by entry otherwise.
struct Chunks {
  uint4 v[4];
  bool ok[4];
};
template <bool KC, bool VEC>
__device__ inline void fetch_tile(Chunks& f, const bf16* P, long long s_row, long long s_k, int row0, int nrows, int k0,
                                  int kend) {
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int row = row0 + chunk_row(KC, p);
    const int k = k0 + chunk_k(KC, p);
    f.ok[p] = row < nrows && k < kend;
    if constexpr (VEC) {
      const int rc = min(row, KC ? nrows - 1 : nrows - 8), kc = min(k, KC ? kend - 8 : kend - 1);
      f.v[p] = *reinterpret_cast<const uint4*>(P + (long long)rc * s_row + (long long)kc * s_k);
    } else {
      f.v[p] = make_uint4(0u, 0u, 0u, 0u);
      if (!f.ok[p]) continue;
      const bf16* src = P + (long long)row * s_row + (long long)k * s_k;
      const int left = KC ? kend - k : nrows - row;  // entries of the 8 inside
      if (left >= 8 && (reinterpret_cast<uintptr_t>(src) & 15u) == 0) {
        f.v[p] = *reinterpret_cast<const uint4*>(src);
        continue;
      }
      uint64_t lo = 0, hi = 0;
#pragma unroll 1
      for (int i = 0; i < min(left, 8); ++i) {
        const uint64_t e = (uint64_t)src[i] << (16 * (i & 3));
        if (i < 4) lo |= e;
        else hi |= e;
      }
      f.v[p] = make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
    }
  }
}

template <bool KC>
__device__ inline void store_tile(bf16* T, const Chunks& f) {
  uint4 v[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) v[p] = f.ok[p] ? f.v[p] : make_uint4(0u, 0u, 0u, 0u);
  if constexpr (KC) {
#pragma unroll
    for (int p = 0; p < 4; ++p)
      *reinterpret_cast<uint4*>(T + tile_at(chunk_row(true, p), (int)threadIdx.x & 15)) = v[p];
  } else {
#pragma unroll
    for (int p = 0; p < 4; p += 2) {
      const int r = chunk_row(false, p), k = chunk_k(false, p);
      const uint32_t a[4] = {v[p].x, v[p].y, v[p].z, v[p].w};
      const uint32_t b[4] = {v[p + 1].x, v[p + 1].y, v[p + 1].z, v[p + 1].w};
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t lo = (i & 1) ? a[i >> 1] >> 16 : a[i >> 1] & 0xffffu;
        const uint32_t hi = (i & 1) ? b[i >> 1] & 0xffff0000u : b[i >> 1] << 16;
        *reinterpret_cast<uint32_t*>(T + tile_at(r + i, k >> 3) + (k & 7)) = lo | hi;
      }
    }
  }
}

// 256 threads = 4 waves in a 2 x 2 arrangement, each wave a 32 x 32 block of 2 x 2 MFMA tiles.
// gfx950 MFMA 16x16x32 bf16 (v_mfma_f32_16x16x32_bf16, one instruction per 32-deep k step of a tile):
// lane l holds rows/cols (l mod 16) at k = 8 (l / 16) + 0..7 (one 16-byte LDS read per operand).  B is
// the first operand, so the accumulator of lane l holds C row (l mod 16), columns 4 (l / 16) + 0..3:
// 16-byte stores.
struct WaveTile {
  int m, n, lr, lk;  // C row of acc[i]: m + 16 i + lr, columns of acc[.][j]: n + 16 j + lk + 0..3
  // narrow: the four waves hold 16 rows x 32 columns each, one below the other
  __device__ inline explicit WaveTile(bool narrow = false) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    m = narrow ? w * 16 : (w >> 1) * 32;
    n = narrow ? 0 : (w & 1) * 32;
    lr = lane & 15;
    lk = 4 * (lane >> 4);
  }
};
template <int I>
__device__ inline void mfma_step(v4f (&acc)[I][2], const bf16* As, const bf16* Bs, const WaveTile& w, int ks) {
  v8bf a[I], b[2];
#pragma unroll
  for (int i = 0; i < I; ++i) a[i] = *reinterpret_cast<const v8bf*>(As + tile_at(w.m + 16 * i + w.lr, 4 * ks + (w.lk >> 2)));
#pragma unroll
  for (int i = 0; i < 2; ++i) b[i] = *reinterpret_cast<const v8bf*>(Bs + tile_at(w.n + 16 * i + w.lr, 4 * ks + (w.lk >> 2)));
#pragma unroll
  for (int i = 0; i < I; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
}
__device__ inline void mfma_tile(v4f (&acc)[2][2], const bf16* As, const bf16* Bs, const WaveTile& w, int depth) {
#pragma unroll
  for (int ks = 0; ks < BK / 32; ++ks)
    if (32 * ks < depth) mfma_step(acc, As, Bs, w, ks);
}

// Four consecutive columns of a row of the product: x + bias into C and bf16(gelu) into act (either may
// be null), or x into C if there is no bias.  wide: rows of C and act are 16- and 8-byte aligned.
__device__ inline void store_row4(v4f x, int col, int N, bool wide, const float* bias, float* C, bf16* act) {
  if (bias) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < N) x[e] += bias[col + e];
  }
  if (wide && col + 3 < N) {
    if (C) *reinterpret_cast<v4f*>(C + col) = x;
    if (act) {
      const uint32_t lo = (uint32_t)to_bf16(gelu(x[0])) | ((uint32_t)to_bf16(gelu(x[1])) << 16);
      const uint32_t hi = (uint32_t)to_bf16(gelu(x[2])) | ((uint32_t)to_bf16(gelu(x[3])) << 16);
      *reinterpret_cast<uint2*>(act + col) = make_uint2(lo, hi);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < N) {
        if (C) C[col + e] = x[e];
        if (act) act[col + e] = to_bf16(gelu(x[e]));
      }
  }
}

// Bound by the latency of the operand loads and the instructions that form their addresses (the products
// of a training step are 50 GFLOP, 40 us at the card's rate): a block keeps the next BK of both operands
// on their way to registers while it multiplies this one (two ahead gained nothing).  With one 32-deep
// step at a time the conv products of 256 cells of 32^3 took, in mean, 67 us (forward, blocks 2-4) and
// 141 us (weight gradient), now 39 and 51 us; block 1's weight gradient 78, now 50 us.
// VA, VB: VEC of the operand in memory.
template <int AOP, int BOP, bool VA, bool VB>
__global__ void __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(3))) k_gemm(GemmArgs g) {
  __shared__ __attribute__((aligned(16))) bf16 As[BM * BK];
  __shared__ __attribute__((aligned(16))) bf16 Bs[BN * BK];
  const int m0 = blockIdx.x * BM;
  const int n0 = blockIdx.y * BN;
  const int kbeg = blockIdx.z * g.kchunk;
  const int kend = min(g.K, kbeg + g.kchunk);
  const WaveTile w;
  v4f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  // OP_COL: the outputs of this thread's rows.  OP_COLT: its tap and channel.
  OutputRef arow[4] = {};
  if constexpr (AOP == OP_COL) {
#pragma unroll
    for (int p = 0; p < 4; ++p) arow[p] = output_ref(g.cv, (uint32_t)min(m0 + chunk_row(true, p), g.M - 1));
  }
  const int kcol = n0 + chunk_row(false, 0);
  int btap = 0;
  TapOffset boff = {};
  if constexpr (BOP == OP_COLT) {
    btap = (int)quot((uint32_t)kcol, g.cv.ci);
    boff = tap_offset(g.cv, min(btap, 26), btap < 27 ? kcol - btap * g.cv.Ci : 0);
  }
  Chunks fa, fb;
  auto fetch = [&](int k0) {
    if constexpr (AOP == OP_COL) {
      const int k = k0 + chunk_k(true, 0);
      const int tap = (int)quot((uint32_t)k, g.cv.ci);
      const TapOffset t = tap_offset(g.cv, min(tap, 26), tap < 27 ? k - tap * g.cv.Ci : 0);
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        fa.ok[p] = m0 + chunk_row(true, p) < g.M && k < kend && tap < 27;
        fa.v[p] = conv_gather(arow[p], t);
      }
    } else {
      fetch_tile<AOP == OP_K, VA>(fa, g.A, g.sam, g.sak, m0, g.M, k0, kend);
    }
    if constexpr (BOP == OP_COLT || BOP == OP_BITS) {
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int row = k0 + chunk_k(false, p), rc = min(row, kend - 1);
        fb.ok[p] = row < kend && kcol < g.N;
        if constexpr (BOP == OP_COLT) {
          fb.ok[p] = fb.ok[p] && btap < 27;
          fb.v[p] = conv_gather(output_ref(g.cv, (uint32_t)rc), boff);
        } else {
          fb.v[p].x = g.bits[4 * (long long)rc + (min(kcol, g.N - 8) >> 3)];  // expanded when it is stored
        }
      }
    } else {
      fetch_tile<BOP == OP_K, VB>(fb, g.B, g.sbn, g.sbk, n0, g.N, k0, kend);
    }
  };
  auto put = [&] {
    if constexpr (BOP == OP_BITS) {
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const uint32_t t = fb.v[p].x;
        auto two = [&](int i) { return ((t >> i) & 1u) * 0x3f80u | ((t >> (i + 1)) & 1u) * 0x3f800000u; };
        fb.v[p] = make_uint4(two(0), two(2), two(4), two(6));
      }
    }
    store_tile<along_k(AOP)>(As, fa);
    store_tile<along_k(BOP)>(Bs, fb);
  };
  fetch(kbeg);
  for (int k0 = kbeg; k0 < kend; k0 += BK) {
    put();
    __syncthreads();
    if (k0 + BK < kend) fetch(k0 + BK);
    mfma_tile(acc, As, Bs, w, kend - k0);
    __syncthreads();
  }
  float* C = g.C ? g.C + (long long)blockIdx.z * g.M * g.N : nullptr;
  const bool wide = (g.N & 3) == 0 && ((reinterpret_cast<uintptr_t>(C) & 15u) == 0);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = m0 + w.m + 16 * i + w.lr;
    if (row >= g.M) continue;
#pragma unroll
    for (int j = 0; j < 2; ++j)
      store_row4(acc[i][j], n0 + w.n + 16 * j + w.lk, g.N, wide, g.bias, C ? C + (long long)row * g.N : nullptr,
                 g.act ? g.act + (long long)row * g.N : nullptr);
  }
}

// First conv block (27 taps of the u8 phase map, K = 32): pre = col W + bias, act = bf16(gelu(pre)).
// Bound by those stores, 134 + 67 MB for 256 cells of 32^3 with 32 channels.  A wave builds the MFMA
// operands of 64 output rows from the phase bytes (lane l: row l mod 16, taps 8 (l / 16) + 0..7), keeps
// the taps as bits for the weight gradient (bits nullable), and multiplies without LDS: 90 us.  The
// expanded operand alone took 36 us and a bias and gelu pass 106 us, beside the product.  Ids above 1
// raise *bad.
__global__ void __launch_bounds__(kT) k_conv_phase(const uint8_t* phase, int M, int n, Div m, const bf16* W, int N,
                                                   const float* bias, float* pre, bf16* act, uint8_t* bits, int* bad) {
  const int lane = threadIdx.x & 63, lr = lane & 15, kg = lane >> 4;
  const int row0 = (blockIdx.x * (kT / 64) + (threadIdx.x >> 6)) * 64;
  if (row0 >= M) return;
  v8bf a[4];
  uint32_t over = 0;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int row = row0 + 16 * it + lr;
    const Row w = row_of((uint32_t)min(row, M - 1), m);
    const uint8_t* pb = phase + (long long)w.b * n * n * n;
    uint32_t t8 = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int tap = min(8 * kg + i, 26);
      const int tz = tap / 9, ty = (tap / 3) % 3, tx = tap % 3;
      const uint32_t p = pb[(tap_coord(w.z, tz, n) * n + tap_coord(w.y, ty, n)) * n + tap_coord(w.x, tx, n)];
      over |= p >> 1;
      if (8 * kg + i < 27) t8 |= (p ? 1u : 0u) << i;
    }
    if (bits && row < M) bits[4 * (long long)row + kg] = (uint8_t)t8;
    uint32_t e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i] = ((t8 >> (2 * i)) & 1u) * 0x3f80u | ((t8 >> (2 * i + 1)) & 1u) * 0x3f800000u;
    memcpy(&a[it], e, 16);
  }
  if (over) *bad = 1;
  const bool wide = (N & 3) == 0;
  for (int n0 = 0; n0 < N; n0 += 64) {
    v8bf b[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) b[j] = *reinterpret_cast<const v8bf*>(W + (long long)min(n0 + 16 * j + lr, N - 1) * 32 + 8 * kg);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int row = row0 + 16 * it + lr;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (n0 + 16 * j >= N) continue;
        const v4f x = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[it], v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        if (row < M)
          store_row4(x, n0 + 16 * j + 4 * kg, N, wide, bias, pre ? pre + (long long)row * N : nullptr, act + (long long)row * N);
      }
    }
  }
}

// Input gradient of a conv block l > 1, times gelu'(pre of block l - 1), in fp32 (for the bias gradient) and
// bf16.  For 256 cells of 32^3, blocks 2, 3 and 4: 161 + 46 + 31 us.  (Column sums of the fp32 values made here, without
// storing them, saved another 40 us, but in another order than k_colsum_partial's: Adam's first steps
// turn a last-bit change of a gradient near zero into a change of a weight's step.)
// Voxel i of an axis of length n = 2 m is tap t of output o when 2 o + t - 1 = i (mod n): t = 1 (o = i/2)
// for even i, t = 0 (o = (i+1)/2 mod m) and t = 2 (o = (i-1)/2) for odd i.  So the voxels of one parity
// class (blockIdx.z) share their 1, 2, 4 or 8 taps, and their gradient is a product over taps and output
// channels whose operand rows are those of dpre.  Each tap is summed over the channels by itself and the
// taps are added in order, as if the product had been formed for all taps and then gathered; that took
// 165 + 308 us for the same three, mostly for the fp32 products in memory.
struct DgradArgs {
  int M, Ci, Co, Kp, n;  // M = B m^3 voxels of a class
  Div m, co;             // co: of the 32-padded output channels
  const bf16 *dpre, *W;  // [outputs][Co], [Co][Kp]
  const float* pre;      // [voxels][Ci]
  float* d32;
  bf16* db;
};
// NARROW: at most 32 input channels; the waves split the rows only (half of them would have no column).
template <bool NARROW>
__global__ void __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(3))) k_dgrad(DgradArgs g) {
  constexpr int I = NARROW ? 1 : 2;
  __shared__ __attribute__((aligned(16))) bf16 As[BM * BK];
  __shared__ __attribute__((aligned(16))) bf16 Bs[BN * BK];
  const int m0 = blockIdx.x * BM;
  const int n0 = blockIdx.y * BN;
  const int cls = 7 - blockIdx.z;  // the classes with most taps first
  const int pz = cls >> 2, py = (cls >> 1) & 1, px = cls & 1;
  const int m = (int)g.m.d;
  const WaveTile w(NARROW);
  v4f sum[I][2], acc[I][2];
#pragma unroll
  for (int i = 0; i < I; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) sum[i][j] = acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  // output j of each of this thread's rows, and the way from it to output j + 1 (mod m) along each axis
  const bf16* arow[4];
  int dz[4], dy[4], dx[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const Row r = row_of((uint32_t)min(m0 + chunk_row(true, p), g.M - 1), g.m);
    arow[p] = g.dpre + (((r.b * (long long)m + r.z) * m + r.y) * m + r.x) * g.Co;
    dz[p] = (r.z + 1 == m ? 1 - m : 1) * m * m * g.Co;
    dy[p] = (r.y + 1 == m ? 1 - m : 1) * m * g.Co;
    dx[p] = (r.x + 1 == m ? 1 - m : 1) * g.Co;
  }
  // k axis of the product: (tap, 32-padded channel), the taps' x components fastest
  const int cop = (int)g.co.d;
  const int K = cop << (pz + py + px);
  Chunks fa, fb;
  // tap component of the c-th tap of an axis (c = 0 of an odd voxel is on output j + 1, all others on j)
  auto tap = [](int par, int c) { return par ? 2 * c : 1; };
  auto fetch = [&](int k0) {
    {
      const int k = k0 + chunk_k(true, 0);
      const int q = (int)quot((uint32_t)k, g.co), c = k - q * cop;
      const int cx = q & px, cy = (q >> px) & py, cz = (q >> (px + py)) & pz;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int off = (dz[p] & (cz - pz)) + (dy[p] & (cy - py)) + (dx[p] & (cx - px)) + min(c, g.Co - 8);
        fa.ok[p] = m0 + chunk_row(true, p) < g.M && k < K && c < g.Co;
        fa.v[p] = *reinterpret_cast<const uint4*>(arow[p] + off);
      }
    }
    const int ci = n0 + chunk_row(false, 0);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int k = k0 + chunk_k(false, p);
      const int q = (int)quot((uint32_t)k, g.co), c = k - q * cop;
      const int cx = q & px, cy = (q >> px) & py, cz = (q >> (px + py)) & pz;
      const int t = (tap(pz, cz) * 3 + tap(py, cy)) * 3 + tap(px, cx);
      fb.ok[p] = k < K && c < g.Co && ci < g.Ci;
      fb.v[p] = *reinterpret_cast<const uint4*>(g.W + (long long)min(c, g.Co - 1) * g.Kp + t * g.Ci + min(ci, g.Ci - 8));
    }
  };
  fetch(0);
  int left = cop;  // channels of this tap still to be summed
  for (int k0 = 0; k0 < K; k0 += BK) {
    store_tile<true>(As, fa);
    store_tile<false>(Bs, fb);
    __syncthreads();
    if (k0 + BK < K) fetch(k0 + BK);
    const int steps = min(BK, K - k0) / 32;
    for (int ks = 0; ks < steps; ++ks) {
      mfma_step(acc, As, Bs, w, ks);
      left -= 32;
      if (left == 0) {
        left = cop;
#pragma unroll
        for (int i = 0; i < I; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            sum[i][j] += acc[i][j];
            acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int row = m0 + w.m + 16 * i + w.lr;
    if (row >= g.M) continue;
    const Row r = row_of((uint32_t)row, g.m);
    const long long vox = ((r.b * (long long)g.n + 2 * r.z + pz) * g.n + 2 * r.y + py) * g.n + 2 * r.x + px;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = n0 + w.n + 16 * j + w.lk;
      if (col >= g.Ci) continue;  // Ci is a multiple of 8
      const v4f pr = *reinterpret_cast<const v4f*>(g.pre + vox * g.Ci + col);
      v4f o;
      uint32_t h[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[e] = sum[i][j][e] * gelu_grad(pr[e]);
        h[e] = to_bf16(o[e]);
      }
      *reinterpret_cast<v4f*>(g.d32 + vox * g.Ci + col) = o;
      *reinterpret_cast<uint2*>(g.db + vox * g.Ci + col) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
    }
  }
}

// k range of each of at most `splits` splits (a multiple of the MFMA's 32), and the splits this makes
int split_chunk(int K, int splits, int* used) {
  splits = std::max(1, std::min(splits, kMaxSplits));
  int chunk = (K + splits - 1) / splits;
  chunk = (chunk + 31) / 32 * 32;
  *used = (K + chunk - 1) / chunk;
  return chunk;
}

// an operand whose rows of `extent` contiguous entries, `stride` apart, are whole aligned chunks of 8
bool vector_chunks(const bf16* P, long long stride, int extent) {
  return extent % 8 == 0 && stride % 8 == 0 && (reinterpret_cast<uintptr_t>(P) & 15u) == 0;
}

// C (and with bias: act) of operands in memory; *used: the k-splits made
hipError_t gemm(int M, int N, int K, const bf16* A, long long sam, long long sak, const bf16* B, long long sbn,
                long long sbk, float* C, int splits, hipStream_t s, const float* bias = nullptr, bf16* act = nullptr,
                int* used = nullptr) {
  if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
  GemmArgs g{};
  g.M = M;
  g.N = N;
  g.K = K;
  int S;
  g.kchunk = split_chunk(K, splits, &S);
  if (used) *used = S;
  g.A = A;
  g.sam = sam;
  g.sak = sak;
  g.B = B;
  g.sbn = sbn;
  g.sbk = sbk;
  g.C = C;
  g.bias = bias;
  g.act = act;
  dim3 grid((M + BM - 1) / BM, (N + BN - 1) / BN, S);
  const bool ak = sak == 1, bk = sbk == 1;
  // each operand by itself: with one ragged operand (the 21 outputs of the last layer, channels that are no
  // multiple of 8) putting both on the other path made a training step of 12, 28, 52 and 100 channels slower
  // than with each chunk deciding for itself (1006 us -> 1161, now 847; 30, 60, 120, 240: 1416, now 1284)
  const bool va = vector_chunks(A, ak ? sam : sak, ak ? K : M), vb = vector_chunks(B, bk ? sbn : sbk, bk ? K : N);
  auto launch = [&](auto a, auto b) {
    constexpr bool VA = decltype(a)::value, VB = decltype(b)::value;
    if (ak && bk) hipLaunchKernelGGL((k_gemm<OP_K, OP_K, VA, VB>), grid, dim3(kT), 0, s, g);
    else if (ak) hipLaunchKernelGGL((k_gemm<OP_K, OP_ROW, VA, VB>), grid, dim3(kT), 0, s, g);
    else if (bk) hipLaunchKernelGGL((k_gemm<OP_ROW, OP_K, VA, VB>), grid, dim3(kT), 0, s, g);
    else hipLaunchKernelGGL((k_gemm<OP_ROW, OP_ROW, VA, VB>), grid, dim3(kT), 0, s, g);
  };
  if (va && vb) launch(std::true_type{}, std::true_type{});
  else if (va) launch(std::true_type{}, std::false_type{});
  else if (vb) launch(std::false_type{}, std::true_type{});
  else launch(std::false_type{}, std::false_type{});
  return hipGetLastError();
}

// The two conv products with the implicit im2col operand (Kp = 32-padded 27 Ci):
//   forward      pre[M][N] = col[M][Kp] . W[N][Kp] + bias, act             (OP_COL)
//   weight grad  dW[z][co][Kp] = sum_{m in split z} dpre[m][co] col[m][Kp]  (A = dpre, [M][co]; OP_COLT,
//                or block 1's taps as bits)
hipError_t gemm_conv_forward(int M, int N, int Kp, const ConvOperand& cv, const bf16* W, const float* bias, float* C,
                             bf16* act, hipStream_t s) {
  if (M <= 0 || N <= 0 || Kp <= 0) return hipSuccess;
  GemmArgs g{};
  g.M = M;
  g.N = N;
  g.K = Kp;
  g.kchunk = Kp;
  g.B = W;
  g.sbn = Kp;
  g.sbk = 1;
  g.C = C;
  g.bias = bias;
  g.act = act;
  g.cv = cv;
  hipLaunchKernelGGL((k_gemm<OP_COL, OP_K, true, true>), dim3((M + BM - 1) / BM, (N + BN - 1) / BN, 1), dim3(kT), 0, s, g);
  return hipGetLastError();
}
hipError_t gemm_conv_wgrad(int Co, int Kp, int M, const bf16* dpre, const ConvOperand* cv, const uint8_t* bits, float* C,
                           int splits, hipStream_t s, int* used) {
  if (M <= 0 || Co <= 0 || Kp <= 0) return hipSuccess;
  GemmArgs g{};
  g.M = Co;
  g.N = Kp;
  g.K = M;
  g.kchunk = split_chunk(M, splits, used);
  g.A = dpre;
  g.sam = 1;
  g.sak = Co;
  g.C = C;
  g.bits = bits;
  const dim3 grid((Co + BM - 1) / BM, (Kp + BN - 1) / BN, *used);
  const bool vec = vector_chunks(dpre, Co, Co);
  if (cv) {
    g.cv = *cv;
    if (vec) hipLaunchKernelGGL((k_gemm<OP_ROW, OP_COLT, true, true>), grid, dim3(kT), 0, s, g);
    else hipLaunchKernelGGL((k_gemm<OP_ROW, OP_COLT, false, true>), grid, dim3(kT), 0, s, g);
  } else {
    if (vec) hipLaunchKernelGGL((k_gemm<OP_ROW, OP_BITS, true, true>), grid, dim3(kT), 0, s, g);
    else hipLaunchKernelGGL((k_gemm<OP_ROW, OP_BITS, false, true>), grid, dim3(kT), 0, s, g);
  }
  return hipGetLastError();
}

// number of k-splits that gives each split about `rows` reduction steps
int splits_for(int K, int rows) { return std::max(1, std::min(kMaxSplits, (K + rows - 1) / rows)); }

// ---------------------------------------------------------------------------
// element-wise and gather kernels
// ---------------------------------------------------------------------------
inline unsigned blocks(long long n) { return (unsigned)std::min<long long>((n + kT - 1) / kT, 1 << 20); }

// im2col of a periodic stride-2 3x3x3 window: col[(b,o)][t * Ci + ci] = a[b, (2 o + t - 1) mod n, ci]
// (zero for k >= 27 Ci).  One thread per (output row, tap) copies the tap's Ci channels, 16 bytes
// at a time when Ci is a multiple of 8 (rows of src and col are then 16-byte aligned).
__global__ void k_im2col(const bf16* src, int B, int n, int Ci, int Kp, bf16* col) {
  const int m = n / 2;
  const long long rows = (long long)B * m * m * m;
  const long long tot = rows * 27;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < tot; e += (long long)gridDim.x * blockDim.x) {
    const long long row = e / 27;
    const int t = (int)(e - row * 27);
    const int tz = t / 9, ty = (t / 3) % 3, tx = t % 3;
    long long r = row;
    const int ox = (int)(r % m);
    r /= m;
    const int oy = (int)(r % m);
    r /= m;
    const int oz = (int)(r % m);
    const long long b = r / m;
    const int iz = (2 * oz + tz - 1 + n) % n, iy = (2 * oy + ty - 1 + n) % n, ix = (2 * ox + tx - 1 + n) % n;
    const bf16* sp = src + (((b * n + iz) * n + iy) * n + ix) * Ci;
    bf16* dp = col + row * Kp + (long long)t * Ci;
    if ((Ci & 7) == 0) {
      for (int c = 0; c < Ci; c += 8) *reinterpret_cast<uint4*>(dp + c) = *reinterpret_cast<const uint4*>(sp + c);
    } else {
      for (int c = 0; c < Ci; ++c) dp[c] = sp[c];
    }
    if (t == 26)
      for (int k = 27 * Ci; k < Kp; ++k) col[row * Kp + k] = 0;
  }
}

// x5[b][:] = [bf16(mean over V voxels of gelu(pre4[b])), bf16(feat[b]), 0 ...]
__global__ void k_pool_concat(const float* pre4, int B, int V, int C, const float* feat, int nf, int Kp, bf16* x5) {
  const long long tot = (long long)B * Kp;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < tot; e += (long long)gridDim.x * blockDim.x) {
    const int b = (int)(e / Kp);
    const int k = (int)(e - (long long)b * Kp);
    float v = 0.f;
    if (k < C) {
      for (int i = 0; i < V; ++i) v += gelu(pre4[((long long)b * V + i) * C + k]);
      v /= (float)V;
    } else if (k < C + nf) {
      v = feat[(long long)b * nf + (k - C)];
    }
    x5[e] = to_bf16(v);
  }
}

// y[b][o] = (C[b][o] + bias[o]) * scale[b]
// y = offset + scale (C + bias) per sample (offset, scale nullable)
__global__ void k_output(const float* C, const float* bias, const float* scale, const float* offset, int B, int O,
                         float* y) {
  const long long tot = (long long)B * O;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < tot; e += (long long)gridDim.x * blockDim.x) {
    const int b = (int)(e / O);
    const int o = (int)(e - (long long)b * O);
    float v = C[e] + bias[o];
    if (scale) v *= scale[b];
    if (offset) v += offset[e];
    y[e] = v;
  }
}

// loss = mean (y - t)^2 over B*O (one block, fixed order); dy = 2 (y - t) / (B O)
__global__ void k_loss(const float* y, const float* t, long long n, float* loss, float* dy32, bf16* dyb) {
  __shared__ double red[1024];
  double acc = 0.0;
  const float inv = 2.0f / (float)n;
  for (long long e = threadIdx.x; e < n; e += blockDim.x) {
    const float d = y[e] - t[e];
    acc += (double)d * d;
    dy32[e] = d * inv;
    dyb[e] = to_bf16(d * inv);
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = (float)(red[0] / (double)n);
}

// column sums of X [M][C] (fp32): partial[blk][c] over the block's row range, fixed order
__global__ void k_colsum_partial(const float* X, long long M, int C, long long rows_per_blk, float* partial) {
  __shared__ float red[kT];
  const long long r0 = blockIdx.x * rows_per_blk;
  const long long r1 = std::min(M, r0 + rows_per_blk);
  for (int c0 = 0; c0 < C; c0 += kT) {
    // thread layout: column c0 + (tid mod cw), row group tid / cw
    const int cw = std::min(kT, C - c0);
    const int groups = kT / cw;
    const int tid = threadIdx.x;
    const int c = c0 + tid % cw;
    const int grp = tid / cw;
    float acc = 0.f;
    // 16 rows on their way at a time, added in order
    if (grp < groups) {
      for (long long r = r0 + grp; r < r1; r += 16LL * groups) {
        float x[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = X[std::min(r + (long long)i * groups, r1 - 1) * C + c];
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (r + (long long)i * groups < r1) acc += x[i];
      }
    }
    red[tid] = (grp < groups) ? acc : 0.f;
    __syncthreads();
    if (tid < cw) {
      float s = 0.f;
      for (int gi = 0; gi < groups; ++gi) s += red[gi * cw + tid];
      partial[(long long)blockIdx.x * C + c0 + tid] = s;
    }
    __syncthreads();
  }
}

// dst[c] = sum over blocks of partial[blk][c]: one block per column, thread-strided partial sums
// combined by a fixed tree
__global__ void k_colsum_final(const float* partial, int nb, int C, float* dst) {
  __shared__ float red[kT];
  const int c = blockIdx.x;
  float acc = 0.f;
  for (int i = threadIdx.x; i < nb; i += kT) acc += partial[(long long)i * C + c];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = kT / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) dst[c] = red[0];
}

// out[r][n] = sum over s of P[s][r][n] in order, n < Nvalid, out [rows][ldo].  Few splits: a thread per
// entry.  Many: 16 entries per block, whose splits are fetched side by side, 256 at a time, and then
// added one after the other (a thread per entry waited 64 us for the 256 splits of 32 x 27 entries; the
// other way round, one split of 256 x 3456 entries took 40 us with 16 threads of a block at work).
constexpr int kFewSplits = 32;
__global__ void __launch_bounds__(kT) k_sum_few_splits(const float* P, int S, long long rows, int N, int Nvalid, float* out, int ldo) {
  const long long tot = rows * Nvalid;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < tot; e += (long long)gridDim.x * blockDim.x) {
    const long long r = e / Nvalid;
    const int n = (int)(e - r * Nvalid);
    float s = 0.f;
#pragma unroll 8
    for (int z = 0; z < S; ++z) s += P[((long long)z * rows + r) * N + n];
    out[r * ldo + n] = s;
  }
}
__global__ void __launch_bounds__(kT) k_sum_splits(const float* P, int S, long long rows, int N, int Nvalid, float* out, int ldo) {
  __shared__ float part[256][16];
  const int le = threadIdx.x & 15, z0 = threadIdx.x >> 4;
  const long long tot = rows * Nvalid;
  for (long long base = blockIdx.x * 16LL; base < tot; base += gridDim.x * 16LL) {
    const long long e = std::min(base + le, tot - 1);
    const long long r = e / Nvalid;
    const int n = (int)(e - r * Nvalid);
    float s = 0.f;
    for (int zb = 0; zb < S; zb += 256) {
      const int nz = min(256, S - zb);
#pragma unroll 8
      for (int z = z0; z < nz; z += 16) part[z][le] = P[((long long)(zb + z) * rows + r) * N + n];
      __syncthreads();
      if (z0 == 0) {
#pragma unroll 8
        for (int z = 0; z < nz; ++z) s += part[z][le];
      }
      __syncthreads();
    }
    if (z0 == 0 && base + le < tot) out[r * ldo + n] = s;
  }
}

// dpre = dA * gelu'(pre), fp32 and bf16 copies; dA read as src[r*lds + c]
__global__ void k_gelu_back(const float* src, int lds, const float* pre, long long M, int C, float scale, float* d32,
                            bf16* db) {
  const long long tot = M * C;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < tot; e += (long long)gridDim.x * blockDim.x) {
    const long long r = e / C;
    const int c = (int)(e - r * C);
    const float v = src[r * lds + c] * scale * gelu_grad(pre[e]);
    d32[e] = v;
    db[e] = to_bf16(v);
  }
}

// pooled features back to the voxels of the last conv block: da4[b][v][c] = dx5[b][c] / V
__global__ void k_unpool_back(const float* dx5, int ldx, const float* pre4, int B, int V, int C, float* d32, bf16* db) {
  const long long tot = (long long)B * V * C;
  const float inv = 1.0f / (float)V;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < tot; e += (long long)gridDim.x * blockDim.x) {
    const int c = (int)(e % C);
    const long long b = e / ((long long)V * C);
    const float v = dx5[b * ldx + c] * inv * gelu_grad(pre4[e]);
    d32[e] = v;
    db[e] = to_bf16(v);
  }
}

// Gather of dcol back to the input voxels of a stride-2 periodic layer, times gelu'(pre_in):
// voxel i of an axis of length n is tap t of output o when 2 o + t - 1 = i (mod n), i.e. t = 1
// (o = i/2) for even i and t = 0 (o = (i+1)/2 mod n/2) or t = 2 (o = (i-1)/2) for odd i.
// One thread per (input voxel, group of 4 channels; 1 channel when Ci is not a multiple of 4):
// consecutive threads read consecutive channels of the same dcol rows.
__global__ void k_col2im_gelu(const float* dcol, int B, int n, int Ci, int Kp, const float* pre_in, float* d32,
                              bf16* db) {
  const int m = n / 2;
  const int w = (Ci & 3) == 0 ? 4 : 1;
  const int groups = Ci / w;
  const long long tot = (long long)B * n * n * n * groups;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < tot; e += (long long)gridDim.x * blockDim.x) {
    const long long vox = e / groups;
    const int ci = (int)(e - vox * groups) * w;
    long long r = vox;
    const int ix = (int)(r % n);
    r /= n;
    const int iy = (int)(r % n);
    r /= n;
    const int iz = (int)(r % n);
    const long long b = r / n;
    int tz[2], oz[2], ty[2], oy[2], tx[2], ox[2];
    int nzc, nyc, nxc;
    auto taps = [&](int i, int* t, int* o, int& cnt) {
      if ((i & 1) == 0) {
        t[0] = 1;
        o[0] = i / 2;
        cnt = 1;
      } else {
        t[0] = 0;
        o[0] = ((i + 1) / 2) % m;
        t[1] = 2;
        o[1] = (i - 1) / 2;
        cnt = 2;
      }
    };
    taps(iz, tz, oz, nzc);
    taps(iy, ty, oy, nyc);
    taps(ix, tx, ox, nxc);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int a = 0; a < nzc; ++a)
      for (int c = 0; c < nyc; ++c)
        for (int d = 0; d < nxc; ++d) {
          const long long orow = ((b * m + oz[a]) * m + oy[c]) * m + ox[d];
          const int t = (tz[a] * 3 + ty[c]) * 3 + tx[d];
          const float* src = dcol + orow * Kp + (long long)t * Ci + ci;
          if (w == 4) {
            const float4 v = *reinterpret_cast<const float4*>(src);
            s.x += v.x;
            s.y += v.y;
            s.z += v.z;
            s.w += v.w;
          } else {
            s.x += src[0];
          }
        }
    const long long base = vox * Ci + ci;
    if (w == 4) {
      const float4 pr = *reinterpret_cast<const float4*>(pre_in + base);
      const float o0 = s.x * gelu_grad(pr.x), o1 = s.y * gelu_grad(pr.y), o2 = s.z * gelu_grad(pr.z),
                  o3 = s.w * gelu_grad(pr.w);
      *reinterpret_cast<float4*>(d32 + base) = make_float4(o0, o1, o2, o3);
      const uint2 packed = make_uint2((uint32_t)to_bf16(o0) | ((uint32_t)to_bf16(o1) << 16),
                                      (uint32_t)to_bf16(o2) | ((uint32_t)to_bf16(o3) << 16));
      *reinterpret_cast<uint2*>(db + base) = packed;
    } else {
      const float v = s.x * gelu_grad(pre_in[base]);
      d32[base] = v;
      db[base] = to_bf16(v);
    }
  }
}

// layer blockIdx.y: W [rows][K] fp32 (flat parameter block) -> Wb [rows][Kp] bf16 with zero padding
struct PackArgs {
  const float* W[6];
  bf16* Wb[6];
  int rows[6], K[6], Kp[6];
};
__global__ void k_pack(PackArgs a) {
  const int l = blockIdx.y;
  const int K = a.K[l], Kp = a.Kp[l];
  const long long tot = (long long)a.rows[l] * Kp;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < tot; e += (long long)gridDim.x * blockDim.x) {
    const long long r = e / Kp;
    const int k = (int)(e - r * Kp);
    a.Wb[l][e] = k < K ? to_bf16(a.W[l][r * K + k]) : (bf16)0;
  }
}

__global__ void k_adam(float* p, float* m, float* v, const float* g, long long n, float lr, float b1, float b2, float eps,
                       float bc1, float bc2) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
  }
}

// positive definiteness of a symmetric 6x6 by Cholesky (double)
__device__ bool spd6(const double (*A)[6]) {
  double L[6][6];
  for (int i = 0; i < 6; ++i)
    for (int j = 0; j <= i; ++j) {
      double s = A[i][j];
      for (int k = 0; k < j; ++k) s -= L[i][k] * L[j][k];
      if (i == j) {
        if (!(s > 0.0)) return false;
        L[i][i] = sqrt(s);
      } else {
        L[i][j] = s / L[j][j];
      }
    }
  return true;
}

__device__ void iso6(double lam, double mu, double (*C)[6]) {
  for (int i = 0; i < 6; ++i)
    for (int j = 0; j < 6; ++j) C[i][j] = 0.0;
  for (int i = 0; i < 3; ++i) {
    for (int j = 0; j < 3; ++j) C[i][j] = lam;
    C[i][i] = lam + 2.0 * mu;
    C[i + 3][i + 3] = mu;
  }
}

// one block per sample: volume fraction, Voigt / Reuss bounds, Cholesky tests, feature range
__global__ void k_check(const uint8_t* phase, long long Nv, const float* lm, const float* feat, int nf, float* C21,
                        const float* C2, float tol, float lo, float hi, float max_spread, int* ok, float* spread_out) {
  __shared__ double red[kT];
  const int b = blockIdx.x;
  // 16 phase ids per load where the map is aligned (Nv is a multiple of 4096)
  const uint8_t* pb = phase + (long long)b * Nv;
  long long ones = 0;
  if ((reinterpret_cast<uintptr_t>(pb) & 15u) == 0) {
    const uint4* p4 = reinterpret_cast<const uint4*>(pb);
#pragma unroll 4
    for (long long v = threadIdx.x; v < Nv / 16; v += blockDim.x) {
      const uint4 q = p4[v];
      const uint32_t wd[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // bit 7 of each byte: the byte is not zero
        const uint32_t nz = ((wd[i] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | wd[i];
        ones += __popc(nz & 0x80808080u);
      }
    }
  } else {
    for (long long v = threadIdx.x; v < Nv; v += blockDim.x) ones += pb[v] ? 1 : 0;
  }
  red[threadIdx.x] = (double)ones;
  __syncthreads();
  for (int s = kT / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  const double f1 = red[0] / (double)Nv, f0 = 1.0 - f1;
  const double l0 = lm[4 * b + 0], m0 = lm[4 * b + 1], l1 = lm[4 * b + 2], m1 = lm[4 * b + 3];
  // Voigt: arithmetic means of lam, mu; Reuss (isotropic phases): harmonic means of bulk and shear moduli
  const double lv = f0 * l0 + f1 * l1, mv = f0 * m0 + f1 * m1;
  const double k0 = l0 + 2.0 * m0 / 3.0, k1 = l1 + 2.0 * m1 / 3.0;
  const double kr = 1.0 / (f0 / k0 + f1 / k1), mr = 1.0 / (f0 / m0 + f1 / m1);
  const double lr = kr - 2.0 * mr / 3.0;
  double Cv[6][6], Cr[6][6], Cp[6][6], A[6][6];
  iso6(lv, mv, Cv);
  iso6(lr, mr, Cr);
  // with a second ensemble member: the prediction becomes the mean of the two, and their
  // spread (2-norm of the difference of the 21 components over that of the mean) is tested
  double d2 = 0.0, n2 = 0.0;
  int k = 0;
  for (int i = 0; i < 6; ++i)
    for (int j = i; j < 6; ++j) {
      double c = C21[(long long)b * 21 + k];
      if (C2) {
        const double c2 = C2[(long long)b * 21 + k];
        d2 += (c - c2) * (c - c2);
        c = 0.5 * (c + c2);
        n2 += c * c;
        C21[(long long)b * 21 + k] = (float)c;
      }
      Cp[i][j] = Cp[j][i] = c;
      ++k;
    }
  bool good = spd6(Cp);
  if (C2) good = good && (sqrt(d2) <= (double)max_spread * sqrt(n2));
  if (spread_out) spread_out[b] = C2 ? (float)(sqrt(d2) / fmax(sqrt(n2), 1e-300)) : 0.0f;
  // bounds with a slack of tol |C_Voigt|_F in every direction (prediction errors are measured
  // in that norm; a per-direction relative slack would reject small errors in the soft
  // shear directions)
  double fro = 0.0;
  for (int i = 0; i < 6; ++i)
    for (int j = 0; j < 6; ++j) fro += Cv[i][j] * Cv[i][j];
  const double slack = (double)tol * sqrt(fro);
  for (int i = 0; i < 6; ++i)
    for (int j = 0; j < 6; ++j) A[i][j] = Cv[i][j] - Cp[i][j] + (i == j ? slack : 0.0);
  good = good && spd6(A);
  for (int i = 0; i < 6; ++i)
    for (int j = 0; j < 6; ++j) A[i][j] = Cp[i][j] - Cr[i][j] + (i == j ? slack : 0.0);
  good = good && spd6(A);
  if (nf > 0) {
    const float x = feat[(long long)b * nf];
    good = good && (x >= lo) && (x <= hi);
  }
  ok[b] = good ? 1 : 0;
}

}  // namespace cnn

using namespace cnn;

struct fft_homog_cnn {
  fft_homog_cnn_desc d;
  hipStream_t s;
  char* ws;
  size_t P;
  // parameter blocks: offsets into the flat vector
  size_t offW[7], offB[7];
  int Kc[7], Kp[7], rows[7];  // per layer 1..6: K of the GEMM, padded K, output width
  int edge[5];                // cell edge at the input of conv block l (edge[0] = n), edge[4] = after block 4
  float *p, *m, *v, *g;
  bf16* Wb[7];
  bf16* col[5];
  float* pre[5];
  bf16* act[5];
  bf16 *x5, *h, *dyb, *dAb, *dBb;
  float *pre5, *y, *dy32, *dA, *dB, *dcol, *scratch, *colpart, *lossd;
  int* flag;
  size_t scratch_floats, colpart_floats;
  int step;
  float *h_loss;
  int* h_flag;
  hipEvent_t e0, e1;
  double fwd_ms, train_ms;
};

namespace {

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
int round32(int k) { return (k + 31) / 32 * 32; }

int validate(const fft_homog_cnn_desc* d) {
  if (!d) return FFT_HOMOG_EINVAL;
  if (d->n < 16 || d->n > 128 || d->n % 16 != 0) return FFT_HOMOG_EINVAL;
  if (d->channels[0] != 1) return FFT_HOMOG_EINVAL;
  for (int l = 1; l < 5; ++l)
    if (d->channels[l] < 1 || d->channels[l] > 1024) return FFT_HOMOG_EINVAL;
  if (d->hidden < 1 || d->hidden > 4096 || d->n_feat < 0 || d->n_feat > 32 || d->n_out < 1 || d->n_out > 4096)
    return FFT_HOMOG_EINVAL;
  if (d->max_batch < 1) return FFT_HOMOG_EINVAL;
  // GEMM rows (outputs of block 1 over the batch) are 32-bit
  const long long m1 = d->n / 2;
  if ((long long)d->max_batch * m1 * m1 * m1 > 0x7fffffffLL) return FFT_HOMOG_EINVAL;
  return FFT_HOMOG_OK;
}

struct Plan {
  size_t P, offW[7], offB[7];
  int Kc[7], Kp[7], rows[7], edge[5];
  size_t o_p, o_m, o_v, o_g, o_Wb[7], o_col[5], o_pre[5], o_act[5], o_x5, o_pre5, o_h, o_y, o_dy32, o_dyb, o_dA,
      o_dAb, o_dB, o_dBb, o_dcol, o_scratch, o_colpart, o_loss, o_flag, total;
  size_t scratch_floats, colpart_floats;
};

void plan(const fft_homog_cnn_desc* d, Plan* L) {
  const int* ch = d->channels;
  const long long Bm = d->max_batch;
  size_t k = 0;
  for (int l = 1; l <= 4; ++l) {
    L->rows[l] = ch[l];
    L->Kc[l] = 27 * ch[l - 1];
    L->Kp[l] = round32(L->Kc[l]);
    L->offW[l] = k;
    k += (size_t)ch[l] * L->Kc[l];
    L->offB[l] = k;
    k += ch[l];
  }
  L->rows[5] = d->hidden;
  L->Kc[5] = ch[4] + d->n_feat;
  L->Kp[5] = round32(L->Kc[5]);
  L->offW[5] = k;
  k += (size_t)d->hidden * L->Kc[5];
  L->offB[5] = k;
  k += d->hidden;
  L->rows[6] = d->n_out;
  L->Kc[6] = d->hidden;
  L->Kp[6] = round32(d->hidden);
  L->offW[6] = k;
  k += (size_t)d->n_out * d->hidden;
  L->offB[6] = k;
  k += d->n_out;
  L->P = k;
  L->edge[0] = d->n;
  for (int l = 1; l <= 4; ++l) L->edge[l] = L->edge[l - 1] / 2;

  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes);
    return o;
  };
  L->o_p = take(L->P * 4);
  L->o_m = take(L->P * 4);
  L->o_v = take(L->P * 4);
  L->o_g = take(L->P * 4);
  for (int l = 1; l <= 6; ++l) L->o_Wb[l] = take((size_t)L->rows[l] * L->Kp[l] * 2);
  size_t maxact = 0, maxcol = 0;
  for (int l = 1; l <= 4; ++l) {
    const long long Ml = Bm * (long long)L->edge[l] * L->edge[l] * L->edge[l];
    // block 1 keeps its taps as bits; blocks 2-4 expand their operand only when their input channels
    // are not a multiple of 8 (else the GEMMs gather it, implicit_conv)
    L->o_col[l] = take(l == 1 ? (size_t)Ml * 4 : ch[l - 1] % 8 != 0 ? (size_t)Ml * L->Kp[l] * 2 : 0);
    L->o_pre[l] = take((size_t)Ml * ch[l] * 4);
    L->o_act[l] = take((size_t)Ml * ch[l] * 2);
    maxact = std::max(maxact, (size_t)Ml * ch[l]);
    if (l >= 2 && !(ch[l - 1] % 8 == 0 && ch[l] % 8 == 0)) maxcol = std::max(maxcol, (size_t)Ml * L->Kp[l]);
  }
  maxact = std::max(maxact, (size_t)Bm * std::max(d->hidden, L->Kp[5]));
  L->o_x5 = take((size_t)Bm * L->Kp[5] * 2);
  L->o_pre5 = take((size_t)Bm * d->hidden * 4);
  L->o_h = take((size_t)Bm * d->hidden * 2);
  L->o_y = take((size_t)Bm * d->n_out * 4);
  L->o_dy32 = take((size_t)Bm * d->n_out * 4);
  L->o_dyb = take((size_t)Bm * d->n_out * 2);
  L->o_dA = take(maxact * 4);
  L->o_dAb = take(maxact * 2);
  L->o_dB = take(maxact * 4);
  L->o_dBb = take(maxact * 2);
  L->o_dcol = take(std::max<size_t>(maxcol, 1) * 4);
  // split-K partials of the weight gradients and the dense-layer products
  size_t sc = 0;
  for (int l = 1; l <= 4; ++l) {
    const long long Ml = Bm * (long long)L->edge[l] * L->edge[l] * L->edge[l];
    sc = std::max(sc, (size_t)splits_for((int)Ml, 4096) * L->rows[l] * L->Kp[l]);
  }
  sc = std::max(sc, (size_t)d->hidden * L->Kp[5]);
  sc = std::max(sc, (size_t)d->n_out * d->hidden);
  sc = std::max(sc, (size_t)Bm * std::max(L->Kp[5], std::max(d->hidden, d->n_out)));
  L->scratch_floats = sc;
  L->o_scratch = take(sc * 4);
  const long long M1 = Bm * (long long)L->edge[1] * L->edge[1] * L->edge[1];
  L->colpart_floats = (size_t)((M1 + kColRows - 1) / kColRows + 1) * std::max(std::max(1024, d->n_out), d->hidden);
  L->o_colpart = take(L->colpart_floats * 4);
  L->o_loss = take(64);
  L->o_flag = take(64);
  L->total = off;
}

#define CK(expr)                                        \
  do {                                                  \
    hipError_t e_ = (expr);                             \
    if (e_ != hipSuccess) return FFT_HOMOG_EDEVICE;     \
  } while (0)

// bias gradient: column sums of X [M][C] into dst[C], two fixed-order stages
hipError_t colsum(fft_homog_cnn_t* h, const float* X, long long M, int C, float* dst) {
  const long long rpb = kColRows;
  const long long nb = (M + rpb - 1) / rpb;
  hipLaunchKernelGGL(k_colsum_partial, dim3((unsigned)nb), dim3(kT), 0, h->s, X, M, C, rpb, h->colpart);
  hipLaunchKernelGGL(k_colsum_final, dim3(C), dim3(kT), 0, h->s, h->colpart, (int)nb, C, dst);
  return hipGetLastError();
}

int check_batch(fft_homog_cnn_t* h, int B) { return (B >= 1 && B <= h->d.max_batch) ? FFT_HOMOG_OK : FFT_HOMOG_EINVAL; }

// conv block l > 1 gathers its im2col operand inside the GEMM when its input channels allow
// 16-byte loads of 8 channels
bool implicit_conv(const fft_homog_cnn_t* h, int l) { return l > 1 && h->d.channels[l - 1] % 8 == 0; }
ConvOperand conv_operand(const fft_homog_cnn_t* h, int l) {
  return ConvOperand{h->act[l - 1], h->edge[l - 1], h->d.channels[l - 1], make_div(h->edge[l]), make_div(h->d.channels[l - 1])};
}
// conv block l > 1 whose input gradient is one product per parity class (k_dgrad): rows of 8 channels on
// both sides; else the products of all taps are formed in memory and gathered
bool implicit_dgrad(const fft_homog_cnn_t* h, int l) { return implicit_conv(h, l) && h->d.channels[l] % 8 == 0; }

// forward pass of B samples into h->y (before output scaling is applied by the caller path).  train:
// keep what the gradient needs (pre-activations, block 1's taps)
int forward(fft_homog_cnn_t* h, const uint8_t* phase, const float* feat, int B, bool train) {
  const int* ch = h->d.channels;
  CK(hipMemsetAsync(h->flag, 0, sizeof(int), h->s));
  for (int l = 1; l <= 4; ++l) {
    const int n = h->edge[l - 1];
    const int Ml = (int)((long long)B * h->edge[l] * h->edge[l] * h->edge[l]);
    // the pooling reads block 4's pre-activations, nothing its activations
    float* pre = train || l == 4 ? h->pre[l] : nullptr;
    bf16* act = l < 4 ? h->act[l] : nullptr;
    const float* bias = h->p + h->offB[l];
    if (l == 1) {
      hipLaunchKernelGGL(k_conv_phase, dim3((Ml + kT - 1) / kT), dim3(kT), 0, h->s, phase, Ml, n, make_div(h->edge[1]),
                         h->Wb[1], ch[1], bias, pre, act, train ? (uint8_t*)h->col[1] : nullptr, h->flag);
      CK(hipGetLastError());
    } else if (implicit_conv(h, l)) {
      CK(gemm_conv_forward(Ml, ch[l], h->Kp[l], conv_operand(h, l), h->Wb[l], bias, pre, act, h->s));
    } else {
      hipLaunchKernelGGL(k_im2col, dim3(blocks(Ml * 27LL)), dim3(kT), 0, h->s, h->act[l - 1], B, n, ch[l - 1], h->Kp[l],
                         h->col[l]);
      CK(hipGetLastError());
      CK(gemm(Ml, ch[l], h->Kp[l], h->col[l], h->Kp[l], 1, h->Wb[l], h->Kp[l], 1, pre, 1, h->s, bias, act));
    }
  }
  const int V = h->edge[4] * h->edge[4] * h->edge[4];
  hipLaunchKernelGGL(k_pool_concat, dim3(blocks((long long)B * h->Kp[5])), dim3(kT), 0, h->s, h->pre[4], B, V, ch[4], feat,
                     h->d.n_feat, h->Kp[5], h->x5);
  CK(hipGetLastError());
  CK(gemm(B, h->d.hidden, h->Kp[5], h->x5, h->Kp[5], 1, h->Wb[5], h->Kp[5], 1, train ? h->pre5 : nullptr, 1, h->s,
          h->p + h->offB[5], h->h));
  CK(gemm(B, h->d.n_out, h->d.hidden, h->h, h->d.hidden, 1, h->Wb[6], h->Kp[6], 1, h->scratch, 1, h->s));
  return FFT_HOMOG_OK;
}

int refresh_weights(fft_homog_cnn_t* h) {
  PackArgs a;
  long long most = 0;
  for (int l = 0; l < 6; ++l) {
    a.W[l] = h->p + h->offW[l + 1];
    a.Wb[l] = h->Wb[l + 1];
    a.rows[l] = h->rows[l + 1];
    a.K[l] = h->Kc[l + 1];
    a.Kp[l] = h->Kp[l + 1];
    most = std::max(most, (long long)a.rows[l] * a.Kp[l]);
  }
  hipLaunchKernelGGL(k_pack, dim3(blocks(most), 6), dim3(kT), 0, h->s, a);
  CK(hipGetLastError());
  return FFT_HOMOG_OK;
}

// out = the sum of S split products
hipError_t sum_splits(fft_homog_cnn_t* h, int S, long long rows, int N, int Nvalid, float* out) {
  const unsigned nb = (unsigned)std::min<long long>((rows * Nvalid + 15) / 16, 1 << 20);
  if (S <= kFewSplits)
    hipLaunchKernelGGL(k_sum_few_splits, dim3(blocks(rows * Nvalid)), dim3(kT), 0, h->s, h->scratch, S, rows, N, Nvalid, out, Nvalid);
  else
    hipLaunchKernelGGL(k_sum_splits, dim3(nb), dim3(kT), 0, h->s, h->scratch, S, rows, N, Nvalid, out, Nvalid);
  return hipGetLastError();
}

int read_flag(fft_homog_cnn_t* h) {
  CK(hipMemcpyAsync(h->h_flag, h->flag, sizeof(int), hipMemcpyDeviceToHost, h->s));
  CK(hipStreamSynchronize(h->s));
  return *h->h_flag ? FFT_HOMOG_EINVAL : FFT_HOMOG_OK;
}

}  // namespace

extern "C" {

int fft_homog_cnn_param_count(const fft_homog_cnn_desc* d, size_t* count) {
  if (!count) return FFT_HOMOG_EINVAL;
  int rc = validate(d);
  if (rc) return rc;
  Plan L;
  plan(d, &L);
  *count = L.P;
  return FFT_HOMOG_OK;
}

int fft_homog_cnn_workspace_size(const fft_homog_cnn_desc* d, size_t* bytes) {
  if (!bytes) return FFT_HOMOG_EINVAL;
  int rc = validate(d);
  if (rc) return rc;
  Plan L;
  plan(d, &L);
  *bytes = L.total;
  return FFT_HOMOG_OK;
}

int fft_homog_cnn_create(const fft_homog_cnn_desc* d, void* ws, size_t bytes, void* stream, fft_homog_cnn_t** out) {
  if (!out) return FFT_HOMOG_EINVAL;
  *out = nullptr;
  int rc = validate(d);
  if (rc) return rc;
  Plan L;
  plan(d, &L);
  if (!ws || bytes < L.total || (reinterpret_cast<uintptr_t>(ws) % kAlign) != 0) return FFT_HOMOG_EWORKSPACE;
  fft_homog_cnn_t* h = new fft_homog_cnn();
  h->d = *d;
  h->s = (hipStream_t)stream;
  h->ws = (char*)ws;
  h->P = L.P;
  for (int l = 1; l <= 6; ++l) {
    h->offW[l] = L.offW[l];
    h->offB[l] = L.offB[l];
    h->Kc[l] = L.Kc[l];
    h->Kp[l] = L.Kp[l];
    h->rows[l] = L.rows[l];
    h->Wb[l] = (bf16*)(h->ws + L.o_Wb[l]);
  }
  for (int l = 0; l < 5; ++l) h->edge[l] = L.edge[l];
  h->p = (float*)(h->ws + L.o_p);
  h->m = (float*)(h->ws + L.o_m);
  h->v = (float*)(h->ws + L.o_v);
  h->g = (float*)(h->ws + L.o_g);
  for (int l = 1; l <= 4; ++l) {
    h->col[l] = (bf16*)(h->ws + L.o_col[l]);
    h->pre[l] = (float*)(h->ws + L.o_pre[l]);
    h->act[l] = (bf16*)(h->ws + L.o_act[l]);
  }
  h->x5 = (bf16*)(h->ws + L.o_x5);
  h->pre5 = (float*)(h->ws + L.o_pre5);
  h->h = (bf16*)(h->ws + L.o_h);
  h->y = (float*)(h->ws + L.o_y);
  h->dy32 = (float*)(h->ws + L.o_dy32);
  h->dyb = (bf16*)(h->ws + L.o_dyb);
  h->dA = (float*)(h->ws + L.o_dA);
  h->dAb = (bf16*)(h->ws + L.o_dAb);
  h->dB = (float*)(h->ws + L.o_dB);
  h->dBb = (bf16*)(h->ws + L.o_dBb);
  h->dcol = (float*)(h->ws + L.o_dcol);
  h->scratch = (float*)(h->ws + L.o_scratch);
  h->colpart = (float*)(h->ws + L.o_colpart);
  h->lossd = (float*)(h->ws + L.o_loss);
  h->flag = (int*)(h->ws + L.o_flag);
  h->scratch_floats = L.scratch_floats;
  h->colpart_floats = L.colpart_floats;
  h->step = 0;
  h->fwd_ms = h->train_ms = 0.0;
  h->h_loss = nullptr;
  h->e0 = h->e1 = nullptr;
  hipError_t e = hipHostMalloc((void**)&h->h_loss, 64, 0);
  if (e == hipSuccess) {
    h->h_flag = (int*)(h->h_loss + 4);
    e = hipEventCreate(&h->e0);
  }
  if (e == hipSuccess) e = hipEventCreate(&h->e1);
  if (e == hipSuccess) e = hipMemsetAsync(h->ws, 0, L.o_Wb[1], h->s);  // parameters, moments, gradient
  if (e == hipSuccess) e = hipStreamSynchronize(h->s);
  if (e != hipSuccess) {
    fft_homog_cnn_destroy(h);
    return FFT_HOMOG_EDEVICE;
  }
  if (refresh_weights(h)) {
    fft_homog_cnn_destroy(h);
    return FFT_HOMOG_EDEVICE;
  }
  *out = h;
  return FFT_HOMOG_OK;
}

int fft_homog_cnn_set_params(fft_homog_cnn_t* h, const float* params) {
  if (!h || !params) return FFT_HOMOG_EINVAL;
  CK(hipMemcpyAsync(h->p, params, h->P * 4, hipMemcpyDeviceToDevice, h->s));
  CK(hipMemsetAsync(h->m, 0, h->P * 4, h->s));
  CK(hipMemsetAsync(h->v, 0, h->P * 4, h->s));
  h->step = 0;
  int rc = refresh_weights(h);
  if (rc) return rc;
  CK(hipStreamSynchronize(h->s));
  return FFT_HOMOG_OK;
}

int fft_homog_cnn_get_params(fft_homog_cnn_t* h, float* params) {
  if (!h || !params) return FFT_HOMOG_EINVAL;
  CK(hipMemcpyAsync(params, h->p, h->P * 4, hipMemcpyDeviceToDevice, h->s));
  CK(hipStreamSynchronize(h->s));
  return FFT_HOMOG_OK;
}

int fft_homog_cnn_forward(fft_homog_cnn_t* h, const uint8_t* phase, const float* feat, const float* out_scale,
                          const float* out_offset, float* out,
                          int batch) {
  if (!h || !phase || !out || (h->d.n_feat > 0 && !feat)) return FFT_HOMOG_EINVAL;
  if (check_batch(h, batch)) return FFT_HOMOG_EINVAL;
  CK(hipEventRecord(h->e0, h->s));
  int rc = forward(h, phase, feat, batch, false);
  if (rc) return rc;
  hipLaunchKernelGGL(k_output, dim3(blocks((long long)batch * h->d.n_out)), dim3(kT), 0, h->s, h->scratch,
                     h->p + h->offB[6], out_scale, out_offset, batch, h->d.n_out, out);
  CK(hipGetLastError());
  CK(hipEventRecord(h->e1, h->s));
  rc = read_flag(h);
  float ms = 0.f;
  CK(hipEventElapsedTime(&ms, h->e0, h->e1));
  h->fwd_ms = ms;
  return rc;
}

int fft_homog_cnn_loss_grad(fft_homog_cnn_t* h, const uint8_t* phase, const float* feat, const float* target, int B,
                            float* loss, float* grad) {
  if (!h || !phase || !target || !loss || (h->d.n_feat > 0 && !feat)) return FFT_HOMOG_EINVAL;
  if (check_batch(h, B)) return FFT_HOMOG_EINVAL;
  const int* ch = h->d.channels;
  const int O = h->d.n_out, H = h->d.hidden;
  CK(hipEventRecord(h->e0, h->s));
  int rc = forward(h, phase, feat, B, true);
  if (rc) return rc;
  hipLaunchKernelGGL(k_output, dim3(blocks((long long)B * O)), dim3(kT), 0, h->s, h->scratch, h->p + h->offB[6],
                     nullptr, nullptr, B, O, h->y);
  hipLaunchKernelGGL(k_loss, dim3(1), dim3(1024), 0, h->s, h->y, target, (long long)B * O, h->lossd, h->dy32, h->dyb);
  CK(hipGetLastError());
  // dense output layer: dW6 = dy^T h, db6 = sum dy, dh = dy W6
  CK(gemm(O, H, B, h->dyb, 1, O, h->h, 1, H, h->scratch, 1, h->s));
  CK(sum_splits(h, 1, O, H, H, h->g + h->offW[6]));
  CK(colsum(h, h->dy32, B, O, h->g + h->offB[6]));
  CK(gemm(B, H, O, h->dyb, O, 1, h->Wb[6], 1, h->Kp[6], h->scratch, 1, h->s));
  hipLaunchKernelGGL(k_gelu_back, dim3(blocks((long long)B * H)), dim3(kT), 0, h->s, h->scratch, H, h->pre5, (long long)B,
                     H, 1.0f, h->dA, h->dAb);
  CK(hipGetLastError());
  // hidden layer: dW5 = dpre5^T x5, db5, dx5 = dpre5 W5
  const int K5 = h->Kc[5], Kp5 = h->Kp[5];
  CK(gemm(H, Kp5, B, h->dAb, 1, H, h->x5, 1, Kp5, h->scratch, 1, h->s));
  CK(sum_splits(h, 1, H, Kp5, K5, h->g + h->offW[5]));
  CK(colsum(h, h->dA, B, H, h->g + h->offB[5]));
  CK(gemm(B, ch[4], H, h->dAb, H, 1, h->Wb[5], 1, Kp5, h->scratch, 1, h->s));
  const int V = h->edge[4] * h->edge[4] * h->edge[4];
  hipLaunchKernelGGL(k_unpool_back, dim3(blocks((long long)B * V * ch[4])), dim3(kT), 0, h->s, h->scratch, ch[4],
                     h->pre[4], B, V, ch[4], h->dB, h->dBb);
  CK(hipGetLastError());
  // conv blocks, last to first; dB/dBb hold dpre of block l
  float* d32 = h->dB;
  bf16* db = h->dBb;
  float* n32 = h->dA;
  bf16* nb = h->dAb;
  for (int l = 4; l >= 1; --l) {
    const long long Ml = (long long)B * h->edge[l] * h->edge[l] * h->edge[l];
    const int S = splits_for((int)Ml, 4096);
    int used = 1;
    if (l == 1) {
      CK(gemm_conv_wgrad(ch[l], h->Kp[l], (int)Ml, db, nullptr, (const uint8_t*)h->col[1], h->scratch, S, h->s, &used));
    } else if (implicit_conv(h, l)) {
      const ConvOperand cv = conv_operand(h, l);
      CK(gemm_conv_wgrad(ch[l], h->Kp[l], (int)Ml, db, &cv, nullptr, h->scratch, S, h->s, &used));
    } else {
      CK(gemm(ch[l], h->Kp[l], (int)Ml, db, 1, ch[l], h->col[l], 1, h->Kp[l], h->scratch, S, h->s, nullptr, nullptr, &used));
    }
    CK(sum_splits(h, used, ch[l], h->Kp[l], h->Kc[l], h->g + h->offW[l]));
    CK(colsum(h, d32, Ml, ch[l], h->g + h->offB[l]));
    if (l == 1) break;
    const int nin = h->edge[l - 1];
    if (implicit_dgrad(h, l)) {
      DgradArgs a;
      a.M = (int)Ml;
      a.Ci = ch[l - 1];
      a.Co = ch[l];
      a.Kp = h->Kp[l];
      a.n = nin;
      a.m = make_div(h->edge[l]);
      a.co = make_div(round32(ch[l]));
      a.dpre = db;
      a.W = h->Wb[l];
      a.pre = h->pre[l - 1];
      a.d32 = n32;
      a.db = nb;
      const unsigned gx = (unsigned)((Ml + BM - 1) / BM);
      const dim3 grid(gx, (a.Ci + BN - 1) / BN, 8);
      if (a.Ci <= 32) hipLaunchKernelGGL(k_dgrad<true>, grid, dim3(kT), 0, h->s, a);
      else hipLaunchKernelGGL(k_dgrad<false>, grid, dim3(kT), 0, h->s, a);
    } else {
      CK(gemm((int)Ml, h->Kp[l], ch[l], db, ch[l], 1, h->Wb[l], 1, h->Kp[l], h->dcol, 1, h->s));
      const long long Min = (long long)B * nin * nin * nin;
      hipLaunchKernelGGL(k_col2im_gelu, dim3(blocks(Min * ch[l - 1])), dim3(kT), 0, h->s, h->dcol, B, nin, ch[l - 1],
                         h->Kp[l], h->pre[l - 1], n32, nb);
    }
    CK(hipGetLastError());
    std::swap(d32, n32);
    std::swap(db, nb);
  }
  if (grad) CK(hipMemcpyAsync(grad, h->g, h->P * 4, hipMemcpyDeviceToDevice, h->s));
  CK(hipMemcpyAsync(h->h_loss, h->lossd, 4, hipMemcpyDeviceToHost, h->s));
  CK(hipEventRecord(h->e1, h->s));
  rc = read_flag(h);
  *loss = h->h_loss[0];
  float ms = 0.f;
  CK(hipEventElapsedTime(&ms, h->e0, h->e1));
  h->train_ms = ms;
  return rc;
}

int fft_homog_cnn_adam_step(fft_homog_cnn_t* h, float lr, float beta1, float beta2, float eps) {
  if (!h || !(lr >= 0.f) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
    return FFT_HOMOG_EINVAL;
  h->step += 1;
  const float bc1 = 1.0f - powf(beta1, (float)h->step);
  const float bc2 = 1.0f - powf(beta2, (float)h->step);
  hipLaunchKernelGGL(k_adam, dim3(blocks((long long)h->P)), dim3(kT), 0, h->s, h->p, h->m, h->v, h->g, (long long)h->P, lr,
                     beta1, beta2, eps, bc1, bc2);
  CK(hipGetLastError());
  int rc = refresh_weights(h);
  if (rc) return rc;
  CK(hipStreamSynchronize(h->s));
  return FFT_HOMOG_OK;
}

int fft_homog_cnn_check(fft_homog_cnn_t* h, const uint8_t* phase, const float* lam_mu, const float* feat, float* C,
                        const float* C2, int batch, float tol, float lo, float hi, float max_spread, int* ok,
                        float* spread_out) {
  if (!h || !phase || !lam_mu || !C || !ok || (h->d.n_feat > 0 && !feat)) return FFT_HOMOG_EINVAL;
  if (h->d.n_out != 21) return FFT_HOMOG_EINVAL;
  if (batch < 1) return FFT_HOMOG_EINVAL;
  const long long Nv = (long long)h->d.n * h->d.n * h->d.n;
  hipLaunchKernelGGL(k_check, dim3(batch), dim3(kT), 0, h->s, phase, Nv, lam_mu, feat, h->d.n_feat, C, C2, tol, lo, hi,
                     max_spread, ok, spread_out);
  CK(hipGetLastError());
  CK(hipStreamSynchronize(h->s));
  return FFT_HOMOG_OK;
}

int fft_homog_cnn_last_ms(const fft_homog_cnn_t* h, double* fwd, double* train) {
  if (!h) return FFT_HOMOG_EINVAL;
  if (fwd) *fwd = h->fwd_ms;
  if (train) *train = h->train_ms;
  return FFT_HOMOG_OK;
}

void fft_homog_cnn_destroy(fft_homog_cnn_t* h) {
  if (!h) return;
  if (h->s) (void)hipStreamSynchronize(h->s);
  else (void)hipDeviceSynchronize();
  if (h->h_loss) (void)hipHostFree(h->h_loss);
  if (h->e0) (void)hipEventDestroy(h->e0);
  if (h->e1) (void)hipEventDestroy(h->e1);
  delete h;
}

int fft_homog_cnn_debug_gemm(fft_homog_cnn_t* h, int M, int N, int K, const uint16_t* A, long long sam, long long sak,
                             const uint16_t* B, long long sbn, long long sbk, float* C, int splits) {
  if (!h || !A || !B || !C || M < 1 || N < 1 || K < 1 || splits < 1 || splits > kMaxSplits) return FFT_HOMOG_EINVAL;
  if (!(sak == 1 || sam == 1) || !(sbk == 1 || sbn == 1)) return FFT_HOMOG_EINVAL;
  CK(gemm(M, N, K, A, sam, sak, B, sbn, sbk, C, splits, h->s));
  CK(hipStreamSynchronize(h->s));
  return FFT_HOMOG_OK;
}

}  // extern "C"
