// Host-only checks of the launch geometry under AddressSanitizer and UndefinedBehaviorSanitizer.  Built with
// the library's launch_geometry.cpp by tests/test_host_plans.py.
#include <cstdio>
#include <initializer_list>
#include <vector>

#include "kernels.h"

static int failures = 0;
#define EXPECT(cond)                                                               \
  do {                                                                             \
    if (!(cond)) {                                                                 \
      std::fprintf(stderr, "expectation failed: %s (line %d, n %d)\n", #cond, __LINE__, n); \
      ++failures;                                                                  \
    }                                                                              \
  } while (0)

// every block of the re-indexed grid once, an XCD's blocks (those equal mod 8) consecutive
static void check_xcd_order() {
  for (int n = 1; n <= 3000; ++n) {
    std::vector<int> seen(n, 0);
    unsigned prev[8];
    for (int lin = 0; lin < n; ++lin) {
      const unsigned b = fh::xcd_order(lin, n);
      EXPECT(b < (unsigned)n);
      if (b < (unsigned)n) ++seen[b];
      if (lin >= 8) EXPECT(b == prev[lin & 7] + 1);
      prev[lin & 7] = b;
    }
    for (int b = 0; b < n; ++b) EXPECT(seen[b] == 1);
  }
}

// plans with the chirp-z limits in use; for every length that runs the folded dense DFT in any grid, the bounds
// its kernel relies on
static void check_plans() {
  int n = 0, dense = 0, chirp = 0;
  for (n = 1; n <= fh::kMaxAxis; ++n) {
    for (int ndim : {2, 3})
      for (int axis = 0; axis < ndim; ++axis)
        for (bool small : {false, true}) {
          const int lim = fh::chirp_limit(n, ndim, axis, small);
          fh::AxisPlan pl;
          EXPECT(lim > 0 && fh::make_plan(n, &pl, lim));
          long long prod = 1;
          for (int st = 0; st < pl.nstages; ++st) prod *= pl.radix[st];
          EXPECT(prod == fh::lds_len(pl) && !pl.dense);
          if (pl.m > 0) {
            ++chirp;
            EXPECT(pl.m >= 2 * n - 1 && pl.m <= 2048);
            EXPECT(fh::plan_table_elems(pl) == (size_t)(pl.m + n + pl.m));
          }
          EXPECT(fh::plan_table_stride(pl) % 16 == 0 && fh::plan_table_stride(pl) >= fh::plan_table_elems(pl));
          // what one grid runs, the query over all grids knows of
          for (long long voxels : {1LL, 1LL << 20})
            if (fh::dense_len(n, ndim, axis, small, voxels)) EXPECT(fh::dense_len(n, ndim));
        }
    if (!fh::dense_len(n, 2) && !fh::dense_len(n, 3)) continue;
    ++dense;
    EXPECT(n >= 17 && n <= fh::kDenseMax && fh::fixed_nstages(n) == 0);
    // the last folded input a tile reads, t = 4 steps, and its mirror n - t are rows of the buffer
    EXPECT(4 * fh::dense_steps(n) <= n - 1 && fh::dense_steps(n) % 4 == 0);
    EXPECT(4 * fh::dense_steps(n) >= n / 2);  // every folded input is read
    EXPECT(16 * fh::dense_rows(n) > n / 2);   // every output row has a tile
    EXPECT(fh::dense_elems(n) == (size_t)fh::dense_rows(n) * fh::dense_steps(n) * 64);
    fh::AxisPlan pl;
    EXPECT(fh::make_plan(n, &pl, 0));
    pl.dense = 1;
    EXPECT(fh::plan_table_elems(pl) == (size_t)n + fh::dense_elems(n));
    for (int nseq = 1; nseq <= 512; ++nseq) {
      // in place: no wavefront has more tiles than it holds in registers
      const int tiles = fh::dense_rows(n) * ((nseq + fh::kDenseCols - 1) / fh::kDenseCols);
      const int waves = fh::kThreads / 64;
      if (fh::inplace_ok(pl, nseq)) EXPECT((tiles + waves - 1) / waves <= fh::kDenseHold);
    }
  }
  EXPECT(dense > 100 && chirp > 100);
}

int main() {
  check_xcd_order();
  check_plans();
  std::printf("launch geometry: %d failures\n", failures);
  return failures == 0 ? 0 : 1;
}
