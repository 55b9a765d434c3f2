// Host-only checks of the launch geometry under AddressSanitizer and UndefinedBehaviorSanitizer.  Built with
// the library's launch_geometry.cpp by tests/test_host_plans.py.
#include <cstdio>
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

int main() {
  check_xcd_order();
  std::printf("launch geometry: %d failures\n", failures);
  return failures == 0 ? 0 : 1;
}
