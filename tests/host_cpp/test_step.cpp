// Host unit tests of the step kernels' host-side rules (csrc/wfd_internal.h,
// csrc/wfd_step.hip): the index of the tables that a plane loop reads ahead.
// Built with g++ against libwfd.so and run without a GPU by
// tests/test_host_step.py.
#include <algorithm>
#include <cstdio>

#include "wfd_internal.h"

static int failures = 0;
#define CHECK(cond)                                                        \
  do {                                                                     \
    if (!(cond)) {                                                         \
      std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #cond);          \
      ++failures;                                                          \
    }                                                                      \
  } while (0)

// Every table index of a marching forward block: its loads before the loop, then
// each plane's, for all chunkings of grids of 1 to 40 planes.
static void test_read_ahead() {
  auto fetch = [](int z, int z1, int nz) {
    const int i = wfd::next_plane(z, nz);
    CHECK(i >= 0 && i < nz);
    if (z + 1 < z1) CHECK(i == z + 1);  // the value that the next turn uses
  };
  for (int nz = 1; nz <= 40; ++nz)
    for (int zc = 1; zc <= nz; ++zc)
      for (int z0 = 0; z0 < nz; z0 += zc) {
        const int z1 = std::min(z0 + zc, nz);
        fetch(z0, z1, nz);
        for (int z = z0; z < z1; ++z) fetch(z + 1, z1, nz);
      }
}

int main() {
  test_read_ahead();
  if (failures) return 1;
  std::printf("ALL PASSED\n");
  return 0;
}
