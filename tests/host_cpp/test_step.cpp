// Host unit tests of the kernels' host-side rules (csrc/wfd_internal.h,
// csrc/wfd_step.hip, csrc/wfd_smooth.hip): the index of the tables that a plane
// loop reads ahead, the launches of many blocks, the chunks of a tuned batch, and
// which Laplace lines go through tiles; with an argument, the plans of grids on the
// device.
// Built with g++ against libwfd.so by tests/test_host_step.py.
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

// Laplace lines marched in memory (0) or in tiles of so many lines.
static void test_laplace_rule() {
  // long axes with many lines march, on either side of the rule
  const int64_t march[][3] = {{1, 1300, 40000},  {2, 1300, 40000}, {2, 1000, 40000},
                              {1, 1000, 90000},  {2, 700, 90000},  {1, 400, 250000},
                              {2, 1000, 250000}, {1, 240, 490000}, {2, 1400, 1},
                              {0, 1400, 40000}};
  for (const auto &c : march) CHECK(wfd::tri_tile_lines((int)c[0], (int)c[1], c[2]) == 0);
  // more blocks than a launch takes: planes of 2^30 points and more
  CHECK(wfd::tri_tile_lines(2, 1, int64_t(1) << 30) == 0);
  CHECK(wfd::tri_tile_lines(1, 3, (int64_t(1) << 30) + 5) == 0);
  const int64_t tile[][4] = {{0, 200, 32000, 64}, {1, 200, 32000, 64}, {2, 160, 40000, 64},
                             {0, 1300, 90000, 8}, {1, 816, 40000, 16}, {2, 816, 40000, 16},
                             {1, 600, 90000, 16}, {2, 240, 250000, 64}, {2, 1300, 400, 8}};
  for (const auto &c : tile) CHECK(wfd::tri_tile_lines((int)c[0], (int)c[1], c[2]) == c[3]);
}

// A batch whose contexts ask for rounds of the device: the windows fill it
// together, so that each keeps chunks of 16 planes or more; a single shot takes
// chunks down to 4.
static void test_tuned_batch() {
  constexpr int n = 24;
  wfd::StepGrid g[n];
  wfd::Tuning tu;
  tu.rounds = tu.adj_rounds = 8;
  const wfd::StepGrid *pg[n];
  const wfd::Tuning *pt[n];
  wfd::TileMap maps[n];
  for (int i = 0; i < n; ++i) {
    g[i] = wfd::StepGrid{};
    g[i].nx = 60 + i, g[i].ny = 70, g[i].nz = i ? 50 + i : 9;
    g[i].pitch = 128, g[i].plane = (int64_t)g[i].pitch * g[i].ny, g[i].zs = wfd::kNoSurface;
    pg[i] = &g[i], pt[i] = &tu;
  }
  for (int adj = 0; adj < 2; ++adj) {
    for (int count : {1, n}) {
      if (adj)
        wfd::plan_adjoint(pg + n - count, pt, count, false, maps);
      else
        wfd::plan_forward(pg + n - count, pt, count, true, maps);
      for (int i = 0; i < count; ++i) {
        const int nz = pg[n - count + i]->nz;
        CHECK(maps[i].zc * maps[i].nchunks >= nz && maps[i].zc <= nz);
        CHECK(count == 1 ? maps[i].zc == 4 : maps[i].zc >= std::min(nz, 13));
        CHECK(count == 1 || maps[i].nchunks <= (nz + 15) / 16);
      }
    }
  }
}

// The launches of a count of blocks cover it in order, each under 2^32 threads (the
// CPML layer of a 2050^3 grid with over 380 border cells, x lines: 2050 * 2050
// blocks of 1024).
static void test_launches() {
  const int64_t counts[] = {1, 4194303, 4194304, 2050 * 2050, 20000000};
  for (int64_t blocks : counts)
    for (int threads : {256, 512, 1024}) {
      int64_t next = 0;
      wfd::for_launches(blocks, threads, [&](uint32_t first, uint32_t count) {
        CHECK(first == next && count > 0);
        CHECK((uint64_t)count * threads < (uint64_t(1) << 32));
        next += count;
      });
      CHECK(next == blocks);
    }
}

// The batch descriptors inside a shot's workspace: no larger than when its sizes
// were published, which callers may have kept.
static void test_workspace_structs() {
  CHECK(sizeof(wfd::GradWindow) <= 328);
  CHECK(sizeof(wfd::WindowStep) <= 224);
}

// The plans of padded grids on the device (MI355X): the shapes that
// tests/test_gpu_batch.py compares bitwise, for one shot and a batch of three.
struct Plan {
  int fwd, fwd_stream, spread, adj, adj_stream;
};
static void test_device_plans() {
  const struct {
    int nx, ny, nz;
    Plan one, three;
  } cases[] = {
      {176, 176, 176, {0, 0, 0, 3, 0}, {0, 1, 0, 3, 1}},
      {160, 200, 176, {5, 0, 0, 4, 0}, {1, 1, 0, 0, 1}},
      {90, 180, 260, {5, 0, 0, 4, 0}, {5, 0, 0, 4, 1}},
      {97, 300, 200, {0, 0, 0, 0, 0}, {1, 1, 0, 0, 1}},
      {420, 400, 400, {1, 1, 1, 0, 1}, {1, 1, 0, 0, 1}},
  };
  for (const auto &c : cases)
    for (int zs : {wfd::kNoSurface, 8}) {
      const float k = 0.0f;
      wfd::StepGrid g{};
      g.nx = c.nx, g.ny = c.ny, g.nz = c.nz, g.pitch = (c.nx + 63) / 64 * 64;
      g.plane = (int64_t)g.pitch * c.ny, g.zs = zs, g.k = &k, g.m2 = &k;
      const wfd::Tuning tu;
      const wfd::StepGrid *pg[3] = {&g, &g, &g};
      const wfd::Tuning *pt[3] = {&tu, &tu, &tu};
      for (int n : {1, 3}) {
        const Plan &want = n == 1 ? c.one : c.three;
        wfd::TileMap f[3], a[3];
        const wfd::StepPlan pf = wfd::plan_forward(pg, pt, n, true, f);
        const wfd::StepPlan pa = wfd::plan_adjoint(pg, pt, n, false, a);
        CHECK(pf.shape == want.fwd && pf.stream == want.fwd_stream && f[0].spread == want.spread);
        CHECK(pa.shape == want.adj && pa.stream == want.adj_stream);
      }
    }
}

int main(int argc, char **) {
  if (argc > 1) {
    test_device_plans();
    if (!failures) std::printf("ALL PASSED\n");
    return failures != 0;
  }
  test_workspace_structs();
  test_launches();
  test_tuned_batch();
  test_read_ahead();
  test_laplace_rule();
  if (failures) return 1;
  std::printf("ALL PASSED\n");
  return 0;
}
