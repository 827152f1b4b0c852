// Leapfrog step kernels for gfx950 (MI355X): the eighth-order 25-point star
// (arXiv 2502.12350, §2.1) in a z-marching, LDS-tiled form.
//
// A block owns a TX x TY column tile of the padded grid (TX = XW NI, TY = NG RY)
// and a chunk of z planes: each thread holds NI column groups (x = x0 + lane +
// XW i) of RY consecutive rows, so every global access is a 256-byte row
// segment (128 bytes for XW = 32).  Each thread keeps, for each of its points,
// the nine z-neighbours in a register queue; the current plane with a 4-cell
// x/y halo is staged in LDS (double-buffered: one barrier per plane).  Queue
// entries and pointwise streams are fetched ahead (forward two iterations,
// adjoint one), the halo with the interior of its plane through a register
// delay line.  Small grids' forward blocks take four planes at once instead of
// marching.  A planner chooses tile, chunks and cache hints for each launch.
//
// HBM traffic per point: forward 16 B (constant density) / 20 B (variable
// density); adjoint + imaging 28 B / 32 B (+ 8 B with illumination).
#include <algorithm>
#include <climits>
#include <cmath>
#include <type_traits>
#include <vector>

#include "wfd_internal.h"

namespace wfd {
namespace {

constexpr float W0 = -205.0f / 72.0f;
constexpr float W1 = 8.0f / 5.0f;
constexpr float W2 = -1.0f / 5.0f;
constexpr float W3 = 8.0f / 315.0f;
constexpr float W4 = -1.0f / 560.0f;

// Calls f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>):
// a compile-time index for register-array access in unrolled loops.
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

// A tile is NG row groups of XW lanes (64: a row group is a wavefront; 32: half
// of one); each thread owns NI column groups of RY rows.
template <int RY_, int NG_, int NI_, int XW_>
struct Tile {
  static constexpr int RY = RY_, NG = NG_, NI = NI_, XW = XW_;
  static constexpr int NTHREADS = XW * NG;
  static constexpr int TX = XW * NI;
  static constexpr int TY = NG * RY;
  static constexpr int NP = RY * NI;  // points per thread: p = j * NI + i
  static constexpr int LX = TX + 8;
  static constexpr int LY = TY + 8;
  static constexpr int NHALO = 8 * TX + 8 * TY;  // y-halo rows + x-halo columns
  static constexpr int HPT = (NHALO + NTHREADS - 1) / NTHREADS;
};

// Block -> (tile x, tile y, z chunk).  Logical tiles are numbered x fastest,
// then y, then z chunk; XCD k (= blockIdx mod 8) gets one contiguous range, so
// that neighbouring tiles share their halos in one L2, or, where m.spread is
// set, the blocks run in tile order over all XCDs: the device then reads each
// plane as a few contiguous stretches, which memory far beyond the last-level
// cache prefers (576^3 VD forward, 64 x 32 tiles: 688 against 728 us; 448^3 322 /
// 331; 390 x 340 x 320, under 1 GB a step, 158 / 154; 296^3 97 / 95).
__device__ __forceinline__ void tile_of(const TileMap &m, int b, int &tx, int &ty, int &tz) {
  const int nb = m.nblocks;
  const int per = nb / 8, rem = nb % 8;
  const int xcd = b % 8, slot = b / 8;
  const int logical =
      m.spread ? b
               : (xcd < rem ? xcd * (per + 1) + slot
                            : rem * (per + 1) + (xcd - rem) * per + slot);
  tx = logical % m.tiles_x;
  const int r = logical / m.tiles_x;
  ty = r % m.tiles_y;
  tz = r / m.tiles_y;
}

// Halo element h of a tile plane: global (gx, gy) and its LDS row / column.
template <class T, int K>
__device__ __forceinline__ void halo_slot(int h, int x0, int y0, int &gx, int &gy, int &lrow,
                                          int &lcol) {
  constexpr int TX = T::TX;
  constexpr int TY = T::TY;
  if (h < 8 * TX) {  // four rows above and four below the tile
    const int r = h / TX, col = h % TX;
    gx = x0 + col;
    lcol = 4 + col;
    if (r < 4) {
      gy = y0 - 4 + r;
      lrow = r;
    } else {
      gy = y0 + TY + (r - 4);
      lrow = TY + r;
    }
  } else {  // four columns left and four right of each tile row
    const int hh = h - 8 * TX;
    const int row = hh / 8, c = hh % 8;
    gy = y0 + row;
    lrow = 4 + row;
    if (c < 4) {
      gx = x0 - 4 + c;
      lcol = c;
    } else {
      gx = x0 + TX + (c - 4);
      lcol = TX + c;
    }
  }
}

// Single-use streams (previous state, coefficients, gradient) bypass the
// cache's normal retention so that L2 keeps the stenciled planes.
template <bool NT>
__device__ __forceinline__ float ld_once(const float *p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  return *p;
}
// The adjoint's form: a lane outside the grid (or a plane past the chunk)
// reads the field's first element and drops the value instead of skipping
// the load.  Together with the branch-free stores below and the sponge factor
// read a plane ahead this took the 576^3 adjoint step from 1218 to 1158 us.
template <bool NT>
__device__ __forceinline__ float ld_stream_nb(const float *f, const StepGrid &g, int z,
                                              uint32_t o, bool ok) {
  const float v = ld_once<NT>(f + (ok ? (int64_t)z * g.plane + o : 0));
  return ok ? v : 0.0f;
}
// Nontemporal store of one value per lane into plane z of a field through a
// buffer resource over that plane (under 2^32 bytes: the host caps a pitched
// plane below 2^30 points).  A lane outside the grid passes kDropOffset, past
// every plane, and the hardware drops its store, so the store needs no
// branch (the adjoint's stores).
constexpr uint32_t kDropOffset = 0xFFFFFFF0u;
template <bool NT>
__device__ __forceinline__ void st_plane(float *f, const StepGrid &g, int z, uint32_t ob,
                                         float v) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
      f + (int64_t)z * g.plane, (short)0, (int)(uint32_t)(g.plane * 4), 0x00020000);
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, ob, 0, NT ? 2 /* nt */ : 0);
}

// Sums of the x, y and z second differences (before 1/h^2 weights) of the point
// in row J, column group I of the thread, on the plane whose z neighbours are
// q[point][Z .. Z + 8] and whose tile with halo is staged in s.
template <class T, int J, int I, int Z, int NQ>
__device__ __forceinline__ void point_diffs(const float (&q)[T::NP][NQ],
                                            const float (*s)[T::LX], int wave, int lane,
                                            float &sx, float &sy, float &sz) {
  constexpr int RY = T::RY, NI = T::NI, P = J * NI + I;
  const int ly = 4 + wave * RY + J, lx = 4 + T::XW * I + lane;
  const float *row = s[ly];
  sx = W1 * (row[lx - 1] + row[lx + 1]) + W2 * (row[lx - 2] + row[lx + 2]) +
       W3 * (row[lx - 3] + row[lx + 3]) + W4 * (row[lx - 4] + row[lx + 4]);
  float up[4], dn[4];
#pragma unroll
  for (int k = 1; k <= 4; ++k) {
    up[k - 1] = (J - k >= 0) ? q[((J - k >= 0) ? J - k : 0) * NI + I][Z + 4] : s[ly - k][lx];
    dn[k - 1] = (J + k < RY) ? q[((J + k < RY) ? J + k : 0) * NI + I][Z + 4] : s[ly + k][lx];
  }
  sy = W1 * (up[0] + dn[0]) + W2 * (up[1] + dn[1]) + W3 * (up[2] + dn[2]) + W4 * (up[3] + dn[3]);
  sz = W1 * (q[P][Z + 3] + q[P][Z + 5]) + W2 * (q[P][Z + 2] + q[P][Z + 6]) +
       W3 * (q[P][Z + 1] + q[P][Z + 7]) + W4 * (q[P][Z] + q[P][Z + 8]);
}

// The adjoint's per-thread view of one stenciled field: register queue + halo
// staging.
// The halo of a plane is loaded together with the plane's interior (five
// planes ahead of its use), when the neighbouring tiles load the same lines
// as their interior, and waits in a register delay line; loading it one plane
// ahead instead needed L2 to keep four planes of every resident tile, and the
// adjoint (two stenciled fields) then re-read its halo from HBM.
// DL is the delay-line depth: the halo of plane z is loaded DL planes before
// it is staged (5: with the interior of that plane; 1: one plane ahead).
// K tags the kernel family (0 forward, 1 adjoint) of the tile helpers: with
// shared ones, hipcc allocated the adjoint 137 VGPRs instead of 123 once a
// forward shape used the same tile, dropping it from 4 to 3 waves per SIMD.
// FS: the grid may have a free surface.  Without one, plane loads carry no
// image branch: a uniform branch in every load cost 7 % of the step time.
template <class T, int K, bool FS, int DL = 5>
struct Marcher {
  static constexpr int NP = T::NP, RY = T::RY, NI = T::NI, XW = T::XW;
  float q[NP][9];        // planes z-4 .. z+4 of the thread's points
  float nxt[NP];         // plane z+5 (in flight)
  float hq[DL][T::HPT];  // halo of planes z .. z+DL-1 (hq[0] is staged next)

  // Plane z of the field at offset o: zero past the grid, and above a free
  // surface the negated mirror image about it.
  __device__ __forceinline__ static float ld(const float *f, const StepGrid &g, int z, uint32_t o,
                                             bool ok) {
    if (FS && z < g.zs) {
      const int zm = 2 * g.zs - z;
      return (ok && zm < g.nz) ? -f[(int64_t)zm * g.plane + o] : 0.0f;
    }
    const bool in = ok && z >= 0 && z < g.nz;
    const float v = f[in ? (int64_t)z * g.plane + o : 0];  // as ld_stream_nb
    return in ? v : 0.0f;
  }
  __device__ __forceinline__ void prime(const float *f, const StepGrid &g, int z0,
                                        const uint32_t *off, const bool *in,
                                        const uint32_t *hoff, const bool *hin) {
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int i = 0; i < 9; ++i) q[p][i] = ld(f, g, z0 - 4 + i, off[p], in[p]);
#pragma unroll
    for (int d = 0; d < DL; ++d)
#pragma unroll
      for (int i = 0; i < T::HPT; ++i) hq[d][i] = ld(f, g, z0 + d, hoff[i], hin[i]);
  }
  __device__ __forceinline__ void stage(float (*s)[T::LX], int wave, int lane,
                                        const int *hslot) {
#pragma unroll
    for (int j = 0; j < RY; ++j)
#pragma unroll
      for (int i = 0; i < NI; ++i) s[4 + wave * RY + j][4 + XW * i + lane] = q[j * NI + i][4];
#pragma unroll
    for (int i = 0; i < T::HPT; ++i)
      if (hslot[i] >= 0) (&s[0][0])[hslot[i]] = hq[0][i];
  }
  // After stage(): the interior of plane z+5 and the halo of plane z+DL.
  __device__ __forceinline__ void fetch(const float *f, const StepGrid &g, int z,
                                        const uint32_t *off, const bool *in,
                                        const uint32_t *hoff, const bool *hin) {
#pragma unroll
    for (int p = 0; p < NP; ++p) nxt[p] = ld(f, g, z + 5, off[p], in[p]);
#pragma unroll
    for (int d = 0; d < DL - 1; ++d)
#pragma unroll
      for (int i = 0; i < T::HPT; ++i) hq[d][i] = hq[d + 1][i];
#pragma unroll
    for (int i = 0; i < T::HPT; ++i) hq[DL - 1][i] = ld(f, g, z + DL, hoff[i], hin[i]);
  }
  __device__ __forceinline__ void shift() {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
#pragma unroll
      for (int i = 0; i < 8; ++i) q[p][i] = q[p][i + 1];
      q[p][8] = nxt[p];
    }
  }
  // Sum of the x, y and z second differences (before 1/h^2 weights) of the
  // point in row J, column group I of the thread.
  template <int J, int I>
  __device__ __forceinline__ void diffs(const float (*s)[T::LX], int wave, int lane, float &sx,
                                        float &sy, float &sz) const {
    point_diffs<T, J, I, 0>(q, s, wave, lane, sx, sy, sz);
  }
};

// Common per-thread tile geometry.
template <class T, int K>
struct Geo {
  static constexpr int NP = T::NP, RY = T::RY, NI = T::NI, XW = T::XW;
  int lane, wave, x0, y0, z0, z1;
  int xs[NI];     // x of column group i
  int yv[RY];     // y of row j
  bool in[NP];
  uint32_t off[NP];
  uint32_t hoff[T::HPT];
  bool hin[T::HPT];
  int hslot[T::HPT];

  __device__ __forceinline__ bool init(const StepGrid &g, const TileMap &map, int b) {
    int tx, ty, tz;
    tile_of(map, b, tx, ty, tz);
    z0 = tz * map.zc;
    z1 = min(z0 + map.zc, g.nz);
    lane = threadIdx.x % XW;
    wave = threadIdx.x / XW;
    x0 = tx * T::TX;
    y0 = ty * T::TY;
#pragma unroll
    for (int i = 0; i < NI; ++i) xs[i] = x0 + XW * i + lane;
#pragma unroll
    for (int j = 0; j < RY; ++j) yv[j] = y0 + wave * RY + j;
#pragma unroll
    for (int j = 0; j < RY; ++j)
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int p = j * NI + i;
        in[p] = xs[i] < g.nx && yv[j] < g.ny;
        off[p] = in[p] ? (uint32_t)yv[j] * (uint32_t)g.pitch + (uint32_t)xs[i] : 0u;
      }
#pragma unroll
    for (int i = 0; i < T::HPT; ++i) {
      const int h = threadIdx.x + i * T::NTHREADS;
      if (h < T::NHALO) {
        int gx, gy, lrow, lcol;
        halo_slot<T, K>(h, x0, y0, gx, gy, lrow, lcol);
        hin[i] = gx >= 0 && gx < g.nx && gy >= 0 && gy < g.ny;
        hoff[i] = hin[i] ? (uint32_t)gy * (uint32_t)g.pitch + (uint32_t)gx : 0u;
        hslot[i] = lrow * T::LX + lcol;
      } else {
        hin[i] = false;
        hoff[i] = 0u;
        hslot[i] = -1;
      }
    }
    return z0 < g.nz;
  }
};

// Receiver nodes of one column, walked in z order: the next one's plane and the
// sum of the residuals injected there (res_row holds them node by node).  Both
// are read when the cursor gets there, at the latest with the block's first
// loads: read at the node's own plane, the chain column -> node -> residuals
// held every wavefront of the plane for three memory latencies.
struct ColCursor {
  int e, ee, ez;
  float sum;
  __device__ __forceinline__ void load(const RecTable &rec, const float *__restrict__ res_row,
                                       int z0) {
    ez = INT_MAX;
    for (; e < ee; ++e) {
      const int z = rec.ent_z[e], r0 = rec.ent_rp[e], r1 = rec.ent_rp[e + 1];
      if (z < z0) continue;
      sum = 0.0f;
      for (int r = r0; r < r1; ++r) sum += res_row[r];
      ez = z;
      break;
    }
  }
  __device__ __forceinline__ void init(const RecTable &rec, const float *__restrict__ res_row,
                                       int col, int z0, bool ok) {
    e = ok ? rec.col_start[col] : 0;
    ee = ok ? rec.col_start[col + 1] : 0;
    load(rec, res_row, z0);
  }
  __device__ __forceinline__ void advance(const RecTable &rec, const float *__restrict__ res_row) {
    ++e;
    load(rec, res_row, 0);
  }
};

// Recording.  Sample n - 1 is read from w^n, the current state of step n, by
// blocks of their own beside the step's: a recording in the blocks that write
// w^{n+1} held the plane of the receivers for four dependent memory latencies
// (80^3, a receiver every 8 cells: 9.0 us a step, 7.5 without).
constexpr int kRecordBlock = 256;
__device__ __forceinline__ void record_block(const Record &rec, const float *__restrict__ field,
                                             float *__restrict__ row, int b) {
  const int r = b * kRecordBlock + threadIdx.x;
  if (threadIdx.x < kRecordBlock && r < rec.nrec) row[r] = rec.scale[r] * field[rec.idx[r]];
}
int record_blocks(int nrec) { return (nrec + kRecordBlock - 1) / kRecordBlock; }

// One LDS plane of a tile with its halo.
template <class T>
using LdsPlane = float[T::LY][T::LX];

// Plane z of a field as a buffer: reads at a lane's offset in bytes, zero past
// the plane (a lane outside the grid passes kDropOffset) and on planes outside
// the grid (an empty buffer), without branches or address arithmetic per lane.
// Above a free surface the mirror plane; its sign is image_sign's.
template <bool FS>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_of(const float *f, const StepGrid &g,
                                                           int z, bool more = true) {
  if (FS && z < g.zs) z = 2 * g.zs - z;
  const bool in = more && z >= 0 && z < g.nz;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(f) + (in ? (int64_t)z * g.plane : 0),
                                           (short)0, in ? (int)(uint32_t)(g.plane * 4) : 0,
                                           0x00020000);
}
template <bool NT>
__device__ __forceinline__ float ld_plane(__amdgpu_buffer_rsrc_t r, uint32_t ob) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, ob, 0, NT ? 2 : 0));
}
template <bool FS>
__device__ __forceinline__ float image(const StepGrid &g, int z, float v) {
  return FS && z < g.zs ? -v : v;
}

// What the plane loop of a forward tile loads two planes ahead.
template <class T>
struct InFlight {
  float q[T::NP], h[T::HPT];                // w: interior and halo of plane z + 6
  float p[T::NP], k[T::NP], m[T::NP], gz;  // streams of plane z + 2
};

// One leapfrog step over tile block b of a grid.  The loads of an iteration are
// used at the end of the next one: two sets of registers take turns, since
// moving a register waits for its load.  Loads carry no branch, so that the
// compiler's wait counts are exact.  (One plane ahead, and with the sponge
// factor loaded in the plane that used it, every plane waited for all of its
// own loads: 296^3 VD 102 us instead of 92, 240 x 240 x 200 CD 38 instead of 33.)
template <class T, bool VD, bool FS, bool NT>
__device__ __forceinline__ void forward_tile(
    LdsPlane<T> *sm, const StepGrid &g,
    const float *__restrict__ cur, const float *prev, float *out, const Source &src, int n,
    const TileMap &map, int b) {
  constexpr int NP = T::NP, RY = T::RY, NI = T::NI, HPT = T::HPT, DL = 5;
  Geo<T, 0> geo;
  if (!geo.init(g, map, b)) return;
  uint32_t ob[NP], hb[HPT];
#pragma unroll
  for (int p = 0; p < NP; ++p) ob[p] = geo.in[p] ? 4u * geo.off[p] : kDropOffset;
#pragma unroll
  for (int i = 0; i < HPT; ++i) hb[i] = geo.hin[i] ? 4u * geo.hoff[i] : kDropOffset;
  float q[NP][9], hq[DL][HPT], pv[NP], kv[NP], mv[NP], gz;
  auto fetch = [&](InFlight<T> &f, int z) {  // for the plane loop's iteration z - 1
    const auto rw = plane_of<FS>(cur, g, z + 5);
    const bool more = z + 1 < geo.z1;
    const auto rp = plane_of<false>(prev, g, z + 1, more), rk = plane_of<false>(g.k, g, z + 1, more);
#pragma unroll
    for (int p = 0; p < NP; ++p) f.q[p] = ld_plane<false>(rw, ob[p]);
#pragma unroll
    for (int i = 0; i < HPT; ++i) f.h[i] = ld_plane<false>(rw, hb[i]);
#pragma unroll
    for (int p = 0; p < NP; ++p) f.p[p] = ld_plane<NT>(rp, ob[p]);
#pragma unroll
    for (int p = 0; p < NP; ++p) f.k[p] = ld_plane<NT>(rk, ob[p]);
    if constexpr (VD) {
      const auto rm = plane_of<false>(g.m2, g, z + 1, more);
#pragma unroll
      for (int p = 0; p < NP; ++p) f.m[p] = ld_plane<NT>(rm, ob[p]);
    }
    f.gz = g.gz[next_plane(z, g.nz)];
  };
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const int z = geo.z0 - 4 + i;
    const auto r = plane_of<FS>(cur, g, z);
#pragma unroll
    for (int p = 0; p < NP; ++p) q[p][i] = image<FS>(g, z, ld_plane<false>(r, ob[p]));
    if (i >= 4) {
#pragma unroll
      for (int k = 0; k < HPT; ++k) hq[i - 4][k] = image<FS>(g, z, ld_plane<false>(r, hb[k]));
    }
  }
  {
    const auto rp = plane_of<false>(prev, g, geo.z0), rk = plane_of<false>(g.k, g, geo.z0);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      pv[p] = ld_plane<NT>(rp, ob[p]);
      kv[p] = ld_plane<NT>(rk, ob[p]);
      mv[p] = VD ? ld_plane<NT>(plane_of<false>(g.m2, g, geo.z0), ob[p]) : 0.0f;
    }
    gz = g.gz[geo.z0];
  }
  InFlight<T> f0, f1;
  fetch(f1, geo.z0);
  float gxv[NI], gyv[RY];
#pragma unroll
  for (int i = 0; i < NI; ++i) gxv[i] = geo.xs[i] < g.nx ? g.gx[geo.xs[i]] : 0.0f;
#pragma unroll
  for (int j = 0; j < RY; ++j) gyv[j] = geo.yv[j] < g.ny ? g.gy[geo.yv[j]] : 0.0f;
  const float sigma = src.sigma[0], wavelet = src.wavelet[n];
  const float c0 = W0 * (g.cx + g.cy + g.cz);

  auto plane = [&](int z, InFlight<T> &next, const InFlight<T> &ready) {
    float(*s)[T::LX] = sm[z & 1];
#pragma unroll
    for (int j = 0; j < RY; ++j)
#pragma unroll
      for (int i = 0; i < NI; ++i)
        s[4 + geo.wave * RY + j][4 + T::XW * i + geo.lane] = q[j * NI + i][4];
#pragma unroll
    for (int i = 0; i < HPT; ++i)
      if (geo.hslot[i] >= 0) (&s[0][0])[geo.hslot[i]] = hq[0][i];
    fetch(next, z + 1);
    __syncthreads();
    const auto ro = __builtin_amdgcn_make_buffer_rsrc(
        out + (int64_t)z * g.plane, (short)0, (int)(uint32_t)(g.plane * 4), 0x00020000);
    static_for<RY>([&](auto Jc) {
      constexpr int J = decltype(Jc)::value;
      static_for<NI>([&](auto Ic) {
        constexpr int I = decltype(Ic)::value;
        constexpr int P = J * NI + I;
        float sx, sy, sz;
        point_diffs<T, J, I, 0>(q, s, geo.wave, geo.lane, sx, sy, sz);
        const float c = q[P][4];
        const float lap = c0 * c + g.cx * sx + g.cy * sy + g.cz * sz;
        float acc = VD ? 2.0f * c + kv[P] * (lap - mv[P] * c) : 2.0f * c + kv[P] * lap;
        if (z == src.z && ob[P] == src.offset) acc = __builtin_fmaf(sigma, wavelet, acc);
        const float G = gxv[I] * gyv[J] * gz;
        const float o = (!FS || z > g.zs) ? G * (acc - G * pv[P]) : 0.0f;  // zero at/above a free surface
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o), ro, ob[P], 0, NT ? 2 : 0);
      });
    });
    // to plane z + 1
#pragma unroll
    for (int p = 0; p < NP; ++p) {
#pragma unroll
      for (int i = 0; i < 8; ++i) q[p][i] = q[p][i + 1];
      q[p][8] = image<FS>(g, z + 5, ready.q[p]);
      pv[p] = ready.p[p];
      kv[p] = ready.k[p];
      if (VD) mv[p] = ready.m[p];
    }
#pragma unroll
    for (int d = 0; d < DL - 1; ++d)
#pragma unroll
      for (int i = 0; i < HPT; ++i) hq[d][i] = hq[d + 1][i];
#pragma unroll
    for (int i = 0; i < HPT; ++i) hq[DL - 1][i] = image<FS>(g, z + 5, ready.h[i]);
    gz = ready.gz;
  };
  for (int z = geo.z0; z < geo.z1; z += 2) {
    plane(z, f0, f1);
    if (z + 1 >= geo.z1) break;
    plane(z + 1, f1, f0);
  }
}

// The same step over a block of a tile times ZC planes that does not march: every
// load of the block is issued before its one barrier, so that the block takes
// about one memory latency instead of one per plane.
template <class T, int ZC, bool VD, bool FS, bool NT>
__device__ __forceinline__ void forward_slab(
    LdsPlane<T> *sm, const StepGrid &g, const float *__restrict__ cur, const float *prev,
    float *out, const Source &src, int n, const TileMap &map, int b) {
  constexpr int NP = T::NP, RY = T::RY, NI = T::NI;
  Geo<T, 0> geo;
  if (!geo.init(g, map, b)) return;
  float q[NP][ZC + 8], h[ZC][T::HPT], pv[ZC][NP], kv[ZC][NP], mv[ZC][NP];
  uint32_t ob[NP], hb[T::HPT];
#pragma unroll
  for (int p = 0; p < NP; ++p) ob[p] = geo.in[p] ? 4u * geo.off[p] : kDropOffset;
#pragma unroll
  for (int i = 0; i < T::HPT; ++i) hb[i] = geo.hin[i] ? 4u * geo.hoff[i] : kDropOffset;
#pragma unroll
  for (int i = 0; i < ZC + 8; ++i) {
    const int z = geo.z0 - 4 + i;
    const auto r = plane_of<FS>(cur, g, z);
#pragma unroll
    for (int p = 0; p < NP; ++p) q[p][i] = image<FS>(g, z, ld_plane<false>(r, ob[p]));
    if (i >= 4 && i < ZC + 4) {
#pragma unroll
      for (int k = 0; k < T::HPT; ++k)
        h[i >= 4 && i < ZC + 4 ? i - 4 : 0][k] = image<FS>(g, z, ld_plane<false>(r, hb[k]));
    }
  }
#pragma unroll
  for (int z = 0; z < ZC; ++z) {
    const bool more = geo.z0 + z < geo.z1;
    const auto rp = plane_of<false>(prev, g, geo.z0 + z, more),
               rk = plane_of<false>(g.k, g, geo.z0 + z, more);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      pv[z][p] = ld_plane<NT>(rp, ob[p]);
      kv[z][p] = ld_plane<NT>(rk, ob[p]);
      mv[z][p] = VD ? ld_plane<NT>(plane_of<false>(g.m2, g, geo.z0 + z, more), ob[p]) : 0.0f;
    }
  }
  const float sigma = src.sigma[0], wavelet = src.wavelet[n];
  float gzv[ZC];
#pragma unroll
  for (int z = 0; z < ZC; ++z) gzv[z] = g.gz[min(geo.z0 + z, g.nz - 1)];
  float gxv[NI], gyv[RY];
#pragma unroll
  for (int i = 0; i < NI; ++i) gxv[i] = geo.xs[i] < g.nx ? g.gx[geo.xs[i]] : 0.0f;
#pragma unroll
  for (int j = 0; j < RY; ++j) gyv[j] = geo.yv[j] < g.ny ? g.gy[geo.yv[j]] : 0.0f;
#pragma unroll
  for (int z = 0; z < ZC; ++z) {
#pragma unroll
    for (int j = 0; j < RY; ++j)
#pragma unroll
      for (int i = 0; i < NI; ++i)
        sm[z][4 + geo.wave * RY + j][4 + T::XW * i + geo.lane] = q[j * NI + i][z + 4];
#pragma unroll
    for (int i = 0; i < T::HPT; ++i)
      if (geo.hslot[i] >= 0) (&sm[z][0][0])[geo.hslot[i]] = h[z][i];
  }
  __syncthreads();
  const float c0 = W0 * (g.cx + g.cy + g.cz);
  static_for<ZC>([&](auto Zc) {
    constexpr int Z = decltype(Zc)::value;
    const int z = geo.z0 + Z;
    if (z >= geo.z1) return;
    const auto ro = __builtin_amdgcn_make_buffer_rsrc(
        out + (int64_t)z * g.plane, (short)0, (int)(uint32_t)(g.plane * 4), 0x00020000);
    static_for<RY>([&](auto Jc) {
      constexpr int J = decltype(Jc)::value;
      static_for<NI>([&](auto Ic) {
        constexpr int I = decltype(Ic)::value;
        constexpr int P = J * NI + I;
        float sx, sy, sz;
        point_diffs<T, J, I, Z>(q, sm[Z], geo.wave, geo.lane, sx, sy, sz);
        const float c = q[P][Z + 4];
        const float lap = c0 * c + g.cx * sx + g.cy * sy + g.cz * sz;
        float acc = VD ? 2.0f * c + kv[Z][P] * (lap - mv[Z][P] * c) : 2.0f * c + kv[Z][P] * lap;
        if (z == src.z && ob[P] == src.offset) acc = __builtin_fmaf(sigma, wavelet, acc);
        const float G = gxv[I] * gyv[J] * gzv[Z];
        const float o = (!FS || z > g.zs) ? G * (acc - G * pv[Z][P]) : 0.0f;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o), ro, ob[P], 0, NT ? 2 : 0);
      });
    });
  });
}

template <class S, bool VD, bool FS, bool NT>
__device__ __forceinline__ void forward_block(const StepGrid &g, const float *__restrict__ cur,
                                              const float *prev, float *out, const Source &src,
                                              int n, const TileMap &map, int b) {
  using T = Tile<S::RY, S::NG, S::NI, S::XW>;
  __shared__ float sm[S::ZC > 0 ? S::ZC : 2][T::LY][T::LX];
  if constexpr (S::ZC > 0)
    forward_slab<T, S::ZC, VD, FS, NT>(sm, g, cur, prev, out, src, n, map, b);
  else
    forward_tile<T, VD, FS, NT>(sm, g, cur, prev, out, src, n, map, b);
}

// Blocks from map.nblocks on record row (sample n - 1).
template <class S, bool VD, bool FS, bool NT>
__global__ void __launch_bounds__(S::NTHREADS, S::WAVES)
    k_forward(StepGrid g, const float *__restrict__ cur, const float *prev, float *out,
              Source src, int n, Record rec, float *__restrict__ row, TileMap map) {
  const int b = blockIdx.x;
  if (b >= map.nblocks) return record_block(rec, cur, row, b - map.nblocks);
  forward_block<S, VD, FS, NT>(g, cur, prev, out, src, n, map, b);
}

// Several grids (one per shot) advanced by one launch: block b belongs to the
// last window whose block_begin it reaches.  Ranges follow one another without
// gaps: a window that starts off a multiple of 8 has its XCD ranges rotated, while
// ranges padded to multiples of 8 gave XCD 0 up to twice the blocks of the others
// (24 small windows, adjoint: 138 us a step instead of 78).
template <class S, bool VD, bool FS, bool NT>
__global__ void __launch_bounds__(S::NTHREADS, S::WAVES)
    k_forward_multi(const WindowStep *__restrict__ wins, int nwin, int n) {
  const int b = blockIdx.x;
  int w = 0;
  while (w + 1 < nwin && b >= wins[w + 1].block_begin) ++w;
  const WindowStep &d = wins[w];
  const int t = b - d.block_begin;
  if (t >= d.map.nblocks) {
    if (n > 0)
      record_block(d.rec, d.cur, d.seis_tm + (int64_t)(n - 1) * d.rec.nrec, t - d.map.nblocks);
    return;
  }
  forward_block<S, VD, FS, NT>(d.g, d.cur, d.prev, d.out, d.src, n, d.map, t);
}

// DL: halo delay-line depth of the adjoint's two fields (the tile shapes
// below choose it: each delay stage costs two registers per halo value).
// One adjoint step fused with the imaging condition over tile block b of a
// grid: psi^m (out, in place over psi^{m+2} = prev) from psi^{m+1} (cur), the
// residuals of sample m-1 injected at the receivers, and
// g += psi^{m+1} (L w^m - m2 w^m) (+ the illumination).  sm[0] stages psi,
// sm[1] w.
template <class T, int DL, bool VD, bool ILLUM, bool FS, bool NT>
__device__ __forceinline__ void adjoint_tile(
    const StepGrid g, const float *__restrict__ cur, const float *prev,
    float *out, const RecTable rec, const float *__restrict__ res_tm, int m,
    const float *__restrict__ wm, float *__restrict__ grad, const IllumOut il,
    const TileMap map, int b) {
  constexpr int NP = T::NP, RY = T::RY, NI = T::NI;
  __shared__ float sm[2][2][T::LY][T::LX];  // [field][buffer]
  Geo<T, 1> geo;
  if (!geo.init(g, map, b)) return;
  Marcher<T, 1, FS, DL> fa;  // adjoint state psi^{m+1}
  Marcher<T, 1, FS, DL> fw;  // forward state w^m
  fa.prime(cur, g, geo.z0, geo.off, geo.in, geo.hoff, geo.hin);
  fw.prime(wm, g, geo.z0, geo.off, geo.in, geo.hoff, geo.hin);
  float gxv[NI], gyv[RY];
#pragma unroll
  for (int i = 0; i < NI; ++i) gxv[i] = geo.xs[i] < g.nx ? g.gx[geo.xs[i]] : 0.0f;
#pragma unroll
  for (int j = 0; j < RY; ++j) gyv[j] = geo.yv[j] < g.ny ? g.gy[geo.yv[j]] : 0.0f;
  const float *res_row = res_tm + (int64_t)(m - 1) * rec.nrec;
  const float c0 = W0 * (g.cx + g.cy + g.cz);
  const int iexp = ILLUM ? il.out_exp2 - 2 * il.sc->e : 0;  // (2^e w)^2 -> 2^out_exp2 w^2
  float gzv = g.gz[geo.z0];  // the z sponge factor, read one plane ahead
  float pv[NP], kv[NP], mv[NP], gv[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    pv[p] = ld_stream_nb<NT>(prev, g, geo.z0, geo.off[p], geo.in[p]);
    kv[p] = ld_stream_nb<NT>(g.k, g, geo.z0, geo.off[p], geo.in[p]);
    mv[p] = VD ? ld_stream_nb<NT>(g.m2, g, geo.z0, geo.off[p], geo.in[p]) : 0.0f;
    gv[p] = ld_stream_nb<NT>(grad, g, geo.z0, geo.off[p], geo.in[p]);
  }
  ColCursor cc[NP];
#pragma unroll
  for (int j = 0; j < RY; ++j)
#pragma unroll
    for (int i = 0; i < NI; ++i)
      cc[j * NI + i].init(rec, res_row, geo.yv[j] * g.nx + geo.xs[i], geo.z0, geo.in[j * NI + i]);
  for (int z = geo.z0; z < geo.z1; ++z) {
    float(*sa)[T::LX] = sm[0][z & 1];
    float(*sw)[T::LX] = sm[1][z & 1];
    fa.stage(sa, geo.wave, geo.lane, geo.hslot);
    fw.stage(sw, geo.wave, geo.lane, geo.hslot);
    const float gzn = g.gz[z + 1 < g.nz ? z + 1 : z];
    fa.fetch(cur, g, z, geo.off, geo.in, geo.hoff, geo.hin);
    fw.fetch(wm, g, z, geo.off, geo.in, geo.hoff, geo.hin);
    const bool more = z + 1 < geo.z1;
    float pn[NP], kn[NP], mn[NP], gn[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      pn[p] = ld_stream_nb<NT>(prev, g, z + 1, geo.off[p], geo.in[p] && more);
      kn[p] = ld_stream_nb<NT>(g.k, g, z + 1, geo.off[p], geo.in[p] && more);
      mn[p] = VD ? ld_stream_nb<NT>(g.m2, g, z + 1, geo.off[p], geo.in[p] && more) : 0.0f;
      gn[p] = ld_stream_nb<NT>(grad, g, z + 1, geo.off[p], geo.in[p] && more);
    }
    __syncthreads();
    static_for<RY>([&](auto Jc) {
      constexpr int J = decltype(Jc)::value;
      static_for<NI>([&](auto Ic) {
        constexpr int I = decltype(Ic)::value;
        constexpr int P = J * NI + I;
        float ax, ay, az, wx, wy, wz;
        fa.template diffs<J, I>(sa, geo.wave, geo.lane, ax, ay, az);
        fw.template diffs<J, I>(sw, geo.wave, geo.lane, wx, wy, wz);
        const float ca = fa.q[P][4], cw = fw.q[P][4];
        const float lap_a = c0 * ca + g.cx * ax + g.cy * ay + g.cz * az;
        const float lap_w = c0 * cw + g.cx * wx + g.cy * wy + g.cz * wz;
        float acc = VD ? 2.0f * ca + kv[P] * (lap_a - mv[P] * ca) : 2.0f * ca + kv[P] * lap_a;
        if (cc[P].ez == z) {  // receiver residuals injected at this node
          acc += cc[P].sum;
          cc[P].advance(rec, res_row);
        }
        const float G = gxv[I] * gyv[J] * gzv;
        const bool live = !FS || z > g.zs;  // at and above a free surface psi and w stay zero
        const uint32_t ob = geo.in[P] ? 4u * geo.off[P] : kDropOffset;
        st_plane<NT>(out, g, z, ob, live ? G * (acc - G * pv[P]) : 0.0f);
        st_plane<NT>(grad, g, z, ob, live ? gv[P] + ca * (VD ? lap_w - mv[P] * cw : lap_w) : gv[P]);
        if (ILLUM && geo.in[P]) {
          const int ix = geo.xs[I] - il.border, iy = geo.yv[J] - il.border, iz = z - il.border;
          if (ix >= 0 && ix < il.mnx && iy >= 0 && iy < il.mny && iz >= 0 && iz < il.mnz)
            il.p[((int64_t)iz * il.mny + iy) * il.mnx + ix] += ldexpf(cw * cw, iexp);
        }
      });
    });
    fa.shift();
    fw.shift();
    gzv = gzn;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      pv[p] = pn[p];
      kv[p] = kn[p];
      mv[p] = mn[p];
      gv[p] = gn[p];
    }
  }
}

// The single-shot kernel keeps its own copy of the tile body: sharing the
// device function with the batched kernel cost two VGPR spills in the plane
// loop (1238 against 1220 us per step at 576^3).
template <class T, int DL, bool VD, bool ILLUM, bool FS, bool NT>
__global__ void __launch_bounds__(T::NTHREADS)
    k_adjoint(StepGrid g, const float *__restrict__ cur, const float *prev, float *out,
              RecTable rec, const float *__restrict__ res_tm, int m,
              const float *__restrict__ wm, float *__restrict__ grad, IllumOut il,
              TileMap map) {
  constexpr int NP = T::NP, RY = T::RY, NI = T::NI;
  __shared__ float sm[2][2][T::LY][T::LX];  // [field][buffer]
  Geo<T, 1> geo;
  if (!geo.init(g, map, blockIdx.x)) return;
  Marcher<T, 1, FS, DL> fa;  // adjoint state psi^{m+1}
  Marcher<T, 1, FS, DL> fw;  // forward state w^m
  fa.prime(cur, g, geo.z0, geo.off, geo.in, geo.hoff, geo.hin);
  fw.prime(wm, g, geo.z0, geo.off, geo.in, geo.hoff, geo.hin);
  float gxv[NI], gyv[RY];
#pragma unroll
  for (int i = 0; i < NI; ++i) gxv[i] = geo.xs[i] < g.nx ? g.gx[geo.xs[i]] : 0.0f;
#pragma unroll
  for (int j = 0; j < RY; ++j) gyv[j] = geo.yv[j] < g.ny ? g.gy[geo.yv[j]] : 0.0f;
  const float *res_row = res_tm + (int64_t)(m - 1) * rec.nrec;
  const float c0 = W0 * (g.cx + g.cy + g.cz);
  const int iexp = ILLUM ? il.out_exp2 - 2 * il.sc->e : 0;  // (2^e w)^2 -> 2^out_exp2 w^2
  float gzv = g.gz[geo.z0];  // the z sponge factor, read one plane ahead
  float pv[NP], kv[NP], mv[NP], gv[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    pv[p] = ld_stream_nb<NT>(prev, g, geo.z0, geo.off[p], geo.in[p]);
    kv[p] = ld_stream_nb<NT>(g.k, g, geo.z0, geo.off[p], geo.in[p]);
    mv[p] = VD ? ld_stream_nb<NT>(g.m2, g, geo.z0, geo.off[p], geo.in[p]) : 0.0f;
    gv[p] = ld_stream_nb<NT>(grad, g, geo.z0, geo.off[p], geo.in[p]);
  }
  ColCursor cc[NP];
#pragma unroll
  for (int j = 0; j < RY; ++j)
#pragma unroll
    for (int i = 0; i < NI; ++i)
      cc[j * NI + i].init(rec, res_row, geo.yv[j] * g.nx + geo.xs[i], geo.z0, geo.in[j * NI + i]);
  for (int z = geo.z0; z < geo.z1; ++z) {
    float(*sa)[T::LX] = sm[0][z & 1];
    float(*sw)[T::LX] = sm[1][z & 1];
    fa.stage(sa, geo.wave, geo.lane, geo.hslot);
    fw.stage(sw, geo.wave, geo.lane, geo.hslot);
    const float gzn = g.gz[z + 1 < g.nz ? z + 1 : z];
    fa.fetch(cur, g, z, geo.off, geo.in, geo.hoff, geo.hin);
    fw.fetch(wm, g, z, geo.off, geo.in, geo.hoff, geo.hin);
    const bool more = z + 1 < geo.z1;
    float pn[NP], kn[NP], mn[NP], gn[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      pn[p] = ld_stream_nb<NT>(prev, g, z + 1, geo.off[p], geo.in[p] && more);
      kn[p] = ld_stream_nb<NT>(g.k, g, z + 1, geo.off[p], geo.in[p] && more);
      mn[p] = VD ? ld_stream_nb<NT>(g.m2, g, z + 1, geo.off[p], geo.in[p] && more) : 0.0f;
      gn[p] = ld_stream_nb<NT>(grad, g, z + 1, geo.off[p], geo.in[p] && more);
    }
    __syncthreads();
    static_for<RY>([&](auto Jc) {
      constexpr int J = decltype(Jc)::value;
      static_for<NI>([&](auto Ic) {
        constexpr int I = decltype(Ic)::value;
        constexpr int P = J * NI + I;
        float ax, ay, az, wx, wy, wz;
        fa.template diffs<J, I>(sa, geo.wave, geo.lane, ax, ay, az);
        fw.template diffs<J, I>(sw, geo.wave, geo.lane, wx, wy, wz);
        const float ca = fa.q[P][4], cw = fw.q[P][4];
        const float lap_a = c0 * ca + g.cx * ax + g.cy * ay + g.cz * az;
        const float lap_w = c0 * cw + g.cx * wx + g.cy * wy + g.cz * wz;
        float acc = VD ? 2.0f * ca + kv[P] * (lap_a - mv[P] * ca) : 2.0f * ca + kv[P] * lap_a;
        if (cc[P].ez == z) {  // receiver residuals injected at this node
          acc += cc[P].sum;
          cc[P].advance(rec, res_row);
        }
        const float G = gxv[I] * gyv[J] * gzv;
        const bool live = !FS || z > g.zs;  // at and above a free surface psi and w stay zero
        const uint32_t ob = geo.in[P] ? 4u * geo.off[P] : kDropOffset;
        st_plane<NT>(out, g, z, ob, live ? G * (acc - G * pv[P]) : 0.0f);
        st_plane<NT>(grad, g, z, ob, live ? gv[P] + ca * (VD ? lap_w - mv[P] * cw : lap_w) : gv[P]);
        if (ILLUM && geo.in[P]) {
          const int ix = geo.xs[I] - il.border, iy = geo.yv[J] - il.border, iz = z - il.border;
          if (ix >= 0 && ix < il.mnx && iy >= 0 && iy < il.mny && iz >= 0 && iz < il.mnz)
            il.p[((int64_t)iz * il.mny + iy) * il.mnx + ix] += ldexpf(cw * cw, iexp);
        }
      });
    });
    fa.shift();
    fw.shift();
    gzv = gzn;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      pv[p] = pn[p];
      kv[p] = kn[p];
      mv[p] = mn[p];
      gv[p] = gn[p];
    }
  }
}

// Buffer k of a batched gradient's forward pool: W1, W2, then the stored
// checkpoint volumes.
__device__ __forceinline__ float *pool_buffer(const GradWindow &d, int k) {
  return k == 0 ? d.W1 : (k == 1 ? d.W2 : d.store + (int64_t)(k - 2) * d.g.plane * d.g.nz);
}

// One forward step of every window of a batched gradient: block b belongs to
// the last window whose fblock_begin it reaches; the step reads pool buffers
// cur_k (w^n) and prev_k (w^{n-1}) and writes out_k, recording the receivers when
// `record` is set.
template <class S, bool VD, bool FS, bool NT>
__global__ void __launch_bounds__(S::NTHREADS, S::WAVES)
    k_forward_pool(const GradWindow *__restrict__ wins, int nwin, int n, int cur_k, int prev_k,
                   int out_k, int record) {
  const int b = blockIdx.x;
  int w = 0;
  while (w + 1 < nwin && b >= wins[w + 1].fblock_begin) ++w;
  const GradWindow &d = wins[w];
  const int t = b - d.fblock_begin;
  const float *cur = pool_buffer(d, cur_k);
  if (t >= d.fmap.nblocks) {
    if (record && n > 0)
      record_block(d.out, cur, d.seis_tm + (int64_t)(n - 1) * d.out.nrec, t - d.fmap.nblocks);
    return;
  }
  forward_block<S, VD, FS, NT>(d.g, cur, pool_buffer(d, prev_k), pool_buffer(d, out_k), d.src, n,
                               d.fmap, t);
}

// The last sample of every window, from its final state.
__global__ void __launch_bounds__(kRecordBlock)
    k_record_windows(const WindowStep *__restrict__ wins, int n) {
  const WindowStep &d = wins[blockIdx.y];
  record_block(d.rec, d.cur, d.seis_tm + (int64_t)n * d.rec.nrec, blockIdx.x);
}
__global__ void __launch_bounds__(kRecordBlock)
    k_record_pool(const GradWindow *__restrict__ wins, int n, int cur_k) {
  const GradWindow &d = wins[blockIdx.y];
  record_block(d.out, pool_buffer(d, cur_k), d.seis_tm + (int64_t)n * d.out.nrec, blockIdx.x);
}

// One adjoint step (with imaging) of every window: psi^{m+1} is P1 (parity 0)
// or P2 (parity 1) and psi^m overwrites the other; w^m is pool buffer wm_k.
template <class T, int DL, bool VD, bool ILLUM, bool FS, bool NT>
__global__ void __launch_bounds__(T::NTHREADS)
    k_adjoint_multi(const GradWindow *__restrict__ wins, int nwin, int m, int parity, int wm_k) {
  const int b = blockIdx.x;
  int w = 0;
  while (w + 1 < nwin && b >= wins[w + 1].ablock_begin) ++w;
  const GradWindow &d = wins[w];
  float *a1 = parity ? d.P2 : d.P1, *a2 = parity ? d.P1 : d.P2;
  adjoint_tile<T, DL, VD, ILLUM, FS, NT>(d.g, a1, a2, a2, d.rec, d.res_tm, m,
                                              pool_buffer(d, wm_k), d.gimg, d.il, d.amap,
                                              b - d.ablock_begin);
}

int device_cus() {
  static const int cus = [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n <= 0)
      n = 256;
    return n;
  }();
  return cus;
}

template <class K>
int blocks_per_cu(K kernel, int threads) {
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess ||
      per_cu <= 0)
    per_cu = 4;
  return per_cu;
}

// Forward tile shapes (rows per thread, row groups, column groups per thread,
// lanes per row): 0 to 4 by tuning; the planner takes 0, 1 (with streaming hints)
// or 5, 32 x 32 x 4 points in one go (without).
template <int RY, int NG, int NI, int XW, int ZC_ = 0>
struct Shape : Tile<RY, NG, NI, XW> {
  static constexpr int ZC = ZC_;  // planes of a block that does not march, else 0
  static constexpr int WAVES = 0;  // least waves per SIMD (0: the compiler's choice)
};
template <int V>
struct FwdShape;
template <>
struct FwdShape<0> : Shape<2, 8, 1, 64> {};  // 64 x 16
template <>
struct FwdShape<1> : Shape<2, 16, 1, 64> {};  // 64 x 32
template <>
struct FwdShape<2> : Shape<2, 4, 1, 64> {};  // 64 x 8
template <>
struct FwdShape<3> : Shape<4, 4, 1, 64> {  // 64 x 16
  // 163 VGPRs instead of 174: three blocks per CU, not two, without spills (two
  // rounds at 296^3 VD: 102 us instead of 118; 448^3 with four 356 and 343)
  static constexpr int WAVES = 3;
};
template <>
struct FwdShape<4> : Shape<1, 16, 3, 64> {};  // 192 x 16
template <>
struct FwdShape<5> : Shape<2, 16, 1, 32, 4> {};  // 32 x 32 x 4

// Adjoint tile shapes, with their halo delay-line depth: 0 to 3 by tuning, 4 by
// the planner only.  With two stenciled fields, the 64 x 32 tile (one halo value
// per thread per plane, five-plane delay) stays within 128 VGPRs (4 waves per
// SIMD): 1213 us per step at 576^3 against 1432 us (64 x 8) and 1654 us
// (64 x 16, five-plane delay: 137 VGPRs, 3 waves per SIMD).  A two-plane delay
// keeps the 64 x 16 tile at 125 VGPRs: two blocks per CU.
template <int V>
struct AdjShape;
template <>
struct AdjShape<0> : Tile<2, 16, 1, 64> {  // 64 x 32
  static constexpr int DL = 5;
};
template <>
struct AdjShape<1> : Tile<2, 8, 1, 64> {  // 64 x 16
  static constexpr int DL = 2;
};
template <>
struct AdjShape<2> : Tile<2, 4, 1, 64> {  // 64 x 8
  static constexpr int DL = 5;
};
template <>
struct AdjShape<3> : Tile<2, 8, 1, 64> {  // 64 x 16, halo one plane ahead
  static constexpr int DL = 1;
};
template <>
struct AdjShape<4> : Tile<2, 16, 1, 32> {  // 32 x 32
  static constexpr int DL = 5;
};

template <class S>
using TileOf = Tile<S::RY, S::NG, S::NI, S::XW>;

template <bool B>
using Bool = std::integral_constant<bool, B>;
template <class F>
auto with_bool(bool b, F f) {
  return b ? f(Bool<true>{}) : f(Bool<false>{});
}

// Calls f(shape, variable density, free surface, streaming hints).  Only the
// shapes that the planner chooses come without the hints.
template <class F>
auto with_forward(int shape, bool vd, bool fs, bool stream, F f) {
  return with_bool(vd, [&](auto VD) {
    return with_bool(fs, [&](auto FS) {
      auto both = [&](auto S) {
        return with_bool(stream, [&](auto NT) { return f(S, VD, FS, NT); });
      };
      switch (shape) {
        case 1: return f(FwdShape<1>{}, VD, FS, Bool<true>{});
        case 2: return f(FwdShape<2>{}, VD, FS, Bool<true>{});
        case 3: return f(FwdShape<3>{}, VD, FS, Bool<true>{});
        case 4: return f(FwdShape<4>{}, VD, FS, Bool<true>{});
        case 5: return f(FwdShape<5>{}, VD, FS, Bool<false>{});
        default: return both(FwdShape<0>{});
      }
    });
  });
}
template <class F>
auto with_adjoint(int shape, bool vd, bool illum, bool fs, bool stream, F f) {
  return with_bool(vd, [&](auto VD) {
    return with_bool(illum, [&](auto IL) {
      return with_bool(fs, [&](auto FS) {
        auto both = [&](auto S) {
          return with_bool(stream, [&](auto NT) { return f(S, VD, IL, FS, NT); });
        };
        switch (shape) {
          case 1: return f(AdjShape<1>{}, VD, IL, FS, Bool<true>{});
          case 2: return f(AdjShape<2>{}, VD, IL, FS, Bool<true>{});
          case 3: return both(AdjShape<3>{});
          case 4: return both(AdjShape<4>{});
          default: return both(AdjShape<0>{});
        }
      });
    });
  });
}

// A tile shape as the planner sees it: tile, resident blocks per CU, and its time
// for a full round against shape 0's (below).
struct Candidate {
  int shape, tx, ty, per_cu;
  double weight;
  int slab;  // planes of a block that does not march, else 0
};

template <class S, class = void>
struct HasSlab : std::false_type {};
template <class S>
struct HasSlab<S, std::void_t<decltype(S::ZC)>> : std::true_type {};

template <class K, class S>
Candidate candidate(int shape, K kernel, S, double weight) {
  int slab = 0;
  if constexpr (HasSlab<S>::value) slab = S::ZC;
  return Candidate{shape, S::TX, S::TY, blocks_per_cu(kernel, S::NTHREADS), weight, slab};
}

// Weights.  Forward, with streaming hints: 64 x 32 tiles against 64 x 16, 95 / 98
// us at 296^3, 154 / 164 at 390 x 340 x 320, 330 / 341 at 448^3, 728 / 755 at
// 576^3.  Adjoint, 240 x 240 x 200: 64 x 16 tiles 91 / 87 us, 32 x 32 99 / 87 with
// hints and 75 / 72 without; those pay where a grid's last 64-wide tile is mostly
// empty.
Candidate forward_candidate(int shape, bool vd, bool fs, bool stream) {
  return with_forward(shape, vd, fs, stream, [&](auto S, auto VD, auto FS, auto NT) {
    using Sh = decltype(S);
    static const Candidate c = candidate(
        shape, k_forward<Sh, decltype(VD)::value, decltype(FS)::value, decltype(NT)::value>,
        S, shape == 1 ? 0.95 : 1.0);
    return c;
  });
}
Candidate adjoint_candidate(int shape, bool vd, bool illum, bool fs, bool stream) {
  return with_adjoint(shape, vd, illum, fs, stream, [&](auto S, auto VD, auto IL, auto FS, auto NT) {
    using Sh = decltype(S);
    static const Candidate c =
        candidate(shape,
                  k_adjoint<TileOf<Sh>, Sh::DL, decltype(VD)::value, decltype(IL)::value,
                            decltype(FS)::value, decltype(NT)::value>,
                  S, shape == 3 ? 1.04 : shape == 4 ? (NT.value ? 1.12 : 1.05) : 1.0);
    return c;
  });
}

// z chunks at least this deep (shallower ones gave nothing: 80^3 11.0 us at 4
// planes, 11.2 at 2).
constexpr int kMinZc = 4;
// At least this deep for a batch's windows whose contexts set the rounds: the
// windows fill the device together, and 4-plane chunks would only add halo (24
// windows of 49 to 80 cells, gradients over 120 steps with 2 to 8 rounds: 35.1 ms
// against 30.5).
constexpr int kBatchMinZc = 16;

// Time of a launch of `blocks` blocks that march zc planes each, in planes of a
// full device, from the rounds R = blocks / resident slots:
//   R <= 1:  one round.  A plane takes less where fewer points share a CU: 1.30
//            us with one 64 x 16 tile per CU, 1.65 with two (240 x 240 x 200 and
//            296^3, 190 to 480 blocks).
//   R > 1:   floor(R) full rounds and a last one that costs its fill, but at
//            least kTailFloor of a round (a block alone takes as long as a full
//            device's).
// Each round lasts zc planes plus kHalo for the queue's first planes and the
// 8-plane z halo.  Step times over 1 to 50 chunks at 144^3, 233 x 247 x 201,
// 240 x 240 x 200, 296^3, 390 x 340 x 320 and 576^3 keep a ratio to this within
// 10 per cent, and its best chunk count (the smallest within 2 per cent) is the
// measured best or within 2 per cent of it.  (With a floor of 0.47, fitted to 576^3 alone, 296^3 ran 1.48
// rounds of 37 planes: 125 us instead of 105 us for 0.93 of 60; the adjoint 278
// instead of 240 us.)
constexpr double kTailFloor = 0.9, kHalo = 4.0;

// A block that does not march costs its share of the device's throughput: with
// about 1.15 us a plane above, 80^3 (180 blocks) 5.9 us, 144^3 (900) 13.7, 240 x 240
// x 200 (3200) 36; the marching tiles take 7.1, 14.6 and 33.
constexpr double kSlabBase = 2.6, kSlabBlock = 0.0095;

double launch_cost(const Candidate &c, int64_t blocks, int zc) {
  const int64_t cus = device_cus();
  if (c.slab > 0) return kSlabBase + kSlabBlock * (double)blocks * 256.0 / (double)cus;
  const double R = (double)blocks / (double)(c.per_cu * cus), full = std::floor(R), f = R - full;
  double rounds;
  if (R <= 1.0) {
    const double share = (double)((blocks + cus - 1) / cus) * c.tx * c.ty / 2048.0;
    rounds = std::min(1.0, 0.58 + 0.42 * share);
  } else {
    rounds = full + (f > 0.0 ? std::max(f, kTailFloor) : 0.0);
  }
  return c.weight * rounds * (zc + kHalo);
}

int64_t tiles_of(const StepGrid &g, const Candidate &c) {
  return (int64_t)((g.nx + c.tx - 1) / c.tx) * ((g.ny + c.ty - 1) / c.ty);
}

TileMap map_of(const StepGrid &g, const Candidate &c, int nch, int min_zc) {
  TileMap m;
  m.tiles_x = (g.nx + c.tx - 1) / c.tx;
  m.tiles_y = (g.ny + c.ty - 1) / c.ty;
  nch = std::max(1, std::min(nch, (g.nz + min_zc - 1) / min_zc));
  m.zc = (g.nz + nch - 1) / nch;
  m.nchunks = (g.nz + m.zc - 1) / m.zc;
  m.nblocks = (int)((int64_t)m.tiles_x * m.tiles_y * m.nchunks);
  m.spread = 0;
  return m;
}

// Tile maps of a launch over n grids: one shape for all, chosen with the chunk
// depth by the cost above from ncand candidates; `rounds` > 0 sets each grid's
// chunk count to that many rounds of the device instead.  Returns the shape.
int plan_maps(const StepGrid *const *grids, const int *rounds, int n, const Candidate *cand,
              int ncand, TileMap *maps) {
  int deepest = 1;
  for (int i = 0; i < n; ++i) deepest = std::max(deepest, grids[i]->nz);
  const Candidate *best = &cand[0];
  int best_zc = deepest;
  double best_cost = 1e300;
  for (int k = 0; k < ncand; ++k)
    for (int nch = 1; nch <= (deepest + kMinZc - 1) / kMinZc; ++nch) {
      const int zc = (deepest + nch - 1) / nch;
      if ((deepest + zc - 1) / zc != nch) continue;  // same chunks as a smaller count
      if (cand[k].slab > 0 && zc > cand[k].slab) continue;
      int64_t blocks = 0;
      for (int i = 0; i < n; ++i) blocks += tiles_of(*grids[i], cand[k]) * ((grids[i]->nz + zc - 1) / zc);
      const double cost = launch_cost(cand[k], blocks, zc);
      if (cost < 0.98 * best_cost) {
        best_cost = cost;
        best = &cand[k];
        best_zc = zc;
      }
    }
  const int64_t slots = (int64_t)best->per_cu * device_cus();
  for (int i = 0; i < n; ++i) {
    const int64_t tiles = tiles_of(*grids[i], *best);
    const int nch = rounds[i] > 0 ? (int)((rounds[i] * slots + tiles / 2) / tiles)
                                  : (grids[i]->nz + best_zc - 1) / best_zc;
    maps[i] = map_of(*grids[i], *best, nch, rounds[i] > 0 && n > 1 ? kBatchMinZc : kMinZc);
  }
  return best->shape;
}

// Streaming hints keep single-use data out of the 256 MB last-level cache; a
// step whose volumes all fit it runs faster without them, since the next step
// finds its operands there: 144^3 VD 23.7 -> 20.5 us, 233 x 247 x 201 VD (185
// MB) 53.7 -> 46.2, 250 x 250 x 240 VD (240 MB) 61.2 -> 52.2; 270 x 260 x 250
// (281 MB) is even and 296^3 (415 MB) loses, 105 -> 118.  An adjoint step's stored
// state w^m comes from memory all the same: 24 windows (175 MB) 99 -> 92 us, 240 x
// 240 x 200 with illumination (276 MB) 85 -> 88.
constexpr double kCachedBytes = 256e6;
// Forward steps over more than this run their blocks in tile order (tile_of).
constexpr double kSpreadBytes = 1e9;

bool step_streams(const StepGrid *const *grids, int n, int volumes) {
  double bytes = 0.0;
  for (int i = 0; i < n; ++i)
    bytes += 4.0 * volumes * (double)grids[i]->nx * grids[i]->ny * grids[i]->nz;
  return bytes > kCachedBytes;
}

}  // namespace

StepPlan plan_forward(const StepGrid *const *grids, const Tuning *const *tu, int n,
                      bool out_of_place, TileMap *maps) {
  bool vd = false, fs = false, tuned = false;
  std::vector<int> rounds(n);
  for (int i = 0; i < n; ++i) {
    vd = vd || grids[i]->m2;
    fs = fs || grids[i]->zs != kNoSurface;
    rounds[i] = tu[i]->rounds;
    tuned = tuned || rounds[i] > 0;
  }
  StepPlan p;
  p.stream = step_streams(grids, n, 3 + (vd ? 1 : 0) + (out_of_place ? 1 : 0));
  Candidate c[2] = {forward_candidate(tu[0]->variant, vd, fs, p.stream), {}};
  int nc = 1;
  if (tu[0]->variant == 0 && !tuned) c[nc++] = forward_candidate(p.stream ? 1 : 5, vd, fs, p.stream);
  p.shape = plan_maps(grids, rounds.data(), n, c, nc, maps);
  const double bytes = 4.0 * (vd ? 4 : 3) * (double)grids[0]->nx * grids[0]->ny * grids[0]->nz;
  if (n == 1 && bytes > kSpreadBytes) maps[0].spread = 1;
  return p;
}

StepPlan plan_adjoint(const StepGrid *const *grids, const Tuning *const *tu, int n, bool illum,
                      TileMap *maps) {
  bool vd = false, fs = false, tuned = false;
  std::vector<int> rounds(n);
  for (int i = 0; i < n; ++i) {
    vd = vd || grids[i]->m2;
    fs = fs || grids[i]->zs != kNoSurface;
    rounds[i] = tu[i]->adj_rounds;
    tuned = tuned || rounds[i] > 0;
  }
  StepPlan p;
  // psi^{m+1}, psi^m, w^m, g, k (m2, illumination)
  p.stream = step_streams(grids, n, 5 + (vd ? 1 : 0) + (illum ? 1 : 0));
  Candidate c[3] = {adjoint_candidate(tu[0]->adj_variant, vd, illum, fs, p.stream), {}, {}};
  int nc = 1;
  if (tu[0]->adj_variant == 0 && !tuned) {
    c[nc++] = adjoint_candidate(3, vd, illum, fs, p.stream);
    c[nc++] = adjoint_candidate(4, vd, illum, fs, p.stream);
  }
  p.shape = plan_maps(grids, rounds.data(), n, c, nc, maps);
  return p;
}

hipError_t launch_forward_step(const StepPlan &plan, const TileMap &map, const StepGrid &g,
                               const float *cur, const float *prev, float *out, const Source &src,
                               int n, const Record &rec, float *row, hipStream_t stream) {
  return with_forward(plan.shape, g.m2 != nullptr, g.zs != kNoSurface, plan.stream,
                      [&](auto S, auto VD, auto FS, auto NT) {
    using Sh = decltype(S);
    hipLaunchKernelGGL((k_forward<Sh, decltype(VD)::value, decltype(FS)::value,
                                  decltype(NT)::value>),
                       dim3(map.nblocks + (row ? record_blocks(rec.nrec) : 0)),
                       dim3(Sh::NTHREADS), 0, stream, g, cur, prev, out, src, n, rec, row, map);
    return hipGetLastError();
  });
}

int window_blocks(const TileMap &map, int nrec) { return map.nblocks + record_blocks(nrec); }

hipError_t launch_record_windows(const WindowStep *wins, int nwin, int nrec_max, int n,
                                 hipStream_t stream) {
  if (nrec_max <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_record_windows, dim3(record_blocks(nrec_max), nwin), dim3(kRecordBlock), 0,
                     stream, wins, n);
  return hipGetLastError();
}

hipError_t launch_record_pool(const GradWindow *wins, int nwin, int nrec_max, int n, int cur_k,
                              hipStream_t stream) {
  if (nrec_max <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_record_pool, dim3(record_blocks(nrec_max), nwin), dim3(kRecordBlock), 0,
                     stream, wins, n, cur_k);
  return hipGetLastError();
}

hipError_t launch_forward_multi(const StepPlan &plan, const WindowStep *wins, int nwin,
                                int nblocks, int n, bool vd, bool fs, hipStream_t stream) {
  return with_forward(plan.shape, vd, fs, plan.stream, [&](auto S, auto VD, auto FS, auto NT) {
    using Sh = decltype(S);
    hipLaunchKernelGGL((k_forward_multi<Sh, decltype(VD)::value, decltype(FS)::value,
                                        decltype(NT)::value>),
                       dim3(nblocks), dim3(Sh::NTHREADS), 0, stream, wins, nwin, n);
    return hipGetLastError();
  });
}

hipError_t launch_forward_pool(const StepPlan &plan, const GradWindow *wins, int nwin, int nblocks,
                               int n, int cur_k, int prev_k, int out_k, int record, bool vd,
                               bool fs, hipStream_t stream) {
  return with_forward(plan.shape, vd, fs, plan.stream, [&](auto S, auto VD, auto FS, auto NT) {
    using Sh = decltype(S);
    hipLaunchKernelGGL((k_forward_pool<Sh, decltype(VD)::value, decltype(FS)::value,
                                       decltype(NT)::value>),
                       dim3(nblocks), dim3(Sh::NTHREADS), 0, stream, wins, nwin, n, cur_k, prev_k,
                       out_k, record);
    return hipGetLastError();
  });
}

hipError_t launch_adjoint_step(const StepPlan &plan, const TileMap &map, const StepGrid &g,
                               const float *cur, const float *prev, float *out,
                               const RecTable &rec, const float *res_tm, int m, const float *wm,
                               float *grad, const IllumOut &illum, hipStream_t stream) {
  return with_adjoint(plan.shape, g.m2 != nullptr, illum.p != nullptr, g.zs != kNoSurface,
                      plan.stream, [&](auto S, auto VD, auto IL, auto FS, auto NT) {
    using Sh = decltype(S);
    hipLaunchKernelGGL((k_adjoint<TileOf<Sh>, Sh::DL, decltype(VD)::value, decltype(IL)::value,
                                  decltype(FS)::value, decltype(NT)::value>),
                       dim3(map.nblocks), dim3(Sh::NTHREADS), 0, stream, g, cur, prev, out, rec,
                       res_tm, m, wm, grad, illum, map);
    return hipGetLastError();
  });
}

hipError_t launch_adjoint_multi(const StepPlan &plan, const GradWindow *wins, int nwin,
                                int nblocks, int m, int parity, int wm_k, bool vd, bool illum,
                                bool fs, hipStream_t stream) {
  return with_adjoint(plan.shape, vd, illum, fs, plan.stream,
                      [&](auto S, auto VD, auto IL, auto FS, auto NT) {
    using Sh = decltype(S);
    hipLaunchKernelGGL((k_adjoint_multi<TileOf<Sh>, Sh::DL, decltype(VD)::value,
                                        decltype(IL)::value, decltype(FS)::value,
                                        decltype(NT)::value>),
                       dim3(nblocks), dim3(Sh::NTHREADS), 0, stream, wins, nwin, m, parity, wm_k);
    return hipGetLastError();
  });
}

}  // namespace wfd
