// CPML absorbing layer (§2.1: the convolutional PML of Roden and Gedney, the
// paper's alternative to damping), on the second-order equation.
//
// In the layer each second derivative is taken in stretched coordinates,
// d2/dx~2 w = D2 w + D1 psi + zeta, with the recursive convolutions
//   psi_d  = b_d psi_d  + a_d D1_d w
//   zeta_d = b_d zeta_d + a_d (D2_d w + D1_d psi_d)
// so the leapfrog step gains k C with C = sum_d (D1_d psi_d + zeta_d).  The
// step kernels do everything else (with unit sponge tables); these kernels
// add the layer's terms on the shell, the points within reach of them.  The
// adjoint is the exact transpose:
//   nu_d = phi^{m+1} + b_d nu_d,   mu_d = b_d mu_d - D1_d (a_d nu_d + phi^{m+1}),
//   phi^m += k sum_d [D2_d (a_d nu_d) - D1_d (a_d mu_d)],
// and the imaging condition gains phi^{m+1} C^m.
//
// D1 is the eighth-order central first difference (4/5, -1/5, 4/105, -1/280)
// and D2 the second difference of L; cells outside the padded grid are zero,
// and D2 along z reads the free surface's negated image like L does.
//
// Everything an axis adds depends on that axis' lines alone, so one kernel per
// axis and direction does all of it: a block takes a tile of lines over one
// end's segment (the layer and the 4 cells beyond), loads each array once,
// keeps w and psi (a nu + phi1, a nu, then a mu) in LDS between the two
// recursions and writes psi, zeta and the correction: 36 B per point forward,
// 44 B adjoint with imaging, every load issued before the first barrier.  The
// axes' kernels follow one another (x, y, z) because their corrections add up
// where the layers cross.  240 x 240 x 200 with a 20-cell layer (7.4 M line
// points): 73 us a forward step and 81 us an adjoint step, 3.7-4.1 TB/s, where
// kernels that walked the shell's points and read every neighbour line through
// the caches took 141 and 363 us.  What is left is the start and end of three
// short launches and the x kernels' partial cache lines.
//
// A memory variable of axis d is nonzero only on that axis' layer, the B
// border cells at each end of the padded axis, and is stored as two slabs of
// W = B + 8 cells, [0, W) and [N - W, N) (the whole axis when they would
// meet): x as [Nz][Ny][2W], y as [Nz][2W][Nx], z as [2W][Ny][Nx].  A point
// within reach of the layer (4 cells) reads the variable at most 4 cells
// further, so every read lands in the point's own slab and a line of the
// variable is addressed like a line of a full volume.  Psi and zeta (or mu
// and nu) of an axis take 4 W / N of a volume rather than two volumes, and
// every checkpoint of the gradient's forward sweep holds a set of six.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "wfd_internal.h"

namespace wfd {
namespace {

__device__ __forceinline__ float d1c(int j) {
  return j == 1 ? 0.8f : j == 2 ? -0.2f : j == 3 ? (float)(4.0 / 105.0) : (float)(-1.0 / 280.0);
}
__device__ __forceinline__ float d2c(int j) {
  return j == 0   ? (float)(-205.0 / 72.0)
         : j == 1 ? 1.6f
         : j == 2 ? -0.2f
         : j == 3 ? (float)(8.0 / 315.0)
                  : (float)(-1.0 / 560.0);
}

// Stored index of cell i on an axis of n cells with slab width `half` and
// stored length `len` (above).
__device__ __forceinline__ int cidx(int i, int half, int len, int n) {
  return i < half ? i : i - (n - len);
}

// A shell point's index in the correction store's layout is the x = 0 index of
// its row plus x; x matters for the choice of the box between the x layers.
__device__ __forceinline__ int64_t shell_row(const Shell &sh, int b, int y, int z) {
  return sh.start[b] + ((int64_t)(z - sh.z0[b]) * sh.ny[b] + (y - sh.y0[b])) * sh.nx[b] -
         sh.x0[b];
}
// Box of the points of a row within reach of a y or z layer.
__device__ __forceinline__ int row_box(const Shell &sh, int y, int z) {
  return z < sh.lo[2] ? sh.id[0] : z > sh.hi[2] ? sh.id[1] : y < sh.lo[1] ? sh.id[2] : sh.id[3];
}
__device__ __forceinline__ bool near(const Shell &sh, int d, int i) {
  return i < sh.lo[d] || i > sh.hi[d];
}

// What one axis' kernel needs besides the grid.
struct AxisJob {
  const float *a, *b;  // recursion coefficients per index
  float ih, c2;        // 1 / h, 1 / h^2
  int n, half, len;    // axis length, slab width and stored length
  int L, s0[2];        // segment length, first cell of each end's segment
  int nseg;            // segments (1: the whole axis, or the far end only)
  int rows;            // x kernels: rows of a plane per block
  int tiles;           // tiles of a plane's y range (x kernels) or x range
  uint32_t first;      // first block of this launch
};

// b u + a t.  The rounding of every forward sum is written out (which product
// is rounded, which is fused), so that traces keep their bits whatever the
// kernel's shape.
template <int AXIS>
__device__ __forceinline__ float recursion(float b, float u, float a, float t) {
  return AXIS < 2 ? __builtin_fmaf(b, u, a * t) : __builtin_fmaf(t, a, b * u);
}

// First and second difference around v[0], neighbours `st` apart.
__device__ __forceinline__ float first_diff(const float *v, int st) {
  float s = 0.0f;
#pragma unroll
  for (int j = 1; j <= 4; ++j) s += d1c(j) * (v[j * st] - v[-j * st]);
  return s;
}
__device__ __forceinline__ float second_diff(const float *v, int st) {
  float s = d2c(0) * v[0];
#pragma unroll
  for (int j = 1; j <= 4; ++j) s += d2c(j) * (v[j * st] + v[-j * st]);
  return s;
}
// The second difference at cell i of an axis that a tile holds whole, with a
// free surface at zs: cells before it are the negated image.
__device__ __forceinline__ float second_diff_image(const float *v, int st, int i, int n, int zs) {
  auto cell = [&](int o) {
    if (i + o >= zs) return v[o * st];
    const int m = 2 * zs - (i + o);
    return m < n ? -v[(m - i) * st] : 0.0f;
  };
  float s = d2c(0) * cell(0);
#pragma unroll
  for (int j = 1; j <= 4; ++j) s += d2c(j) * (cell(j) + cell(-j));
  return s;
}

// ---- y and z: T neighbouring x of a plane (y: of z, z: of y), one segment ----
// Thread group g of the block's NT / T takes cells g R .. g R + R - 1 of the
// segment, kept in registers; the four cells on either side come through LDS,
// whose row 4 + c is cell c (zero past the segment's ends).  T = 64: a group is
// a wavefront, so cells, coefficients and row addresses are scalars.
template <int AXIS, int NT, int T, int R>
struct PlaneTile {
  static constexpr int G = NT / T, ROWS = G * R + 8;
  int lane, first, s0, x, other;
  bool ok;
  int64_t fb, fs, mb, ms;  // field and memory element of cell 0, step per cell
  __device__ __forceinline__ PlaneTile(const StepGrid &g, const AxisJob &j) {
    int b = blockIdx.x + j.first;
    s0 = j.s0[b % j.nseg];
    b /= j.nseg;
    other = b / j.tiles;
    lane = threadIdx.x % T;
    const int grp = threadIdx.x / T;
    first = (T == 64 ? __builtin_amdgcn_readfirstlane(grp) : grp) * R;
    x = (b - other * j.tiles) * T + lane;
    ok = x < g.nx;
    fb = AXIS == 1 ? (int64_t)other * g.plane : (int64_t)other * g.pitch;
    fs = AXIS == 1 ? (int64_t)g.pitch : g.plane;
    mb = AXIS == 1 ? (int64_t)other * j.len * g.nx : (int64_t)other * g.nx;
    ms = AXIS == 1 ? (int64_t)g.nx : (int64_t)g.ny * g.nx;
  }
  __device__ __forceinline__ int64_t field(int i) const { return fb + i * fs; }
  __device__ __forceinline__ int64_t mem(const AxisJob &j, int i) const {
    return mb + cidx(i, j.half, j.len, j.n) * ms;
  }
  __device__ __forceinline__ int y(int i) const { return AXIS == 1 ? i : other; }
  __device__ __forceinline__ int z(int i) const { return AXIS == 1 ? other : i; }
  __device__ __forceinline__ float *slot(float *s, int c) const {
    return s + (first + c + 4) * T + lane;
  }
  // the group's cells with four on either side: v[4 + c] is cell first + c
  __device__ __forceinline__ void with_neighbours(float *s, const float *own, float *v) const {
#pragma unroll
    for (int c = 0; c < R + 8; ++c)
      v[c] = c >= 4 && c < 4 + R ? own[c >= 4 && c < 4 + R ? c - 4 : 0] : *slot(s, c - 4);
  }
  __device__ __forceinline__ void zero_ends(float *s) const {
    for (int e = threadIdx.x; e < 8 * T; e += NT)
      s[e < 4 * T ? e : e + (ROWS - 8) * T] = 0.0f;
  }
};

// The memory variables of an axis whose kernel has run, for the points where its
// layer crosses the present one.
struct Crossed {
  const float *psi, *zeta;
  float ih;
  int n, half, len;
  // c plus the axis' terms at its cell i, as its kernel summed them (the same
  // roundings; zeta is zero off the layer); base: element of cell 0 of the
  // point's line, st per cell.  A cell past an end reads the last one, unused.
  __device__ __forceinline__ float add(float c, int64_t base, int st, int i) const {
    const int64_t e = base + (int64_t)cidx(i, half, len, n) * st;
    const float z = zeta[e];
    float up[4], dn[4], s = 0.0f;
#pragma unroll
    for (int j = 1; j <= 4; ++j) {
      up[j - 1] = psi[e + min(j, n - 1 - i) * st];
      dn[j - 1] = psi[e - min(j, i) * st];
    }
#pragma unroll
    for (int j = 1; j <= 4; ++j)
      s = __builtin_fmaf(d1c(j), (i + j < n ? up[j - 1] : 0.0f) - (i >= j ? dn[j - 1] : 0.0f), s);
    return __builtin_fmaf(ih, s, c) + z;
  }
};

// Where layers cross, the last of their axes adds k C to out.  The earlier axes'
// terms come from cstore, which then holds C at every point of the shell (STORE:
// the gradient), or are formed again from their memory variables (cx, cy; the
// same bits), so that a forward sweep's workspace holds no C: 24 MB less at 240 x
// 240 x 200 with a 20-cell layer, 97 us a step instead of 93, and 252 MB at 576^3
// with 32 cells, 1167 instead of 1181.
template <int AXIS, int NT, int T, int R, bool IMG, bool STORE>
__global__ void __launch_bounds__(NT)
    k_cpml_forward(StepGrid g, AxisJob j, Shell sh, const float *__restrict__ w,
                   float *__restrict__ psi, float *__restrict__ zeta, float *__restrict__ out,
                   float *__restrict__ cstore, Crossed cx, Crossed cy) {
  const PlaneTile<AXIS, NT, T, R> t(g, j);
  __shared__ float sw[t.ROWS * T], sp[t.ROWS * T];
  t.zero_ends(sw);
  t.zero_ends(sp);
  const bool near_x = near(sh, 0, t.x);
  float wv[R], ps[R], ze[R], ov[R], kv[R], cv[R];
#pragma unroll
  for (int c = 0; c < R; ++c) {
    wv[c] = ps[c] = ze[c] = ov[c] = kv[c] = cv[c] = 0.0f;
    if (t.first + c >= j.L || !t.ok) continue;
    const int i = t.s0 + t.first + c;
    wv[c] = w[t.field(i) + t.x];
    if (j.a[i] != 0.0f) {
      ps[c] = psi[t.mem(j, i) + t.x];
      ze[c] = zeta[t.mem(j, i) + t.x];
    }
    if (!near(sh, AXIS, i)) continue;
    if (out && (AXIS == 2 || !near(sh, 2, t.z(i)))) {
      ov[c] = out[t.field(i) + t.x];
      kv[c] = g.k[t.field(i) + t.x];
    }
    const bool near_y = AXIS == 2 && near(sh, 1, t.y(i));
    if constexpr (STORE) {
      if (near_x || near_y)
        cv[c] = cstore[shell_row(sh, row_box(sh, t.y(i), t.z(i)), t.y(i), t.z(i)) + t.x];
    } else if (AXIS == 2 || !near(sh, 2, t.z(i))) {
      if (near_x) cv[c] = cx.add(cv[c], ((int64_t)t.z(i) * g.ny + t.y(i)) * cx.len, 1, t.x);
      if (near_y) cv[c] = cy.add(cv[c], (int64_t)t.z(i) * cy.len * g.nx + t.x, g.nx, t.y(i));
    }
  }
#pragma unroll
  for (int c = 0; c < R; ++c) *t.slot(sw, c) = wv[c];
  __syncthreads();
  float v[R + 8];
  t.with_neighbours(sw, wv, v);
#pragma unroll
  for (int c = 0; c < R; ++c) {
    const int i = t.s0 + t.first + c;
    float d2 = 0.0f;
    if (t.first + c < j.L && t.ok && j.a[i] != 0.0f) {
      ps[c] = recursion<AXIS>(j.b[i], ps[c], j.a[i], j.ih * first_diff(v + c + 4, 1));
      psi[t.mem(j, i) + t.x] = ps[c];
      d2 = IMG ? second_diff_image(t.slot(sw, c), T, i, j.n, g.zs) : second_diff(v + c + 4, 1);
    }
    *t.slot(sp, c) = ps[c];
    wv[c] = d2;
  }
  __syncthreads();
  t.with_neighbours(sp, ps, v);
#pragma unroll
  for (int c = 0; c < R; ++c) {
    const int i = t.s0 + t.first + c;
    if (t.first + c >= j.L || !t.ok || !near(sh, AXIS, i)) continue;
    const float d1 = first_diff(v + c + 4, 1), d1p = j.ih * d1;
    float cc = __builtin_fmaf(j.ih, d1, cv[c]);
    if (j.a[i] != 0.0f) {
      const float z = recursion<AXIS>(j.b[i], ze[c], j.a[i], __builtin_fmaf(j.c2, wv[c], d1p));
      zeta[t.mem(j, i) + t.x] = z;
      cc += z;
    }
    const bool more = AXIS == 1 && near(sh, 2, t.z(i));
    if (out && !more && t.z(i) > g.zs)
      out[t.field(i) + t.x] = __builtin_fmaf(cc, kv[c], ov[c]);
    if constexpr (STORE)
      cstore[shell_row(sh, row_box(sh, t.y(i), t.z(i)), t.y(i), t.z(i)) + t.x] = cc;
  }
}

template <int AXIS, int NT, int T, int R, bool IMG>
__global__ void __launch_bounds__(NT)
    k_cpml_adjoint(StepGrid g, AxisJob j, Shell sh, const float *__restrict__ phi1,
                   float *__restrict__ nu, float *__restrict__ mu, float *__restrict__ phi,
                   const float *__restrict__ cstore, float *__restrict__ grad) {
  const PlaneTile<AXIS, NT, T, R> t(g, j);
  __shared__ float sf[t.ROWS * T], sn[t.ROWS * T];
  t.zero_ends(sf);
  t.zero_ends(sn);
  float fv[R], an[R], mv[R], pv[R], kv[R];
#pragma unroll
  for (int c = 0; c < R; ++c) {
    fv[c] = an[c] = mv[c] = pv[c] = kv[c] = 0.0f;
    if (t.first + c >= j.L || !t.ok) continue;
    const int i = t.s0 + t.first + c;
    fv[c] = phi1[t.field(i) + t.x];
    if (j.a[i] != 0.0f) {
      an[c] = nu[t.mem(j, i) + t.x];
      mv[c] = mu[t.mem(j, i) + t.x];
    }
    if (!near(sh, AXIS, i)) continue;
    pv[c] = phi[t.field(i) + t.x];
    kv[c] = g.k[t.field(i) + t.x];
    // imaging once per point: by the last axis whose layer it is near
    if (cstore && (AXIS == 2 || !near(sh, 2, t.z(i))))
      grad[t.field(i) + t.x] +=
          fv[c] * cstore[shell_row(sh, row_box(sh, t.y(i), t.z(i)), t.y(i), t.z(i)) + t.x];
  }
#pragma unroll
  for (int c = 0; c < R; ++c) {
    const int i = t.s0 + t.first + c;
    if (t.first + c < j.L && t.ok && j.a[i] != 0.0f) {
      const float v = fv[c] + j.b[i] * an[c];
      nu[t.mem(j, i) + t.x] = v;
      an[c] = j.a[i] * v;
    }
    fv[c] += an[c];
    *t.slot(sn, c) = an[c];
    *t.slot(sf, c) = fv[c];
  }
  __syncthreads();
  float v[R + 8];
  t.with_neighbours(sf, fv, v);
#pragma unroll
  for (int c = 0; c < R; ++c) {
    const int i = t.s0 + t.first + c;
    if (t.first + c < j.L && t.ok && j.a[i] != 0.0f) {
      const float m = j.b[i] * mv[c] - first_diff(v + c + 4, 1) * j.ih;
      mu[t.mem(j, i) + t.x] = m;
      mv[c] = j.a[i] * m;
    }
  }
  t.with_neighbours(sn, an, v);
#pragma unroll
  for (int c = 0; c < R; ++c) {
    const int i = t.s0 + t.first + c;
    fv[c] = j.c2 * (IMG ? second_diff_image(t.slot(sn, c), T, i, j.n, g.zs)
                        : second_diff(v + c + 4, 1));
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < R; ++c) *t.slot(sf, c) = mv[c];  // a mu, zero off the layer
  __syncthreads();
  t.with_neighbours(sf, mv, v);
#pragma unroll
  for (int c = 0; c < R; ++c) {
    const int i = t.s0 + t.first + c;
    if (t.first + c >= j.L || !t.ok || !near(sh, AXIS, i) || t.z(i) <= g.zs) continue;
    phi[t.field(i) + t.x] = pv[c] + kv[c] * (fv[c] - first_diff(v + c + 4, 1) * j.ih);
  }
}

// ---- y and z: segments too long for a tile (plane_shape) ----------------------
// A thread marches kLongCells cells of a line with the nine values around the
// present one in registers; a block is 64 lines in each of four planes.  Between
// the recursions the arrays go through memory: each kernel writes only what no
// other thread of it reads.
constexpr int kLongCells = 16;

template <int AXIS>
struct LongLine {
  int i0, i1;  // cells of this thread
  int x, other;
  bool ok;
  int64_t fb, fs, mb, ms;  // field and memory element of cell 0, step per cell
  __device__ __forceinline__ LongLine(const StepGrid &g, const AxisJob &j) {
    int b = blockIdx.x + j.first;
    const int chunks = (j.L + kLongCells - 1) / kLongCells;
    x = b % j.tiles * 64 + threadIdx.x % 64;
    b /= j.tiles;
    const int s0 = j.s0[b / chunks % j.nseg];
    i0 = s0 + b % chunks * kLongCells;
    i1 = min(i0 + kLongCells, s0 + j.L);
    other = b / (chunks * j.nseg) * 4 + threadIdx.x / 64;
    ok = x < g.nx && other < (AXIS == 1 ? g.nz : g.ny);
    fb = (AXIS == 1 ? (int64_t)other * g.plane : (int64_t)other * g.pitch) + x;
    fs = AXIS == 1 ? (int64_t)g.pitch : g.plane;
    mb = (AXIS == 1 ? (int64_t)other * j.len * g.nx : (int64_t)other * g.nx) + x;
    ms = AXIS == 1 ? (int64_t)g.nx : (int64_t)g.ny * g.nx;
  }
  __device__ __forceinline__ int64_t field(int i) const { return fb + i * fs; }
  __device__ __forceinline__ int64_t mem(const AxisJob &j, int i) const {
    return mb + cidx(i, j.half, j.len, j.n) * ms;
  }
  __device__ __forceinline__ int y(int i) const { return AXIS == 1 ? i : other; }
  __device__ __forceinline__ int z(int i) const { return AXIS == 1 ? other : i; }
  // Cell i of a field or a memory variable u: zero outside the grid (and where the
  // variable is not stored: cells that no point of the layer's reach uses), with
  // `image` the negated mirror before a free surface.
  __device__ __forceinline__ float cell(const float *u, const StepGrid &g, const AxisJob &j, int i,
                                        bool image = false) const {
    if (image && AXIS == 2 && i < g.zs) {
      const int m = 2 * g.zs - i;
      return m < j.n ? -u[field(m)] : 0.0f;
    }
    return i >= 0 && i < j.n ? u[field(i)] : 0.0f;
  }
  __device__ __forceinline__ bool stored(const AxisJob &j, int i) const {
    return i >= 0 && i < j.n && (i < j.half || i >= j.n - (j.len - j.half));
  }
};

// f(cell) of cells i - 4 .. i + 4: v[4] is cell i.
struct Window {
  float v[9];
  template <class F>
  __device__ __forceinline__ void prime(F f, int i) {
#pragma unroll
    for (int c = 0; c < 9; ++c) v[c] = f(i - 4 + c);
  }
  template <class F>
  __device__ __forceinline__ void advance(F f, int i) {  // to cell i + 1
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = v[c + 1];
    v[8] = f(i + 5);
  }
};

template <int AXIS>
__global__ void __launch_bounds__(256)
    k_cpml_psi_long(StepGrid g, AxisJob j, const float *__restrict__ w, float *__restrict__ psi) {
  const LongLine<AXIS> t(g, j);
  if (!t.ok) return;
  auto fw = [&](int i) { return t.cell(w, g, j, i); };
  Window q;
  q.prime(fw, t.i0);
  for (int i = t.i0; i < t.i1; ++i) {
    if (j.a[i] != 0.0f) {
      float &u = psi[t.mem(j, i)];
      u = recursion<AXIS>(j.b[i], u, j.a[i], j.ih * first_diff(q.v + 4, 1));
    }
    q.advance(fw, i);
  }
}

// As the last part of k_cpml_forward.
template <int AXIS>
__global__ void __launch_bounds__(256)
    k_cpml_zeta_long(StepGrid g, AxisJob j, Shell sh, const float *__restrict__ w,
                     const float *__restrict__ psi, float *__restrict__ zeta,
                     float *__restrict__ out, float *__restrict__ cstore, Crossed cx, Crossed cy) {
  const LongLine<AXIS> t(g, j);
  if (!t.ok) return;
  auto fw = [&](int i) { return t.cell(w, g, j, i, true); };
  auto fp = [&](int i) { return t.stored(j, i) ? psi[t.mem(j, i)] : 0.0f; };
  const bool near_x = near(sh, 0, t.x);
  Window qw, qp;
  qw.prime(fw, t.i0);
  qp.prime(fp, t.i0);
  for (int i = t.i0; i < t.i1; ++i) {
    if (near(sh, AXIS, i)) {
      const int y = t.y(i), z = t.z(i);
      const bool near_y = AXIS == 2 && near(sh, 1, y), more = AXIS == 1 && near(sh, 2, z);
      const int64_t q = shell_row(sh, row_box(sh, y, z), y, z) + t.x;
      float c = 0.0f;
      if (cstore) {
        if (near_x || near_y) c = cstore[q];
      } else if (!more) {
        if (near_x) c = cx.add(c, ((int64_t)z * g.ny + y) * cx.len, 1, t.x);
        if (near_y) c = cy.add(c, (int64_t)z * cy.len * g.nx + t.x, g.nx, y);
      }
      const float d1 = first_diff(qp.v + 4, 1), d1p = j.ih * d1;
      c = __builtin_fmaf(j.ih, d1, c);
      if (j.a[i] != 0.0f) {
        float &u = zeta[t.mem(j, i)];
        u = recursion<AXIS>(j.b[i], u, j.a[i], __builtin_fmaf(j.c2, second_diff(qw.v + 4, 1), d1p));
        c += u;
      }
      if (out && !more && z > g.zs)
        out[t.field(i)] = __builtin_fmaf(c, g.k[t.field(i)], out[t.field(i)]);
      if (cstore) cstore[q] = c;
    }
    qw.advance(fw, i);
    qp.advance(fp, i);
  }
}

// nu = phi1 + b nu, and the imaging term (k_cpml_adjoint).
template <int AXIS>
__global__ void __launch_bounds__(256)
    k_cpml_nu_long(StepGrid g, AxisJob j, Shell sh, const float *__restrict__ phi1,
                   float *__restrict__ nu, const float *__restrict__ cstore,
                   float *__restrict__ grad) {
  const LongLine<AXIS> t(g, j);
  if (!t.ok) return;
  for (int i = t.i0; i < t.i1; ++i) {
    const float f = phi1[t.field(i)];
    const int y = t.y(i), z = t.z(i);
    if (j.a[i] != 0.0f) {
      float &u = nu[t.mem(j, i)];
      u = f + j.b[i] * u;
    }
    if (cstore && near(sh, AXIS, i) && (AXIS == 2 || !near(sh, 2, z)))
      grad[t.field(i)] += f * cstore[shell_row(sh, row_box(sh, y, z), y, z) + t.x];
  }
}

template <int AXIS>
__global__ void __launch_bounds__(256)
    k_cpml_mu_long(StepGrid g, AxisJob j, const float *__restrict__ phi1,
                   const float *__restrict__ nu, float *__restrict__ mu) {
  const LongLine<AXIS> t(g, j);
  if (!t.ok) return;
  auto f = [&](int i) {
    const float an = t.stored(j, i) ? j.a[i] * nu[t.mem(j, i)] : 0.0f;
    return t.cell(phi1, g, j, i) + an;
  };
  Window q;
  q.prime(f, t.i0);
  for (int i = t.i0; i < t.i1; ++i) {
    if (j.a[i] != 0.0f) {
      float &u = mu[t.mem(j, i)];
      u = j.b[i] * u - first_diff(q.v + 4, 1) * j.ih;
    }
    q.advance(f, i);
  }
}

template <int AXIS>
__global__ void __launch_bounds__(256)
    k_cpml_phi_long(StepGrid g, AxisJob j, Shell sh, const float *__restrict__ nu,
                    const float *__restrict__ mu, float *__restrict__ phi) {
  const LongLine<AXIS> t(g, j);
  if (!t.ok) return;
  auto weighted = [&](const float *u, int i) {
    return t.stored(j, i) ? j.a[i] * u[t.mem(j, i)] : 0.0f;
  };
  auto fn = [&](int i) {  // before a free surface the negated image
    if (AXIS == 2 && i < g.zs) return -weighted(nu, 2 * g.zs - i);
    return weighted(nu, i);
  };
  auto fm = [&](int i) { return weighted(mu, i); };
  Window qn, qm;
  qn.prime(fn, t.i0);
  qm.prime(fm, t.i0);
  for (int i = t.i0; i < t.i1; ++i) {
    if (near(sh, AXIS, i) && t.z(i) > g.zs)
      phi[t.field(i)] +=
          g.k[t.field(i)] * (j.c2 * second_diff(qn.v + 4, 1) - first_diff(qm.v + 4, 1) * j.ih);
    qn.advance(fn, i);
    qm.advance(fm, i);
  }
}

// ---- x: rows of a plane, both segments, consecutive elements along x ---------
// Element e = thread + NT k of the block's rows x segments x cells.
template <int NT, int N>
struct RowTile {
  int y0, z, pitch;   // first row, plane, LDS pitch of a line
  int P, total;       // positions per row, elements of the block
  int64_t fb, mb;     // field and memory element of the first row
  int line[N], pos[N];
  __device__ __forceinline__ RowTile(const StepGrid &g, const AxisJob &j) {
    const uint32_t b = blockIdx.x + j.first;
    z = b / j.tiles;
    y0 = (b - z * j.tiles) * j.rows;
    pitch = j.L + 8;
    P = j.nseg * j.L;
    total = min(j.rows, g.ny - y0) * P;
    fb = (int64_t)z * g.plane + (int64_t)y0 * g.pitch;
    mb = ((int64_t)z * g.ny + y0) * j.len;
    const int dl = NT / P, dp = NT - dl * P;
    int l = threadIdx.x / P, p = threadIdx.x - l * P;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      line[k] = l, pos[k] = p;
      l += dl, p += dp;
      if (p >= P) p -= P, ++l;
    }
  }
  __device__ __forceinline__ bool ok(int k) const {
    return (int)threadIdx.x + k * NT < total;
  }
  __device__ __forceinline__ int x(const AxisJob &j, int k) const {
    return pos[k] < j.L ? j.s0[0] + pos[k] : j.s0[1] + pos[k] - j.L;
  }
  __device__ __forceinline__ int field(const StepGrid &g, int k, int x) const {
    return line[k] * g.pitch + x;
  }
  __device__ __forceinline__ int mem(const AxisJob &j, int k, int x) const {
    return line[k] * j.len + cidx(x, j.half, j.len, j.n);
  }
  __device__ __forceinline__ int slot(const AxisJob &j, int k) const {
    const int seg = pos[k] < j.L ? 0 : 1;
    return (line[k] * j.nseg + seg) * pitch + 4 + pos[k] - seg * j.L;
  }
  __device__ __forceinline__ int64_t shell(const Shell &sh, int k, int x) const {
    const int y = y0 + line[k];
    const int b = near(sh, 2, z) || near(sh, 1, y) ? row_box(sh, y, z)
                  : x < sh.lo[0]                   ? sh.id[4]
                                                   : sh.id[5];
    return shell_row(sh, b, y, z) + x;
  }
  __device__ __forceinline__ void zero_ends(float *s, const AxisJob &j) const {
    for (int e = threadIdx.x; e < j.rows * j.nseg * 8; e += NT) {
      const int l = e / 8, c = e % 8;
      s[l * pitch + (c < 4 ? c : j.L + c)] = 0.0f;
    }
  }
};

template <int NT, int N>
__global__ void __launch_bounds__(NT)
    k_cpml_forward_x(StepGrid g, AxisJob j, Shell sh, const float *__restrict__ w,
                     float *__restrict__ psi, float *__restrict__ zeta, float *__restrict__ out,
                     float *__restrict__ cstore) {
  extern __shared__ float smem[];
  const RowTile<NT, N> t(g, j);
  float *sw = smem, *sp = smem + j.rows * j.nseg * t.pitch;
  t.zero_ends(sw, j);
  t.zero_ends(sp, j);
  const bool near_z = near(sh, 2, t.z);
  w += t.fb, psi += t.mb, zeta += t.mb;
  const float *kk = g.k + t.fb;
  float *o = out ? out + t.fb : nullptr;
  float ps[N], ze[N], ov[N], kv[N];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    ps[k] = ze[k] = ov[k] = kv[k] = 0.0f;
    if (!t.ok(k)) continue;
    const int x = t.x(j, k);
    sw[t.slot(j, k)] = w[t.field(g, k, x)];
    if (j.a[x] != 0.0f) {
      ps[k] = psi[t.mem(j, k, x)];
      ze[k] = zeta[t.mem(j, k, x)];
    }
    if (o && near(sh, 0, x) && !near_z && !near(sh, 1, t.y0 + t.line[k])) {
      ov[k] = o[t.field(g, k, x)];
      kv[k] = kk[t.field(g, k, x)];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if (!t.ok(k)) continue;
    const int x = t.x(j, k);
    const float a = j.a[x];
    if (a != 0.0f) {
      ps[k] = recursion<0>(j.b[x], ps[k], a, j.ih * first_diff(sw + t.slot(j, k), 1));
      psi[t.mem(j, k, x)] = ps[k];
    }
    sp[t.slot(j, k)] = ps[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const int x = t.x(j, k);
    if (!t.ok(k) || !near(sh, 0, x)) continue;
    const float a = j.a[x], d1 = first_diff(sp + t.slot(j, k), 1), d1p = j.ih * d1;
    float c = d1p;
    if (a != 0.0f) {
      const float d2 = second_diff(sw + t.slot(j, k), 1);
      const float v = recursion<0>(j.b[x], ze[k], a, __builtin_fmaf(j.c2, d2, d1p));
      zeta[t.mem(j, k, x)] = v;
      c += v;
    }
    const bool more = near_z || near(sh, 1, t.y0 + t.line[k]);
    if (o && !more && t.z > g.zs) o[t.field(g, k, x)] = __builtin_fmaf(c, kv[k], ov[k]);
    if (cstore) cstore[t.shell(sh, k, x)] = c;
  }
}

template <int NT, int N>
__global__ void __launch_bounds__(NT)
    k_cpml_adjoint_x(StepGrid g, AxisJob j, Shell sh, const float *__restrict__ phi1,
                     float *__restrict__ nu, float *__restrict__ mu, float *__restrict__ phi,
                     const float *__restrict__ cstore, float *__restrict__ grad) {
  extern __shared__ float smem[];
  const RowTile<NT, N> t(g, j);
  float *sf = smem, *sn = smem + j.rows * j.nseg * t.pitch;
  t.zero_ends(sf, j);
  t.zero_ends(sn, j);
  const bool near_z = near(sh, 2, t.z);
  phi1 += t.fb, phi += t.fb, grad += t.fb, nu += t.mb, mu += t.mb;
  const float *kk = g.k + t.fb;
  float mv[N], pv[N], kv[N];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    mv[k] = pv[k] = kv[k] = 0.0f;
    if (!t.ok(k)) continue;
    const int x = t.x(j, k), f = t.field(g, k, x);
    const float fv = phi1[f], a = j.a[x];
    float an = 0.0f;
    if (a != 0.0f) {
      mv[k] = mu[t.mem(j, k, x)];
      const float v = fv + j.b[x] * nu[t.mem(j, k, x)];
      nu[t.mem(j, k, x)] = v;
      an = a * v;
    }
    sn[t.slot(j, k)] = an;
    sf[t.slot(j, k)] = an + fv;
    if (!near(sh, 0, x)) continue;
    pv[k] = phi[f];
    kv[k] = kk[f];
    if (cstore && !near_z && !near(sh, 1, t.y0 + t.line[k]))
      grad[f] += fv * cstore[t.shell(sh, k, x)];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if (!t.ok(k)) continue;
    const int x = t.x(j, k);
    const float a = j.a[x];
    if (a != 0.0f) {
      const float v = j.b[x] * mv[k] - first_diff(sf + t.slot(j, k), 1) * j.ih;
      mu[t.mem(j, k, x)] = v;
      mv[k] = a * v;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k)
    if (t.ok(k)) sf[t.slot(j, k)] = mv[k];  // a mu, zero off the layer
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const int x = t.x(j, k);
    if (!t.ok(k) || !near(sh, 0, x) || t.z <= g.zs) continue;
    const float d2 = second_diff(sn + t.slot(j, k), 1);
    phi[t.field(g, k, x)] =
        pv[k] + kv[k] * (d2 * j.c2 - first_diff(sf + t.slot(j, k), 1) * j.ih);
  }
}

__global__ void k_record(const float *__restrict__ field, const int64_t *__restrict__ idx,
                         const float *__restrict__ scale, int nrec, int n,
                         float *__restrict__ seis_tm) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < nrec) seis_tm[(int64_t)n * nrec + r] = scale[r] * field[idx[r]];
}

AxisJob axis_job(const StepGrid &g, const CpmlTables &t, const Shell &sh, int d) {
  AxisJob j{};
  const int n = d == 0 ? g.nx : d == 1 ? g.ny : g.nz;
  j.a = d == 0 ? t.ax : d == 1 ? t.ay : t.az;
  j.b = d == 0 ? t.bx : d == 1 ? t.by : t.bz;
  j.ih = d == 0 ? t.ihx : d == 1 ? t.ihy : t.ihz;
  j.c2 = d == 0 ? g.cx : d == 1 ? g.cy : g.cz;
  j.n = n, j.half = t.half[d], j.len = t.len[d];
  if (t.len[d] == n) {  // the two ends' slabs meet: the whole axis
    j.nseg = 1, j.L = n;
  } else {
    j.L = n - 1 - sh.hi[d];
    j.nseg = sh.lo[d] > 0 ? 2 : 1;
    j.s0[0] = j.nseg == 2 ? 0 : n - j.L;
    j.s0[1] = n - j.L;
  }
  return j;
}

// Calls f(threads, tile width T, cells per thread R, image) with the smallest
// tile that takes a segment of L cells: 64 lines up to 96 cells (borders to 92), 32
// up to 192, so that a tile's LDS stays below 64 KB and a thread's cells in
// registers; false for longer ones, whose lines are marched in memory (forward
// steps of 320^3 with a layer of 100 cells: 772 us in 32 lines, 1451 in tiles of 16;
// 500^3 with 200: 4137 marched, 4768 in 16; 840^3 with 390: 23.6 ms, 81 in tiles of
// 2; the kernels without tiles 854, 3972 and 21.9 ms).  Whole axes with image cells
// are short (under 2 B + 16 cells) and rare: fewer shapes.
template <class F>
bool plane_shape(int L, bool img, F f) {
#define WFD_PLANE(NT, T, R, IMG)                                                      \
  if (L <= NT / T * R) {                                                              \
    f(std::integral_constant<int, NT>{}, std::integral_constant<int, T>{},            \
      std::integral_constant<int, R>{}, std::integral_constant<bool, IMG>{});         \
    return true;                                                                      \
  }
  if (img) {
    WFD_PLANE(512, 64, 6, true)
    WFD_PLANE(1024, 64, 6, true)
    return false;
  }
  WFD_PLANE(256, 64, 3, false)
  WFD_PLANE(256, 64, 5, false)
  WFD_PLANE(256, 64, 6, false)
  WFD_PLANE(512, 64, 5, false)
  WFD_PLANE(512, 64, 6, false)
  WFD_PLANE(1024, 64, 6, false)
  WFD_PLANE(1024, 32, 4, false)
  WFD_PLANE(1024, 32, 6, false)
#undef WFD_PLANE
  return false;
}

// Blocks of the long segments' kernels.
int64_t long_blocks(const StepGrid &g, AxisJob &p, int axis) {
  p.tiles = (g.nx + 63) / 64;
  const int chunks = (p.L + kLongCells - 1) / kLongCells;
  return (int64_t)p.tiles * chunks * p.nseg * (((axis == 1 ? g.nz : g.ny) + 3) / 4);
}

// Calls f(threads) for an x job, three elements per thread: as many rows of a
// plane as 256 threads take, or one row by 1024 threads (segments up to 3072
// cells, as above).
template <class F>
bool row_shape(const StepGrid &g, AxisJob &j, F f) {
  const int P = j.nseg * j.L;
  j.rows = std::max(1, std::min(g.ny, 3 * 256 / P));
  j.tiles = (g.ny + j.rows - 1) / j.rows;
  if (P <= 3 * 256) f(std::integral_constant<int, 256>{});
  else if (P <= 3 * 1024) f(std::integral_constant<int, 1024>{});
  else return false;
  return true;
}

bool image_axis(const StepGrid &g, const AxisJob &j, int axis) {
  return axis == 2 && j.nseg == 1 && j.L == j.n && g.zs != kNoSurface;
}

}  // namespace

hipError_t launch_cpml_forward(const StepGrid &g, const CpmlTables &t, const Shell &sh,
                               const float *cur, float *const mem[6], float *out, float *cstore,
                               hipStream_t stream) {
  if (sh.points == 0) return hipSuccess;
  AxisJob j = axis_job(g, t, sh, 0);
  const bool fits = row_shape(g, j, [&](auto nt) {
    const size_t lds = 2 * sizeof(float) * (size_t)j.rows * j.nseg * (j.L + 8);
    constexpr int NT = decltype(nt)::value;
    for_launches((int64_t)j.tiles * g.nz, NT, [&](uint32_t first, uint32_t count) {
      j.first = first;
      hipLaunchKernelGGL((k_cpml_forward_x<NT, 3>), dim3(count), dim3(NT), lds, stream, g, j, sh,
                         cur, mem[0], mem[3], out, cstore);
    });
  });
  if (!fits) return hipErrorInvalidValue;
  auto crossed = [&](const AxisJob &q, int d) {
    return Crossed{mem[d], mem[3 + d], q.ih, q.n, q.half, q.len};
  };
  const Crossed cx = crossed(j, 0), cy = crossed(axis_job(g, t, sh, 1), 1);
  auto plane = [&](auto ax, auto store) {
    constexpr int A = decltype(ax)::value;
    AxisJob p = axis_job(g, t, sh, A);
    const bool tiled = plane_shape(p.L, image_axis(g, p, A), [&](auto nt, auto t_, auto r, auto img) {
      constexpr int NT = decltype(nt)::value, T = decltype(t_)::value, R = decltype(r)::value;
      constexpr bool IMG = decltype(img)::value, STORE = decltype(store)::value;
      if constexpr (A == 2 || !IMG) {
        p.tiles = (g.nx + T - 1) / T;
        const int64_t blocks = (int64_t)p.tiles * (A == 1 ? g.nz : g.ny) * p.nseg;
        for_launches(blocks, NT, [&](uint32_t first, uint32_t count) {
          p.first = first;
          hipLaunchKernelGGL((k_cpml_forward<A, NT, T, R, IMG, STORE>), dim3(count), dim3(NT), 0,
                             stream, g, p, sh, cur, mem[A], mem[3 + A], out, cstore, cx, cy);
        });
      }
    });
    if (tiled) return;
    const int64_t blocks = long_blocks(g, p, A);
    for_launches(blocks, 256, [&](uint32_t first, uint32_t count) {
      p.first = first;
      hipLaunchKernelGGL(k_cpml_psi_long<A>, dim3(count), dim3(256), 0, stream, g, p, cur, mem[A]);
    });
    for_launches(blocks, 256, [&](uint32_t first, uint32_t count) {
      p.first = first;
      hipLaunchKernelGGL(k_cpml_zeta_long<A>, dim3(count), dim3(256), 0, stream, g, p, sh, cur,
                         mem[A], mem[3 + A], out, cstore, cx, cy);
    });
  };
  auto planes = [&](auto store) {
    plane(std::integral_constant<int, 1>{}, store);
    plane(std::integral_constant<int, 2>{}, store);
  };
  if (cstore) planes(std::true_type{});
  else planes(std::false_type{});
  return hipGetLastError();
}

hipError_t launch_cpml_adjoint(const StepGrid &g, const CpmlTables &t, const Shell &sh,
                               const float *phi1, float *const mem[6], float *phi,
                               const float *cstore, float *grad, hipStream_t stream) {
  if (sh.points == 0) return hipSuccess;
  AxisJob j = axis_job(g, t, sh, 0);
  const bool fits = row_shape(g, j, [&](auto nt) {
    const size_t lds = 2 * sizeof(float) * (size_t)j.rows * j.nseg * (j.L + 8);
    constexpr int NT = decltype(nt)::value;
    for_launches((int64_t)j.tiles * g.nz, NT, [&](uint32_t first, uint32_t count) {
      j.first = first;
      hipLaunchKernelGGL((k_cpml_adjoint_x<NT, 3>), dim3(count), dim3(NT), lds, stream, g, j, sh,
                         phi1, mem[3], mem[0], phi, cstore, grad);
    });
  });
  if (!fits) return hipErrorInvalidValue;
  auto plane = [&](auto ax) {
    constexpr int A = decltype(ax)::value;
    AxisJob p = axis_job(g, t, sh, A);
    const bool tiled = plane_shape(p.L, image_axis(g, p, A), [&](auto nt, auto t_, auto r, auto img) {
      constexpr int NT = decltype(nt)::value, T = decltype(t_)::value, R = decltype(r)::value;
      constexpr bool IMG = decltype(img)::value;
      if constexpr (A == 2 || !IMG) {
        p.tiles = (g.nx + T - 1) / T;
        const int64_t blocks = (int64_t)p.tiles * (A == 1 ? g.nz : g.ny) * p.nseg;
        for_launches(blocks, NT, [&](uint32_t first, uint32_t count) {
          p.first = first;
          hipLaunchKernelGGL((k_cpml_adjoint<A, NT, T, R, IMG>), dim3(count), dim3(NT), 0, stream,
                             g, p, sh, phi1, mem[3 + A], mem[A], phi, cstore, grad);
        });
      }
    });
    if (tiled) return;
    const int64_t blocks = long_blocks(g, p, A);
    for_launches(blocks, 256, [&](uint32_t first, uint32_t count) {
      p.first = first;
      hipLaunchKernelGGL(k_cpml_nu_long<A>, dim3(count), dim3(256), 0, stream, g, p, sh, phi1,
                         mem[3 + A], cstore, grad);
    });
    for_launches(blocks, 256, [&](uint32_t first, uint32_t count) {
      p.first = first;
      hipLaunchKernelGGL(k_cpml_mu_long<A>, dim3(count), dim3(256), 0, stream, g, p, phi1,
                         mem[3 + A], mem[A]);
    });
    for_launches(blocks, 256, [&](uint32_t first, uint32_t count) {
      p.first = first;
      hipLaunchKernelGGL(k_cpml_phi_long<A>, dim3(count), dim3(256), 0, stream, g, p, sh,
                         mem[3 + A], mem[A], phi);
    });
  };
  plane(std::integral_constant<int, 1>{});
  plane(std::integral_constant<int, 2>{});
  return hipGetLastError();
}

hipError_t launch_record(const float *field, const int64_t *idx, const float *scale, int nrec,
                         int n, float *seis_tm, hipStream_t stream) {
  if (nrec <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_record, dim3((unsigned)((nrec + 255) / 256)), dim3(256), 0, stream, field,
                     idx, scale, nrec, n, seis_tm);
  return hipGetLastError();
}

}  // namespace wfd
