// Gradient smoothing (the paper's GradientPreconditioning: Laplace or Bessel
// filter with lengths l_x, l_y, l_z).  Volumes are [z][y][x] FP32.
//
// Laplace filter: along each axis, solve the tridiagonal system
//   [(1 + a^2) I - a (S + S^-1)] u = (1 - a)^2 g,  a = exp(-h / l),
// whose inverse is the exponential kernel (1 - a)/(1 + a) a^|n|; the end rows
// use a mirror (zero-flux) condition so constants are kept.  Solved by the
// Thomas algorithm in FP64, a tile of lines per block.
//
// Bessel filter: u = B^-1 g with B = I - sum_d l_d^2 D_dd (3-point second
// differences, zero-flux ends), symmetric positive definite; conjugate
// gradients with this matrix-vector product and FP64 inner products.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "wfd_internal.h"

namespace wfd {
namespace {

constexpr size_t kTileBytes = 64 << 10;  // LDS of a block's lines: two blocks per CU at least
constexpr size_t kCuLds = 160 << 10;
constexpr double kCachedBytes = 256e6;  // last-level cache

// Line L of an axis: first point and stride between consecutive points.
__device__ __forceinline__ void line_of(int axis, int64_t L, int nx, int ny, int64_t &base,
                                        int64_t &stride) {
  if (axis == 0) {  // x lines
    base = L * nx;
    stride = 1;
  } else if (axis == 1) {  // y lines: L = z * nx + x
    const int64_t x = L % nx, z = L / nx;
    base = z * (int64_t)ny * nx + x;
    stride = nx;
  } else {  // z lines: L = y * nx + x
    base = L;
    stride = (int64_t)nx * ny;
  }
}

// The elimination's denominators and off-diagonals in closed form: with the
// zero-flux ends the leading minors of (1 - a)^2 T are proportional to
// 1 + a^(2i+1), so row i has den_i = (1 + a^(2i+3)) / (1 + a^(2i+1)), the last
// row (1 - a)(1 - a^(2n)) / (1 + a^(2n-1)).  With s_i = (1 - a)^2 / den_i and
// c_i = a / den_i the solution is one multiply-add per point each way:
//   d_i = s_i g_i + c_i d_{i-1},   x_i = d_i + c_i x_{i+1}   (x_{n-1} = d_{n-1}).
struct TriRow {
  double s, c;
};
__device__ __forceinline__ TriRow tri_row(int i, int n, double log_a, double a) {
  const double p = exp((2.0 * i + 1.0) * log_a), q = expm1(log_a);
  const double inv = i + 1 < n ? (1.0 + p) / (1.0 + p * a * a)
                               : (1.0 + p) / (q * expm1(2.0 * n * log_a));
  return TriRow{q * q * inv, a * inv};
}

// A block solves NL neighbouring lines: it loads them into LDS with every
// thread, one thread per line runs the recursion there (FP64, d kept in FP32),
// and every thread writes them back.  Each point moves once in and once out
// (8 B) instead of twice each.  S1: the lines run along x and lie next to one
// another; else their points i are `stride` apart and neighbouring lines are
// neighbouring elements (y lines: within one plane).  200 x 200 x 160: 24, 31
// and 24 us along x, y and z (load, march and store of a block follow one
// another); 146, 106 and 69 us with a thread marching each line in memory.
template <bool S1>
__global__ void __launch_bounds__(256)
    k_tri_tile(const float *in, float *out, int n, int64_t nlines, int nx, int ny, int axis,
               int nl, int pad, double log_a, double a) {
  extern __shared__ char smem[];
  TriRow *row = reinterpret_cast<TriRow *>(smem);
  float *u = reinterpret_cast<float *>(row + n);
  const int64_t l0 = (int64_t)blockIdx.x * nl;
  const int lines = (int)(nlines - l0 < nl ? nlines - l0 : nl);
  const int tid = threadIdx.x;
  // element (line l, point i) sits at u[l * pad + i] (S1) or u[i * nl + l]
  if (S1) {
    // thread tid takes elements tid, tid + 256, ..: (l, i) kept by steps
    const int ql = 256 / n, qi = 256 - ql * n, total = lines * n;
    int l = tid / n, i = tid - l * n;
#pragma unroll 8
    for (int e = tid; e < total; e += 256) {
      u[l * pad + i] = in[l0 * n + e];
      i += qi, l += ql;
      if (i >= n) i -= n, ++l;
    }
  } else {
    const int l = tid % nl;
    int64_t base = 0, stride = 0;
    if (l < lines) line_of(axis, l0 + l, nx, ny, base, stride);
    const int step = 256 / nl;
    if (l < lines)
#pragma unroll 8
      for (int i = tid / nl; i < n; i += step) u[i * nl + l] = in[base + i * stride];
  }
  for (int i = tid; i < n; i += 256) row[i] = tri_row(i, n, log_a, a);
  __syncthreads();
  if (tid < lines) {
    float *p = S1 ? u + tid * pad : u + tid;
    const int st = S1 ? 1 : nl;
    double d = 0.0;
#pragma unroll 8
    for (int i = 0; i < n; ++i) {
      d = fma(row[i].c, d, row[i].s * (double)p[i * st]);
      p[i * st] = (float)d;
    }
    double x = d;
#pragma unroll 8
    for (int i = n - 2; i >= 0; --i) {
      x = fma(row[i].c, x, (double)p[i * st]);
      p[i * st] = (float)x;
    }
  }
  __syncthreads();
  if (S1) {
    const int ql = 256 / n, qi = 256 - ql * n, total = lines * n;
    int l = tid / n, i = tid - l * n;
#pragma unroll 8
    for (int e = tid; e < total; e += 256) {
      out[l0 * n + e] = u[l * pad + i];
      i += qi, l += ql;
      if (i >= n) i -= n, ++l;
    }
  } else {
    const int l = tid % nl;
    int64_t base = 0, stride = 0;
    if (l < lines) line_of(axis, l0 + l, nx, ny, base, stride);
    const int step = 256 / nl;
    if (l < lines)
#pragma unroll 8
      for (int i = tid / nl; i < n; i += step) out[base + i * stride] = u[i * nl + l];
  }
}

// The rows' coefficients, for the kernel below.
__global__ void __launch_bounds__(256) k_tri_rows(TriRow *__restrict__ row, int n, double log_a,
                                                  double a) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) row[i] = tri_row(i, n, log_a, a);
}

// Lines that a tile does not take or takes longer (tri_tile_lines): one thread
// marches each line in memory.
__global__ void k_tri_lines(const float *in, float *out, int axis, int n, int64_t nlines, int nx,
                            int ny, const TriRow *__restrict__ row) {
  const int64_t L = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (L >= nlines) return;
  int64_t base, stride;
  line_of(axis, L, nx, ny, base, stride);
  double d = 0.0;
  for (int i = 0; i < n; ++i) {
    const int64_t p = base + (int64_t)i * stride;
    d = fma(row[i].c, d, row[i].s * (double)in[p]);
    out[p] = (float)d;
  }
  double x = d;
  for (int i = n - 2; i >= 0; --i) {
    const int64_t p = base + (int64_t)i * stride;
    x = fma(row[i].c, x, (double)out[p]);
    out[p] = (float)x;
  }
}

// Conjugate gradients on B u = g from u = 0, two kernels per iteration whose
// scalars stay on the device, so that iterations are enqueued without waiting:
//   direction: beta = rr_k / rr_{k-1};  p_k = r + beta p_{k-1};  <p, B p>
//   update:    alpha = rr_k / <p, B p>;  x += alpha p;  r -= alpha B p;  <r, r>
// Each kernel first sums the partials of the one before (every block, in the
// same order) and does nothing once rr_k <= tol^2 <g, g>.  Both form B p at
// their points themselves (the direction kernel from r and p_{k-1} of the
// seven points), so B p is never stored: 12 and 20 B per point.  A block
// marches 256 consecutive points of an x-y plane (rows of any length fill its
// lanes) along z; the z neighbours are kept in registers, the others come
// through the caches.  200 x 200 x 160: 22 and 25 us, 3.5 and 5.1 TB/s of those
// bytes (30 and 30 with neighbouring rows on different XCDs; loading a plane
// ahead changed nothing); 1024 blocks take 27 and 23 us.
struct Cg {
  double rr[2];  // rr_k in [k & 1]
  double gg;
  int it, pad;   // iterations begun
};
constexpr int kCgBlock = 256;

struct CgGrid {
  int nx, ny, nz, zc, nch;  // z planes per chunk, chunks
  int64_t plane, pblocks, items;
  float cx, cy, cz;
};

// Sum over the block of one FP64 value per thread, to every thread.
__device__ __forceinline__ double cg_block_sum(double v) {
  __shared__ double part[kCgBlock / 64];
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  return (part[0] + part[1]) + (part[2] + part[3]);
}
__device__ __forceinline__ double cg_partials(const double *__restrict__ part, int np) {
  double v = 0.0;
  for (int i = threadIdx.x; i < np; i += kCgBlock) v += part[i];
  return cg_block_sum(v);
}

// Calls f(i, c, v) for the block's points: element i, c = p, v = (B p).
// at(i) gives p at element i.
template <class At, class F>
__device__ __forceinline__ void cg_march(const CgGrid &g, At at, F f) {
  // block b runs on XCD b mod 8: neighbouring rows of a plane share an L2
  const int per = gridDim.x / 8, rem = gridDim.x % 8, xcd = blockIdx.x % 8;
  const int first = xcd * per + (xcd < rem ? xcd : rem) + blockIdx.x / 8;
  for (int64_t item = first; item < g.items; item += gridDim.x) {
    const int64_t ch = item / g.pblocks, l = (item - ch * g.pblocks) * kCgBlock + threadIdx.x;
    if (l >= g.plane) continue;
    const int iy = (int)(l / g.nx), ix = (int)(l - (int64_t)iy * g.nx);
    const int z0 = (int)ch * g.zc, z1 = z0 + g.zc < g.nz ? z0 + g.zc : g.nz;
    // a neighbour past an end reads the point itself: no difference (zero flux)
    const int64_t xm = ix > 0 ? -1 : 0, xp = ix < g.nx - 1 ? 1 : 0;
    const int64_t ym = iy > 0 ? -(int64_t)g.nx : 0, yp = iy < g.ny - 1 ? g.nx : 0;
    int64_t i = z0 * g.plane + l;
    float c = at(i), zm = z0 > 0 ? at(i - g.plane) : c;
    for (int z = z0; z < z1; ++z, i += g.plane) {
      const float zp = z < g.nz - 1 ? at(i + g.plane) : c;
      float dxx = 0.0f, dyy = 0.0f, dzz = 0.0f;
      dxx += at(i + xm) - c;
      dxx += at(i + xp) - c;
      dyy += at(i + ym) - c;
      dyy += at(i + yp) - c;
      dzz += zm - c;
      dzz += zp - c;
      f(i, c, c - (g.cx * dxx + g.cy * dyy + g.cz * dzz));
      zm = c;
      c = zp;
    }
  }
}

template <bool FIRST>
__global__ void __launch_bounds__(kCgBlock, 8)
    k_cg_direction(CgGrid g, int k, double tol2, const float *__restrict__ r,
                   const float *__restrict__ p_old, float *__restrict__ p, Cg *cg,
                   const double *__restrict__ part_rr, double *__restrict__ part_pap) {
  const double rr = cg_partials(part_rr, gridDim.x);
  const double gg = FIRST ? rr : cg->gg;
  const bool go = rr > tol2 * gg;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    cg->rr[k & 1] = rr;
    if (FIRST) cg->gg = gg;
    if (go) cg->it = k + 1;
  }
  if (!go) return;
  const float beta = FIRST ? 0.0f : (float)(rr / cg->rr[(k + 1) & 1]);
  double s = 0.0;
  cg_march(g, [&](int64_t i) { return FIRST ? r[i] : r[i] + beta * p_old[i]; },
           [&](int64_t i, float c, float v) {
             p[i] = c;
             s += (double)c * (double)v;
           });
  s = cg_block_sum(s);
  if (threadIdx.x == 0) part_pap[blockIdx.x] = s;
}

__global__ void __launch_bounds__(kCgBlock, 8)
    k_cg_update(CgGrid g, int k, double tol2, float *__restrict__ x, float *__restrict__ r,
                const float *__restrict__ p, const Cg *cg, const double *__restrict__ part_pap,
                double *__restrict__ part_rr) {
  const double rr = cg->rr[k & 1];
  if (!(rr > tol2 * cg->gg)) return;
  const float alpha = (float)(rr / cg_partials(part_pap, gridDim.x));
  double s = 0.0;
  cg_march(g, [&](int64_t i) { return p[i]; },
           [&](int64_t i, float c, float v) {
             x[i] += alpha * c;
             const float ri = r[i] - alpha * v;
             r[i] = ri;
             s += (double)ri * (double)ri;
           });
  s = cg_block_sum(s);
  if (threadIdx.x == 0) part_rr[blockIdx.x] = s;
}

// rr after the iterations enqueued so far, for the host.
__global__ void __launch_bounds__(kCgBlock)
    k_cg_check(int np, const double *__restrict__ part_rr, const Cg *__restrict__ cg,
               double *__restrict__ out) {
  const double rr = cg_partials(part_rr, np);
  if (threadIdx.x == 0) {
    out[0] = rr;
    out[1] = cg->gg;
    out[2] = (double)cg->it;
  }
}

__global__ void __launch_bounds__(kCgBlock)
    k_cg_start(const float *__restrict__ g, float *__restrict__ r, float *__restrict__ x,
               int64_t n, Cg *cg, double *__restrict__ part_rr) {
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kCgBlock + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kCgBlock) {
    const float v = g[i];
    r[i] = v;
    x[i] = 0.0f;
    s += (double)v * (double)v;
  }
  s = cg_block_sum(s);
  if (threadIdx.x == 0) part_rr[blockIdx.x] = s;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    cg->it = 0;
    cg->gg = 0.0;
  }
}

CgGrid cg_grid(int nx, int ny, int nz, float cx, float cy, float cz) {
  CgGrid g{};
  g.nx = nx, g.ny = ny, g.nz = nz;
  g.plane = (int64_t)nx * ny;
  g.pblocks = (g.plane + kCgBlock - 1) / kCgBlock;
  // as many z chunks as make one item per block of a full device
  const int64_t want = std::max<int64_t>(1, std::min<int64_t>(nz, kCgMaxBlocks / g.pblocks));
  g.zc = (int)((nz + want - 1) / want);
  g.nch = (nz + g.zc - 1) / g.zc;
  g.items = g.pblocks * g.nch;
  g.cx = cx, g.cy = cy, g.cz = cz;
  return g;
}

constexpr int tri_pad(int n) { return n | 1; }  // odd: a wavefront's x lines start in different banks

size_t tri_tile_bytes(int axis, int n, int nl) {
  return (size_t)n * sizeof(TriRow) + (size_t)nl * (axis == 0 ? tri_pad(n) : n) * sizeof(float);
}

}  // namespace

// Lines of a tile of an axis' n-point lines, 0 where each line is marched in
// memory.
int tri_tile_lines(int axis, int n, int64_t nlines) {
  // As many lines per block, 64 at most, as fit the LDS tile; fewer where
  // that leaves compute units without a block (200 x 200 x 160, three axes: 78
  // us with at least one block a unit, 83 with two, 95 with four).
  int nl = 64;
  while (nl > 8 && (tri_tile_bytes(axis, n, nl) > kTileBytes || nlines < (int64_t)nl * 256))
    nl /= 2;
  if (tri_tile_bytes(axis, n, nl) > kTileBytes) return 0;
  // a launch takes less than 2^32 threads (the march one a line)
  if ((nlines + nl - 1) / nl * 256 >= (int64_t(1) << 32)) return 0;
  if (axis == 0) return nl;  // 40000 lines of 1300: 760 us against 1340
  // Along y and z a march is coalesced and every line is a thread, while a tile
  // holds a few lines of a long axis and only they march.  In us per point of a
  // line: tiles 0.093 a round of resident blocks plus 8 B a point at 5 TB/s; a
  // march 0.55 (its latency) and more with the lines, less past 100000 of them.
  // Calls over one axis, tile / march, y and z (the rule's choice first where
  // both are given): 40000 lines of 816 points 424 / 515 and 415 / 471, of 1300
  // march 1072 for 1203 and 859 for 1227; 90000 of 600 tile 524 for 616 on y, of
  // 1000 march 1033 for 1440 and 975 for 1449; 250000 of 240 tile 310 for 361 and
  // 301 for 330, of 400 march 601 for 730 and 550 for 718, of 1000 march 1508 for
  // 3766 and 1421 for 3844.
  const double resident = std::min<double>(8.0, std::floor(kCuLds / tri_tile_bytes(axis, n, nl)));
  const double rounds = std::ceil((double)nlines / (256.0 * resident * nl));
  const double tile = 0.093 * rounds + 1.6e-6 * (double)nlines;
  const double few = std::min(1e5, (double)nlines), more = (double)nlines - few;
  const double march = axis == 1 ? 0.55 + 5.0e-6 * few + 2.6e-6 * more
                                 : 0.55 + 3.6e-6 * few + 2.2e-6 * more;
  return tile <= march ? nl : 0;
}

hipError_t launch_tri_lines(const float *in, float *out, int axis, int n, int64_t nlines, int nx,
                            int ny, double h_over_l, double *table, hipStream_t stream) {
  const double a = std::exp(-h_over_l);
  const int nl = tri_tile_lines(axis, n, nlines);
  if (nl == 0) {
    // In place along x (half the cache lines: 90000 lines of 1400 points 2816 us
    // against 2946) and where the volume fits the last-level cache, which the copy
    // leaves it in (40000 z lines of 1300 859 / 977; 90000 of 816, 294 MB, 862 /
    // 788).
    const int64_t points = (int64_t)n * nlines;
    if (in != out && (axis == 0 || 4.0 * (double)points <= kCachedBytes)) {
      const hipError_t e = hipMemcpyAsync(out, in, (size_t)points * sizeof(float),
                                          hipMemcpyDeviceToDevice, stream);
      if (e != hipSuccess) return e;
      in = out;
    }
    TriRow *row = reinterpret_cast<TriRow *>(table);
    hipLaunchKernelGGL(k_tri_rows, dim3((n + 255) / 256), dim3(256), 0, stream, row, n, -h_over_l,
                       a);
    hipLaunchKernelGGL(k_tri_lines, dim3((unsigned)((nlines + 255) / 256)), dim3(256), 0, stream,
                       in, out, axis, n, nlines, nx, ny, row);
    return hipGetLastError();
  }
  const dim3 grid((unsigned)((nlines + nl - 1) / nl));
  const size_t lds = tri_tile_bytes(axis, n, nl);
  if (axis == 0)
    hipLaunchKernelGGL(k_tri_tile<true>, grid, dim3(256), lds, stream, in, out, n, nlines, nx, ny,
                       axis, nl, tri_pad(n), -h_over_l, a);
  else
    hipLaunchKernelGGL(k_tri_tile<false>, grid, dim3(256), lds, stream, in, out, n, nlines, nx,
                       ny, axis, nl, tri_pad(n), -h_over_l, a);
  return hipGetLastError();
}

// Scratch: Cg, the two kernels' block sums, the check's three values.
size_t cg_scratch_bytes(int blocks) { return sizeof(Cg) + (2 * (size_t)blocks + 4) * sizeof(double); }

// Blocks of a kernel: an item each, as far as the scratch has room for their sums.
int cg_blocks(int nx, int ny, int nz, size_t scratch_bytes) {
  const int64_t room = ((int64_t)scratch_bytes - (int64_t)cg_scratch_bytes(0)) /
                       (int64_t)(2 * sizeof(double));
  return (int)std::min(std::min<int64_t>(kCgMaxBlocks, room),
                       cg_grid(nx, ny, nz, 0, 0, 0).items);
}

hipError_t launch_cg_start(const float *in, float *x, float *vols, int64_t n, int blocks,
                           void *scratch, hipStream_t stream) {
  Cg *cg = static_cast<Cg *>(scratch);
  hipLaunchKernelGGL(k_cg_start, dim3(blocks), dim3(kCgBlock), 0, stream, in, vols, x, n, cg,
                     reinterpret_cast<double *>(cg + 1));
  return hipGetLastError();
}

hipError_t launch_cg_iteration(int k, double tol2, int nx, int ny, int nz, float cx, float cy,
                               float cz, float *x, float *vols, int blocks, void *scratch,
                               hipStream_t stream) {
  const CgGrid g = cg_grid(nx, ny, nz, cx, cy, cz);
  const int64_t n = g.plane * nz;
  Cg *cg = static_cast<Cg *>(scratch);
  double *rr = reinterpret_cast<double *>(cg + 1), *pap = rr + blocks;
  float *r = vols, *p = vols + n * (1 + (k & 1)), *p_old = vols + n * (2 - (k & 1));
  if (k == 0)
    hipLaunchKernelGGL(k_cg_direction<true>, dim3(blocks), dim3(kCgBlock), 0, stream, g, k, tol2,
                       r, p_old, p, cg, rr, pap);
  else
    hipLaunchKernelGGL(k_cg_direction<false>, dim3(blocks), dim3(kCgBlock), 0, stream, g, k, tol2,
                       r, p_old, p, cg, rr, pap);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_cg_update, dim3(blocks), dim3(kCgBlock), 0, stream, g, k, tol2, x, r, p, cg,
                     pap, rr);
  return hipGetLastError();
}

hipError_t launch_cg_check(int blocks, void *scratch, double **out, hipStream_t stream) {
  Cg *cg = static_cast<Cg *>(scratch);
  double *rr = reinterpret_cast<double *>(cg + 1);
  *out = rr + 2 * blocks;
  hipLaunchKernelGGL(k_cg_check, dim3(1), dim3(kCgBlock), 0, stream, blocks, rr, cg, *out);
  return hipGetLastError();
}

}  // namespace wfd

// ---- time resampling of traces -------------------------------------------------
// Trace sample k sits at (k + 1) dt.  nearest: round half up, clamped.  sinc:
// out[m] = sum_n in[n] sinc(a_m - n) with a_m = t_m / dt_in - 1; using
// sin(pi (a - n)) = (-1)^n sin(pi a) each weight is one reciprocal (FP64);
// an integer a_m selects the input sample.
//
// The sinc sum over all traces is a matrix product, in [nrec][nt_in] times
// W [nt_in][nt_out] with W[n][m] = (-1)^n / (a_m - n), on the FP64 matrix
// cores (FP64 products and sums).  A wavefront owns 16 RT traces x 16 output
// samples; for every 16 input samples it forms its 16 x 16 weights, four per
// lane, once, and uses them for RT products of each of four K steps.  The K
// index of a step is free as long as both operands agree: lane group g takes
// samples 4 g .. 4 g + 3, so that a lane's four samples of a trace are one
// 16-byte load.  Bound by the FP64 matrix rate (69 TFLOP/s measured on a large
// product): 2500 traces of 1200 -> 2400 samples (14.4 GFLOP) take 283 us, 65 %
// of them in products (the FP64 vector work of the weights and conversions does
// not overlap with them); one division per term on the vector unit took 4160.
namespace wfd {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
struct __attribute__((packed, aligned(4))) Quad {
  float v[4];
};

// Position of output sample m in input samples, as both modes take it.
__device__ __forceinline__ double sample_pos(int m, double dt_in, double dt_out) {
  return (double)(m + 1) * dt_out / dt_in - 1.0;
}

// Output elements of all traces in a row, so that every wavefront writes whole
// cache lines (8192 traces of 3000 samples: 46 us; 53 with blocks of one trace's
// samples, which start anywhere in a line).
__global__ void __launch_bounds__(256)
    k_resample_nearest(const float *__restrict__ in, int nrec, int nt_in, double dt_in,
                       float *__restrict__ out, int nt_out, double dt_out, uint32_t first) {
  const int64_t i = ((int64_t)first + blockIdx.x) * 256 + threadIdx.x;
  if (i >= (int64_t)nrec * nt_out) return;
  const int r = (int)(i / nt_out), m = (int)(i % nt_out);
  const double a = sample_pos(m, dt_in, dt_out);
  int n = (int)floor(a + 1.0 + 0.5) - 1;
  n = n < 0 ? 0 : (n > nt_in - 1 ? nt_in - 1 : n);
  out[i] = in[(int64_t)r * nt_in + n];
}

// 1 / x for a finite x of ordinary size: the hardware's estimate and two
// Newton steps.
__device__ __forceinline__ double reciprocal(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}

// Matrix-core mapping of v_mfma_f64_16x16x4_f64 (lane l): A[i][k] in lane
// i + 16 k, B[k][j] in lane j + 16 k, D[i][j] in lane j + 16 (i % 4), element
// i / 4.
template <int RT>
__global__ void __launch_bounds__(256)
    k_resample_sinc(const float *__restrict__ in, int nrec, int nt_in, double dt_in,
                    float *__restrict__ out, int nt_out, double dt_out, uint32_t col_blocks) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = lane & 15, g = lane >> 4;
  const uint32_t rb = blockIdx.x / col_blocks, cb = blockIdx.x - rb * col_blocks;
  const int64_t m0 = ((int64_t)cb * 4 + wave) * 16;
  if (m0 >= nt_out) return;
  const int64_t m = m0 + j < nt_out ? m0 + j : nt_out - 1;
  const double a = sample_pos((int)m, dt_in, dt_out);
  const double an = rint(a);
  const bool on = fabs(a - an) < 1e-12;  // on an input sample
  const double aw = on ? -0.5 : a;  // an on-sample column's weights are unused
  // sin(pi a) of the exact remainder: of a itself its error is a ulp of a, as
  // large as a position a rounding off its sample is away (1.2 or 0.1 for 1 past
  // sample 8192)
  const double scale = ((int64_t)an & 1 ? -sinpi(a - an) : sinpi(a - an)) / M_PI;
  const bool hit = on && an >= 0.0 && an < (double)nt_in;
  const int64_t rows = (int64_t)(gridDim.x / col_blocks) * (16 * RT);
  for (int64_t r0 = (int64_t)rb * (16 * RT); r0 < nrec; r0 += rows) {
    const float *row[RT];  // the lane's trace of every row tile, clamped to the last
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int64_t r = r0 + 16 * t + j;
      row[t] = in + (r < nrec ? r : (int64_t)nrec - 1) * nt_in + 4 * g;
    }
    f64x4 acc[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    // products of input samples n .. n + 3 (n = 4 g past a multiple of 16)
    auto products = [&](double n, const Quad *x) {
      const double d = aw - n;  // d and d - s are exact next to the sample at a
      double w[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) w[s] = reciprocal(s & 1 ? (double)s - d : d - (double)s);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < RT; ++t)
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x[t].v[s], w[s], acc[t], 0, 0, 0);
    };
    const int full = nt_in & ~15;
    double nf = 4.0 * g;
    Quad x[RT], y[RT];
    auto load = [&](Quad *q, int step) {
#pragma unroll
      for (int t = 0; t < RT; ++t) q[t] = *reinterpret_cast<const Quad *>(row[t] + 16 * step);
    };
    // 32 samples a turn, the next ones loading meanwhile (past the last whole
    // 16 the current ones again, unused)
    int n0 = 0;
    if (full > 0) load(x, 0);
    for (; n0 + 32 <= full; n0 += 32) {
      load(y, 1);
      products(nf, x);
#pragma unroll
      for (int t = 0; t < RT; ++t) row[t] += 32;
      load(x, n0 + 32 < full ? 0 : -1);
      products(nf + 16.0, y);
      nf += 32.0;
    }
    if (n0 < full) {
      products(nf, x);
      nf += 16.0;
    }
    if (full < nt_in) {  // the last samples, zeros past the end
      const int n = full + 4 * g;
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int s = 0; s < 4; ++s) x[t].v[s] = n + s < nt_in ? row[t][full - n0 + s] : 0.0f;
      products(nf, x);
    }
    if (m0 + j >= nt_out) continue;
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t r = r0 + 16 * t + 4 * e + g;
        if (r >= nrec) continue;
        float v = (float)(acc[t][e] * scale);
        if (on) v = hit ? in[r * nt_in + (int)an] : 0.0f;
        out[r * nt_out + m] = v;
      }
  }
}

}  // namespace

hipError_t launch_resample(const float *in, int nrec, int nt_in, double dt_in, float *out,
                           int nt_out, double dt_out, int sinc, hipStream_t stream) {
  if (!sinc) {
    for_launches(((int64_t)nrec * nt_out + 255) / 256, 256, [&](uint32_t first, uint32_t count) {
      hipLaunchKernelGGL(k_resample_nearest, dim3(count), dim3(256), 0, stream, in, nrec, nt_in,
                         dt_in, out, nt_out, dt_out, first);
    });
    return hipGetLastError();
  }
  // Row tiles per wavefront: a wavefront's time per 16 input samples is RT
  // times four products of 64 cycles plus about 140 cycles for its weights
  // (fitted to 371, 309 and 283 us for 2500 x 1200 -> 2400 with RT = 1, 2, 4;
  // RT = 8 took 331: too few wavefronts fit); the cheapest RT over the
  // wavefronts that share a SIMD (1024 of them), which takes few rows where
  // the traces leave the device idle.
  const uint32_t cols = (uint32_t)(((int64_t)nt_out + 63) / 64);
  int rt = 1;
  double best = 1e300;
  for (int t = 1; t <= 4; t *= 2) {
    const double waves = 4.0 * cols * (double)(((int64_t)nrec + 16 * t - 1) / (16 * t));
    const double cost = std::max(1.0, waves / 1024.0) * (256.0 * t + 140.0);
    if (cost < best) best = cost, rt = t;
  }
  const uint32_t row_blocks = (uint32_t)(((int64_t)nrec + 16 * rt - 1) / (16 * rt));
  const unsigned blocks = cols * std::max(1u, std::min(row_blocks, (1u << 20) / cols));
#define WFD_SINC(RT)                                                                            \
  hipLaunchKernelGGL((k_resample_sinc<RT>), dim3(blocks), dim3(256), 0, stream, in, nrec, nt_in, \
                     dt_in, out, nt_out, dt_out, cols)
  switch (rt) {
    case 1: WFD_SINC(1); break;
    case 2: WFD_SINC(2); break;
    default: WFD_SINC(4); break;
  }
#undef WFD_SINC
  return hipGetLastError();
}

}  // namespace wfd
