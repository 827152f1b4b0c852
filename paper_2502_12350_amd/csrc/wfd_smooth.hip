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

// Lines too long for a tile (over kTileBytes even at 8 lines): one thread
// marches each line in memory.
__global__ void k_tri_lines(const float *in, float *out, int axis, int n, int64_t nlines, int nx,
                            int ny, double log_a, double a) {
  const int64_t L = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (L >= nlines) return;
  int64_t base, stride;
  line_of(axis, L, nx, ny, base, stride);
  double d = 0.0;
  for (int i = 0; i < n; ++i) {
    const int64_t p = base + (int64_t)i * stride;
    const TriRow t = tri_row(i, n, log_a, a);
    d = fma(t.c, d, t.s * (double)in[p]);
    out[p] = (float)d;
  }
  double x = d;
  for (int i = n - 2; i >= 0; --i) {
    const int64_t p = base + (int64_t)i * stride;
    x = fma(tri_row(i, n, log_a, a).c, x, (double)out[p]);
    out[p] = (float)x;
  }
}

// y = B x and a per-block partial of <p, y> when p is given.
__global__ void k_bessel_apply(const float *__restrict__ x, float *__restrict__ y, int nx, int ny,
                               int nz, float cx, float cy, float cz, double *__restrict__ part) {
  __shared__ double red[256];
  const int64_t n = (int64_t)nx * ny * nz;
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int ix = (int)(i % nx), iy = (int)((i / nx) % ny), iz = (int)(i / ((int64_t)nx * ny));
    const float c = x[i];
    // zero-flux ends: a missing neighbour contributes no difference
    float dxx = 0.0f, dyy = 0.0f, dzz = 0.0f;
    if (ix > 0) dxx += x[i - 1] - c;
    if (ix < nx - 1) dxx += x[i + 1] - c;
    if (iy > 0) dyy += x[i - nx] - c;
    if (iy < ny - 1) dyy += x[i + nx] - c;
    if (iz > 0) dzz += x[i - (int64_t)nx * ny] - c;
    if (iz < nz - 1) dzz += x[i + (int64_t)nx * ny] - c;
    const float v = c - (cx * dxx + cy * dyy + cz * dzz);
    y[i] = v;
    s += (double)c * (double)v;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// x += alpha p; r -= alpha Ap; per-block partial of <r, r>.
__global__ void k_cg_update(float *__restrict__ x, float *__restrict__ r,
                            const float *__restrict__ p, const float *__restrict__ ap, int64_t n,
                            float alpha, double *__restrict__ part) {
  __shared__ double red[256];
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    x[i] += alpha * p[i];
    const float ri = r[i] - alpha * ap[i];
    r[i] = ri;
    s += (double)ri * (double)ri;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// p = r + beta p (beta = 0: p = r); optionally also x = 0 and r = g first.
__global__ void k_cg_direction(float *__restrict__ p, const float *__restrict__ r, int64_t n,
                               float beta) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = r[i] + beta * p[i];
}

__global__ void k_copy_zero(const float *__restrict__ g, float *__restrict__ r,
                            float *__restrict__ x, int64_t n, double *__restrict__ part) {
  __shared__ double red[256];
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float v = g[i];
    r[i] = v;
    x[i] = 0.0f;
    s += (double)v * (double)v;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

}  // namespace

hipError_t launch_tri_lines(const float *in, float *out, int axis, int n, int64_t nlines, int nx,
                            int ny, double h_over_l, hipStream_t stream) {
  const double a = std::exp(-h_over_l);
  // As many lines per block, 64 at most, as fit the LDS tile; fewer where
  // that leaves compute units without a block (200 x 200 x 160, three axes: 78
  // us with at least one block a unit, 83 with two, 95 with four).
  const int pad = n | 1;  // odd: a wavefront's x lines start in different banks
  auto bytes = [&](int nl) {
    return (size_t)n * sizeof(TriRow) + (size_t)nl * (axis == 0 ? pad : n) * sizeof(float);
  };
  int nl = 64;
  while (nl > 8 && (bytes(nl) > kTileBytes || nlines < (int64_t)nl * 256)) nl /= 2;
  if (bytes(nl) > kTileBytes) {
    hipLaunchKernelGGL(k_tri_lines, dim3((unsigned)((nlines + 255) / 256)), dim3(256), 0, stream,
                       in, out, axis, n, nlines, nx, ny, -h_over_l, a);
    return hipGetLastError();
  }
  const dim3 grid((unsigned)((nlines + nl - 1) / nl));
  if (axis == 0)
    hipLaunchKernelGGL(k_tri_tile<true>, grid, dim3(256), bytes(nl), stream, in, out, n, nlines,
                       nx, ny, axis, nl, pad, -h_over_l, a);
  else
    hipLaunchKernelGGL(k_tri_tile<false>, grid, dim3(256), bytes(nl), stream, in, out, n, nlines,
                       nx, ny, axis, nl, pad, -h_over_l, a);
  return hipGetLastError();
}

hipError_t launch_bessel_apply(const float *x, float *y, int nx, int ny, int nz, float cx,
                               float cy, float cz, double *part, int npart, hipStream_t stream) {
  hipLaunchKernelGGL(k_bessel_apply, dim3(npart), dim3(256), 0, stream, x, y, nx, ny, nz, cx, cy,
                     cz, part);
  return hipGetLastError();
}

hipError_t launch_cg_update(float *x, float *r, const float *p, const float *ap, int64_t n,
                            float alpha, double *part, int npart, hipStream_t stream) {
  hipLaunchKernelGGL(k_cg_update, dim3(npart), dim3(256), 0, stream, x, r, p, ap, n, alpha, part);
  return hipGetLastError();
}

hipError_t launch_cg_direction(float *p, const float *r, int64_t n, float beta, int npart,
                               hipStream_t stream) {
  hipLaunchKernelGGL(k_cg_direction, dim3(npart), dim3(256), 0, stream, p, r, n, beta);
  return hipGetLastError();
}

hipError_t launch_cg_start(const float *g, float *r, float *x, int64_t n, double *part, int npart,
                           hipStream_t stream) {
  hipLaunchKernelGGL(k_copy_zero, dim3(npart), dim3(256), 0, stream, g, r, x, n, part);
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

// A block takes 256 output samples of every gridDim.x / nb th trace.
__global__ void __launch_bounds__(256)
    k_resample_nearest(const float *__restrict__ in, int nrec, int nt_in, double dt_in,
                       float *__restrict__ out, int nt_out, double dt_out, uint32_t nb) {
  const uint32_t r0 = blockIdx.x / nb, b = blockIdx.x - r0 * nb, step = gridDim.x / nb;
  const int64_t m = (int64_t)b * 256 + threadIdx.x;
  if (m >= nt_out) return;
  const double a = sample_pos((int)m, dt_in, dt_out);
  int n = (int)floor(a + 1.0 + 0.5) - 1;
  n = n < 0 ? 0 : (n > nt_in - 1 ? nt_in - 1 : n);
  for (int64_t r = r0; r < nrec; r += step) out[r * nt_out + m] = in[r * nt_in + n];
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
  const double scale = sin(M_PI * a) / M_PI;
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
    const uint32_t nb = (uint32_t)(((int64_t)nt_out + 255) / 256);
    const uint32_t rows = std::max(1u, std::min((uint32_t)nrec, (1u << 20) / nb));
    hipLaunchKernelGGL(k_resample_nearest, dim3(rows * nb), dim3(256), 0, stream, in, nrec, nt_in,
                       dt_in, out, nt_out, dt_out, nb);
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
