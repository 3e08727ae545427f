// soma_sq.hpp -- structure factor of the composition field (Sec. 5.6):
// S(q) = N^2 rho0 / (4 V) |F[phi_A - phi_B](q)|^2 with F the Fourier
// transform on the grid, F = dL^3 sum_c psi(c) exp(-i q.r_c), on the
// reciprocal lattice q = 2 pi (mx/Lx, my/Ly, mz/Lz).  With
// phi_t(c) = n_t(c)/(rho0 dL^3) this is S(q) = N^2 |G(q)|^2 / (4 n_beads),
// G the discrete transform of the count difference n_A - n_B.
//
// The 3-D transform is three passes of 1-D transforms in FP64 (x, then y, then
// z).  The input is real, so only the wave numbers kx <= nx/2 are carried; the
// others are complex conjugates at -q.  A line whose twiddles and two buffers
// fit into LDS is transformed there by mixed-radix steps (sq_fft_kernel); grids
// with a longer axis take direct sums over each line (sq_dft_*_kernel).
#pragma once

#include "soma_device.hpp"

namespace soma {

struct SqArgs {
  const void *counts;
  int count64;
  uint32_t nx, ny, nz;
  double2 *a, *b;             // work planes, n_cells complex each
  const double2 *tw[3];       // twiddles exp(-2 pi i k / n) per axis, k < n
};

// tw[k] = exp(-2 pi i k / n) for k < n.
__global__ __launch_bounds__(256) void sq_twiddle_kernel(double2 *tw, uint32_t n) {
  const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  double s, c;
  sincospi(2.0 * (double)k / (double)n, &s, &c);
  tw[k] = make_double2(c, -s);
}

__device__ __forceinline__ double count_diff(const void *counts, int count64, uint64_t c) {
  if (count64) {
    const unsigned long long w = reinterpret_cast<const unsigned long long *>(counts)[c];
    return (double)(uint32_t)w - (double)(uint32_t)(w >> 32);
  }
  const uint32_t w = reinterpret_cast<const uint32_t *>(counts)[c];
  return (double)(w & 0xFFFFu) - (double)(w >> 16);
}

// Stage 1: a[z][y][k] = sum_x psi(z,y,x) e^{-2 pi i k x / nx}, psi = n_A - n_B.
__global__ __launch_bounds__(256) void sq_dft_x_kernel(const SqArgs a) {
  const uint64_t n = (uint64_t)a.nx * a.ny * a.nz;
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t k = (uint32_t)(i % a.nx);
  const uint64_t row = i - k;
  const double2 *tw = a.tw[0];
  double re = 0.0, im = 0.0;
  uint32_t ph = 0;  // k * x mod nx, advanced by k per step
  for (uint32_t x = 0; x < a.nx; ++x) {
    const double psi = count_diff(a.counts, a.count64, row + x);
    const double2 t = tw[ph];
    re = fma(psi, t.x, re);
    im = fma(psi, t.y, im);
    ph += k;
    if (ph >= a.nx) ph -= a.nx;
  }
  a.a[i] = make_double2(re, im);
}

// Stages 2 and 3: the transform along y (axis 1, stride nx) or z (axis 2,
// stride nx*ny) of `in` into `out`.
__global__ __launch_bounds__(256) void sq_dft_axis_kernel(const double2 *in, double2 *out,
                                                          const double2 *tw, uint32_t nx,
                                                          uint32_t ny, uint32_t nz, int axis) {
  const uint64_t n = (uint64_t)nx * ny * nz;
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t y = (uint32_t)((i / nx) % ny);
  const uint32_t z = (uint32_t)(i / ((uint64_t)nx * ny));
  const uint32_t len = axis == 1 ? ny : nz;
  const uint32_t k = axis == 1 ? y : z;
  const uint64_t stride = axis == 1 ? (uint64_t)nx : (uint64_t)nx * ny;
  const uint64_t base = i - (uint64_t)k * stride;
  double re = 0.0, im = 0.0;
  uint32_t ph = 0;
  for (uint32_t j = 0; j < len; ++j) {
    const double2 v = in[base + (uint64_t)j * stride];
    const double2 t = tw[ph];
    re = fma(v.x, t.x, fma(-v.y, t.y, re));
    im = fma(v.x, t.y, fma(v.y, t.x, im));
    ph += k;
    if (ph >= len) ph -= len;
  }
  out[i] = make_double2(re, im);
}

// S(q) = scale |G(q)|^2.
__global__ __launch_bounds__(256) void sq_power_kernel(const double2 *g, double *sq, uint64_t n,
                                                       double scale) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double2 v = g[i];
  sq[i] = scale * (v.x * v.x + v.y * v.y);
}

// ---------------------------------------------------------------------------
// Mixed-radix passes.  A block takes T lines into LDS, transforms them in
// self-sorting steps between two LDS buffers and writes them back, so each
// pass reads and writes the half spectrum once; the last pass writes S(q)
// itself.  A step of radix R after l = product of the earlier radices:
//   v_q = x[i + q n/R] w_{lR}^{q k},  k = i mod l,  y[(i - k) R + k + q l] = DFT_R(v)_q.
// Cost per element: the sum of the radices instead of n.  96^3 cells, a whole
// call: 29.8 us (three launches of 13, 12 and 9 us on 7 MB each way), where direct
// sums over every line took 258 us.
// ---------------------------------------------------------------------------
constexpr uint32_t kSqThreads = 256u, kSqMaxSteps = 12u;
constexpr uint32_t kSqLdsBytes = 64u << 10;

// Longest line of the LDS passes: two buffers and the twiddles of one line.
constexpr uint32_t kSqMaxLine = kSqLdsBytes / (3u * 16u);

struct SqPass {
  uint32_t n, n_lines;          // line length, number of lines
  uint32_t t, t_shift;          // lines per block (a power of two), its logarithm
  uint32_t nx, ny, nz, hx;      // hx = nx/2 + 1
  uint32_t n_steps;
  uint16_t radix[kSqMaxSteps];
  const void *counts;           // pass 0
  int count64;
  double2 *a;                   // half spectrum [nz][ny][hx]
  double2 *tw_y, *tw_z;         // tables written by pass 0, read by passes 1 and 2
  double *sq;                   // pass 2
  double scale;
};

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmuli(double2 a) { return make_double2(a.y, -a.x); }   // times -i

__device__ __forceinline__ void dft4(double2 &a, double2 &b, double2 &c, double2 &d) {
  const double2 p = cadd(a, c), q = csub(a, c), r = cadd(b, d), s = cmuli(csub(b, d));
  a = cadd(p, r);
  b = cadd(q, s);
  c = csub(p, r);
  d = csub(q, s);
}

// DFT of R values in registers; w[m] = exp(-2 pi i m n_r / n), n_r = n/R apart in `tw`.
template <uint32_t R>
__device__ __forceinline__ void dft_small(double2 (&v)[R], const double2 *tw, uint32_t n_r) {
  if constexpr (R == 2u) {
    const double2 t = v[1];
    v[1] = csub(v[0], t);
    v[0] = cadd(v[0], t);
  } else if constexpr (R == 4u) {
    dft4(v[0], v[1], v[2], v[3]);
  } else if constexpr (R == 8u) {
    constexpr double h = 0.70710678118654752440;
    dft4(v[0], v[2], v[4], v[6]);
    dft4(v[1], v[3], v[5], v[7]);
    const double2 o1 = make_double2(h * (v[3].x + v[3].y), h * (v[3].y - v[3].x));
    const double2 o2 = cmuli(v[5]);
    const double2 o3 = make_double2(h * (v[7].y - v[7].x), -h * (v[7].x + v[7].y));
    const double2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6], o0 = v[1];
    v[0] = cadd(e0, o0); v[4] = csub(e0, o0);
    v[1] = cadd(e1, o1); v[5] = csub(e1, o1);
    v[2] = cadd(e2, o2); v[6] = csub(e2, o2);
    v[3] = cadd(e3, o3); v[7] = csub(e3, o3);
  } else {
    double2 w[R], o[R];
#pragma unroll
    for (uint32_t m = 1; m < R; ++m) w[m] = tw[m * n_r];
#pragma unroll
    for (uint32_t q = 0; q < R; ++q) {
      o[q] = v[0];
#pragma unroll
      for (uint32_t s = 1; s < R; ++s) {
        const uint32_t m = (s * q) % R;
        if (m == 0u) o[q] = cadd(o[q], v[s]);
        else {
          o[q].x = fma(v[s].x, w[m].x, fma(-v[s].y, w[m].y, o[q].x));
          o[q].y = fma(v[s].x, w[m].y, fma(v[s].y, w[m].x, o[q].y));
        }
      }
    }
#pragma unroll
    for (uint32_t q = 0; q < R; ++q) v[q] = o[q];
  }
}

// Position of element e of line c: line-major for the x pass (its lines are
// contiguous in memory), element-major otherwise (neighbouring lines are).
template <int PASS>
__device__ __forceinline__ uint32_t sq_at(const SqPass &a, uint32_t e, uint32_t c) {
  return PASS == 0 ? c * a.n + e : (e << a.t_shift) + c;
}

template <int PASS>
__device__ __forceinline__ void sq_split(const SqPass &a, uint32_t t, uint32_t per_line, uint32_t &i,
                                         uint32_t &c) {
  if (PASS == 0) {
    c = t / per_line;
    i = t - c * per_line;
  } else {
    c = t & (a.t - 1u);
    i = t >> a.t_shift;
  }
}

template <int PASS, uint32_t R>
__device__ __forceinline__ void sq_step(const SqPass &a, const double2 *x, double2 *y,
                                        const double2 *tw, uint32_t l) {
  const uint32_t n_r = a.n / R, step = n_r / l;
  for (uint32_t t = threadIdx.x; t < (n_r << a.t_shift); t += kSqThreads) {
    uint32_t i, c;
    sq_split<PASS>(a, t, n_r, i, c);
    const uint32_t k = l == 1u ? 0u : i % l;
    double2 v[R];
#pragma unroll
    for (uint32_t q = 0; q < R; ++q) {
      v[q] = x[sq_at<PASS>(a, i + q * n_r, c)];
      if (q > 0u && l > 1u) v[q] = cmul(v[q], tw[q * k * step]);
    }
    dft_small<R>(v, tw, n_r);
    const uint32_t j = (i - k) * R + k;
#pragma unroll
    for (uint32_t q = 0; q < R; ++q) y[sq_at<PASS>(a, j + q * l, c)] = v[q];
  }
}

// A step of any other radix r: one output per thread, a direct sum of r terms.
template <int PASS>
__device__ __forceinline__ void sq_step_any(const SqPass &a, const double2 *x, double2 *y,
                                            const double2 *tw, uint32_t l, uint32_t r) {
  const uint32_t n_r = a.n / r, m = l * r, step = a.n / m;
  for (uint32_t t = threadIdx.x; t < (a.n << a.t_shift); t += kSqThreads) {
    uint32_t o, c;
    sq_split<PASS>(a, t, a.n, o, c);
    const uint32_t q = o / n_r, i = o - q * n_r, k = i % l;
    const uint32_t adv = k + l * q;   // phase per term, below m
    double re = 0.0, im = 0.0;
    uint32_t ph = 0u;
    for (uint32_t s = 0; s < r; ++s) {
      const double2 v = x[sq_at<PASS>(a, i + s * n_r, c)], w = tw[ph * step];
      re = fma(v.x, w.x, fma(-v.y, w.y, re));
      im = fma(v.x, w.y, fma(v.y, w.x, im));
      ph += adv;
      if (ph >= m) ph -= m;
    }
    y[sq_at<PASS>(a, (i - k) * r + k + q * l, c)] = make_double2(re, im);
  }
}

__device__ __forceinline__ double2 sq_twiddle(uint32_t k, uint32_t n) {
  double s, c;
  sincospi(2.0 * (double)k / (double)n, &s, &c);
  return make_double2(c, -s);
}

// PASS 0: rows of n_A - n_B along x to the half spectrum; 1: along y in place;
// 2: along z to S(q).  Launched with ceil(n_lines / t) blocks.
template <int PASS>
__global__ __launch_bounds__(kSqThreads) void sq_fft_kernel(const SqPass a) {
  extern __shared__ double2 s_sq[];
  double2 *tw = s_sq, *x = s_sq + a.n, *y = x + (a.n << a.t_shift);
  const uint32_t tid = threadIdx.x, l0 = blockIdx.x << a.t_shift;
  const uint32_t n_here = min(a.t, a.n_lines - l0);
  for (uint32_t k = tid; k < a.n; k += kSqThreads)
    tw[k] = PASS == 0 ? sq_twiddle(k, a.n) : (PASS == 1 ? a.tw_y[k] : a.tw_z[k]);
  if (PASS == 0) {   // the tables of the two passes that follow, one entry per thread
    const uint32_t g = blockIdx.x * kSqThreads + tid, stride = gridDim.x * kSqThreads;
    for (uint32_t k = g; k < a.ny + a.nz; k += stride) {
      if (k < a.ny) a.tw_y[k] = sq_twiddle(k, a.ny);
      else a.tw_z[k - a.ny] = sq_twiddle(k - a.ny, a.nz);
    }
    const uint64_t base = (uint64_t)l0 * a.n;
    for (uint32_t t = tid; t < n_here * a.n; t += kSqThreads)
      x[t] = make_double2(count_diff(a.counts, a.count64, base + t), 0.0);
    for (uint32_t t = n_here * a.n + tid; t < (a.n << a.t_shift); t += kSqThreads)
      x[t] = make_double2(0.0, 0.0);
  } else {
    const uint32_t c = tid & (a.t - 1u);   // kSqThreads is a multiple of t
    const uint32_t line = l0 + min(c, n_here - 1u);
    const uint64_t plane = (uint64_t)a.ny * a.hx;
    const double2 *src = a.a + (PASS == 1 ? (line / a.hx) * plane + line % a.hx : line);
    const uint64_t stride = PASS == 1 ? a.hx : plane;
    for (uint32_t e = tid >> a.t_shift; e < a.n; e += kSqThreads >> a.t_shift)
      x[(e << a.t_shift) + c] = src[e * stride];
  }
  __syncthreads();
  uint32_t l = 1u;
  for (uint32_t s = 0; s < a.n_steps; ++s) {
    const uint32_t r = a.radix[s];
    switch (r) {
      case 2: sq_step<PASS, 2>(a, x, y, tw, l); break;
      case 3: sq_step<PASS, 3>(a, x, y, tw, l); break;
      case 4: sq_step<PASS, 4>(a, x, y, tw, l); break;
      case 5: sq_step<PASS, 5>(a, x, y, tw, l); break;
      case 8: sq_step<PASS, 8>(a, x, y, tw, l); break;
      default: sq_step_any<PASS>(a, x, y, tw, l, r);
    }
    __syncthreads();
    double2 *const swap = x;
    x = y;
    y = swap;
    l *= r;
  }
  if (PASS == 0) {
    const uint64_t base = (uint64_t)l0 * a.hx;
    for (uint32_t t = tid; t < n_here * a.hx; t += kSqThreads) {
      const uint32_t c = t / a.hx;
      a.a[base + t] = x[c * a.n + (t - c * a.hx)];
    }
    return;
  }
  const uint32_t c = tid & (a.t - 1u);
  if (c >= n_here) return;
  const uint32_t line = l0 + c;
  const uint64_t plane = (uint64_t)a.ny * a.hx;
  if (PASS == 1) {
    double2 *dst = a.a + (line / a.hx) * plane + line % a.hx;
    for (uint32_t e = tid >> a.t_shift; e < a.n; e += kSqThreads >> a.t_shift)
      dst[(uint64_t)e * a.hx] = x[(e << a.t_shift) + c];
    return;
  }
  const uint32_t ky = line / a.hx, kx = line - ky * a.hx;
  const uint32_t my = ky == 0u ? 0u : a.ny - ky, mx = a.nx - kx;   // of -q (kx > 0)
  const bool mirror = kx > 0u && 2u * kx != a.nx;
  for (uint32_t kz = tid >> a.t_shift; kz < a.n; kz += kSqThreads >> a.t_shift) {
    const double2 v = x[(kz << a.t_shift) + c];
    const double p = a.scale * (v.x * v.x + v.y * v.y);
    a.sq[((uint64_t)kz * a.ny + ky) * a.nx + kx] = p;
    const uint32_t mz = kz == 0u ? 0u : a.nz - kz;
    if (mirror) a.sq[((uint64_t)mz * a.ny + my) * a.nx + mx] = p;
  }
}

}  // namespace soma
