// gfx950 kernels of the particle-mesh field (Sec. 3.3) and of its
// interpolation scheme (App. B), and a trace kernel that integrates rays
// through that field.
//
// Field build for an isolated lens (the zero-padded case of Sec. 3.3):
//   * Cloud-in-Cell deposit of the particle masses onto the n^3 nodes (FP64
//     atomics; mass whose cloud falls outside the nodes is dropped);
//   * real 3-D transforms of the masses zero-padded to (2n)^3, lines in LDS;
//   * product with the transforms of the Plummer kernels of eq. psi and
//     eq. derivs on the padded grid, which makes the cyclic convolution the exact
//     linear one;  phi = -(G/c^2) sum M (d^2 + eps^2)^(-1/2) and
//     dphi/dx = (G/c^2) sum M d_x (d^2 + eps^2)^(-3/2) at every node;
//   * natural cubic-spline second derivatives of each of the four grids along
//     the line of sight x^3 (computed once per grid, App. B).
// Periodic boxes: the deposit wraps, the node masses' transform is multiplied
// by the continuum Green's function of Poisson's equation (and i k_j for the
// derivatives), and the x^3 spline is the periodic one.
// Evaluation at a point (App. B, n_int nodes on each side): (2 n_int)^2 spline
// evaluations along x^3, 2 n_int local natural splines along x^1, one local
// natural spline along x^2; zero outside the node range.
//
// HBM layout of the field: fields[8][n^3], grid q in [0, 4) = phi, dphi/dx^1,
// dphi/dx^2, dphi/dx^3 and q + 4 = its x^3 spline second derivatives; node
// (i, j, k) at (i n + j) n + k, so every x^3 line is contiguous.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "rt_direct.h"
#include "rt_geodesic.h"
#include "rt_internal.h"

namespace rt {

namespace {


// ------------------------------------------------------------------ build
__global__ void pm_clear_kernel(double* buf, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) buf[i] = 0.0;
}

__global__ void pm_twiddle_kernel(double2* tw, int M) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= M / 2) return;
  double s, c;
  sincospi(2.0 * (double)k / (double)M, &s, &c);
  tw[k] = make_double2(c, -s);   // exp(-2 pi i k / M)
}

// Adds one particle's cloud: add(node, mass) for each of its nodes.
template <class Add>
__device__ __forceinline__ void cic_cloud(const double* __restrict__ xyzm, int64_t np, int64_t p, double ox, double oy, double oz,
                                          double h, int n, int periodic, Add&& add) {
  const double u[3] = {(xyzm[p] - ox) / h, (xyzm[np + p] - oy) / h, (xyzm[2 * np + p] - oz) / h};
  const double m = xyzm[3 * np + p];
  int64_t i0[3];
  double f[3];
  for (int d = 0; d < 3; ++d) {
    const double fl = floor(u[d]);
    i0[d] = (int64_t)fl;
    f[d] = u[d] - fl;
  }
#pragma unroll
  for (int corner = 0; corner < 8; ++corner) {
    const int a = corner >> 2, b = (corner >> 1) & 1, c = corner & 1;
    int64_t i = i0[0] + a, j = i0[1] + b, k = i0[2] + c;
    if (periodic) {
      i = ((i % n) + n) % n;
      j = ((j % n) + n) % n;
      k = ((k % n) + n) % n;
    } else if (i < 0 || i >= n || j < 0 || j >= n || k < 0 || k >= n) {
      continue;
    }
    const double w = (a ? f[0] : 1.0 - f[0]) * (b ? f[1] : 1.0 - f[1]) * (c ? f[2] : 1.0 - f[2]);
    add((i * n + j) * n + k, m * w);
  }
}

__global__ void pm_cic_kernel(const double* __restrict__ xyzm, int64_t np, double ox, double oy, double oz, double h,
                              int n, int periodic, double* rho) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= np) return;
  cic_cloud(xyzm, np, p, ox, oy, oz, h, n, periodic, [&](int64_t node, double m) { atomicAdd(&rho[node], m); });
}

// Grids of at most kCicSmall nodes a side, whose few cache lines of masses every particle's eight additions would meet
// at: each workgroup adds its particles up in LDS first (10^5 particles, 4^3 nodes, whole build: 868 -> 80 us, 442
// when the masses lay 16 B apart).
constexpr int kCicSmall = 8, kCicThreads = 256;
__global__ __launch_bounds__(kCicThreads) void pm_cic_small_kernel(const double* __restrict__ xyzm, int64_t np, double ox,
                                                                   double oy, double oz, double h, int n, int periodic,
                                                                   double* rho) {
  __shared__ double sum[kCicSmall * kCicSmall * kCicSmall];
  for (int i = threadIdx.x; i < n * n * n; i += kCicThreads) sum[i] = 0.0;
  __syncthreads();
  for (int64_t p = (int64_t)blockIdx.x * kCicThreads + threadIdx.x; p < np; p += (int64_t)gridDim.x * kCicThreads)
    cic_cloud(xyzm, np, p, ox, oy, oz, h, n, periodic, [&](int64_t node, double m) {
      __hip_atomic_fetch_add(&sum[node], m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    });
  __syncthreads();
  for (int i = threadIdx.x; i < n * n * n; i += kCicThreads)
    if (sum[i] != 0.0) atomicAdd(&rho[i], sum[i]);
}

// ------------------------------------------------------------------ transforms
// Lines of M points (a power of two, 4 to 1024) are transformed in LDS, kFftElems points per
// workgroup, i.e. L = kFftElems / M lines side by side: point p of line l at
// (p + p / 8) L + l (the gap of one row in nine spreads the last stages' strides over the banks).
// Forward: radix-8 decimation in frequency (and a last stage of radix 4 or 2 where log2 M is no multiple of 3), natural
// order in, digit-reversed out; inverse: its mirror image, digit-reversed in, natural out, unscaled.
// So a product of transforms needs no reordering, and elsewhere the order is mended
// where points are moved to or from HBM.
//
// The masses and the results are real and the kernels are even or odd in each axis, the masses
// fill an eighth of the padded grid and an eighth of the results is kept.  So: two real lines share a
// complex one; only M / 2 + 1 points of the last axis are held; lines that are zero, or not
// wanted, are left out; transforming the first axis, multiplying and transforming back is
// one kernel; and one quarter-size transform of phi + i len d/dx gives all four kernels, which are real
// after it (P, S) and permutations of each other.
// Bound: passes through LDS and HBM, about 80 B per point of the padded grid; nine full complex transforms of the
// padded grid, one line per workgroup, moved about 1100 B a point, 16 B at a time on two axes: 110 ms for
// 256^3 nodes against 4.7 (0.4 of them the splines).  Radix 8 against radix 4, three passes through LDS for 512 points instead of
// five: the transforms of the last and middle axes 8 to 10% faster (0.51 -> 0.46 ms, 0.90 -> 0.82).
constexpr int kFftElems = 2048;
constexpr int kFftThreads = 256;
constexpr int kFftSlots = kFftElems + kFftElems / 8;

struct Fft {
  int M, logM, L, logL;
  const double2* __restrict__ tw;   // exp(-2 pi i k / M), k < M / 2
};

inline Fft make_fft(int M, const double2* tw) {
  Fft f;
  f.M = M;
  f.logM = 0;
  while ((1 << f.logM) < M) ++f.logM;
  f.L = kFftElems / M;
  f.logL = 0;
  while ((1 << f.logL) < f.L) ++f.logL;
  f.tw = tw;
  return f;
}

__device__ __forceinline__ int fft_at(const Fft& f, int p, int line) { return ((p + (p >> 3)) << f.logL) + line; }

// Where frequency k of a forward transform lies.
__device__ __forceinline__ int fft_rev(const Fft& f, int k) {
  int p = 0, rem = f.logM;
  for (; rem >= 3; k >>= 3) {
    rem -= 3;
    p += (k & 7) << rem;
  }
  return p + k;   // the digit that is left, of 4 or 2
}

// The frequency that lies at p: p's digits, most significant first, are its from the least.
__device__ __forceinline__ int fft_freq(const Fft& f, int p) {
  int k = 0, sh = 0, rem = f.logM;
  for (; rem >= 3; sh += 3) {
    rem -= 3;
    k += ((p >> rem) & 7) << sh;
  }
  return k + ((p & ((1 << rem) - 1)) << sh);
}

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// times -i (forward) or i (inverse)
template <bool INV>
__device__ __forceinline__ double2 cturn(double2 a) {
  return INV ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

// Transform of 2^LOG points in registers, natural order in and out.
template <int LOG, bool INV>
__device__ __forceinline__ void fft_points(double2* x) {
  if constexpr (LOG == 1) {
    const double2 d = csub(x[0], x[1]);
    x[0] = cadd(x[0], x[1]);
    x[1] = d;
  } else if constexpr (LOG == 2) {
    const double2 s02 = cadd(x[0], x[2]), d02 = csub(x[0], x[2]), s13 = cadd(x[1], x[3]),
                  d13 = cturn<INV>(csub(x[1], x[3]));
    x[0] = cadd(s02, s13);
    x[1] = cadd(d02, d13);
    x[2] = csub(s02, s13);
    x[3] = csub(d02, d13);
  } else {
    double2 e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
    fft_points<2, INV>(e);
    fft_points<2, INV>(o);
    constexpr double h = 0.70710678118654752440;   // (1 -+ i) / sqrt 2 and (-1 -+ i) / sqrt 2
    const double2 t1 = cturn<INV>(o[1]), t3 = cturn<INV>(o[3]);
    o[1] = make_double2(h * (o[1].x + t1.x), h * (o[1].y + t1.y));
    o[2] = cturn<INV>(o[2]);
    o[3] = make_double2(h * (t3.x - o[3].x), h * (t3.y - o[3].y));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      x[k] = cadd(e[k], o[k]);
      x[k + 4] = csub(e[k], o[k]);
    }
  }
}

// One stage: blocks of 2^s points, of which each thread takes 2^LOG at a time, 2^(s - LOG) apart.
template <int LOG, bool INV>
__device__ __forceinline__ void fft_stage(const Fft& f, double2* b, int s) {
  constexpr int R = 1 << LOG;
  const int step = s - LOG;
#pragma unroll
  for (int r = 0; r < kFftElems / R / kFftThreads; ++r) {
    const int t = threadIdx.x + r * kFftThreads, line = t & (f.L - 1), q = t >> f.logL;
    const int o = q & ((1 << step) - 1), p = ((q >> step) << s) + o;
    double2 x[R];
#pragma unroll
    for (int k = 0; k < R; ++k) x[k] = b[fft_at(f, p + (k << step), line)];
    if constexpr (LOG < 3) {   // the last one forward, the first back: neighbours, no factors
      fft_points<LOG, INV>(x);
    } else {
      double2 w[R];
      w[1] = f.tw[o << (f.logM - s)];
      if (INV) w[1].y = -w[1].y;
#pragma unroll
      for (int k = 2; k < R; ++k) w[k] = cmul(w[k / 2], w[k - k / 2]);
      if (INV) {
#pragma unroll
        for (int k = 1; k < R; ++k) x[k] = cmul(w[k], x[k]);
      }
      fft_points<LOG, INV>(x);
      if (!INV) {
#pragma unroll
        for (int k = 1; k < R; ++k) x[k] = cmul(w[k], x[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < R; ++k) b[fft_at(f, p + (k << step), line)] = x[k];
  }
  __syncthreads();
}

// All lines in place; starts and ends with the points in LDS behind a barrier.
__device__ __forceinline__ void fft_forward(const Fft& f, double2* b) {
  int s = f.logM;
  for (; s >= 3; s -= 3) fft_stage<3, false>(f, b, s);
  if (s == 2) fft_stage<2, false>(f, b, 2);
  if (s == 1) fft_stage<1, false>(f, b, 1);
}

__device__ __forceinline__ void fft_inverse(const Fft& f, double2* b) {
  int s = f.logM % 3;
  if (s == 1) fft_stage<1, true>(f, b, 1);
  if (s == 2) fft_stage<2, true>(f, b, 2);
  for (s += 3; s <= f.logM; s += 3) fft_stage<3, true>(f, b, s);
}

constexpr int kFftMine = kFftElems / kFftThreads;   // points per thread

// The workgroup's place in its grid, with neighbours on one XCD: rows of M / 2 + 1 points are no multiple of a
// 128 B line, so a line is shared by two workgroups, and by the L2s of two XCDs where consecutive ones go to
// different XCDs (the product 3.77 -> 3.35 ms, the middle axis 0.38 -> 0.27 and back 1.06 -> 0.88, 256^3 nodes).
struct FftTile {
  int x, y, z;
};
__device__ __forceinline__ FftTile fft_tile() {
  const unsigned gx = gridDim.x, gy = gridDim.y, total = gx * gy * gridDim.z;
  const unsigned id = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z), xcd = id & 7, share = total >> 3, rest = total & 7;
  const unsigned t = xcd * share + (xcd < rest ? xcd : rest) + (id >> 3);
  FftTile o;
  o.x = (int)(t % gx);
  o.y = (int)(t / gx % gy);
  o.z = (int)(t / gx / gy);
  return o;
}

// Real lines rho[line][n] (n_lines of them, zero-padded to M), two to a complex line, forward
// along the last axis: out[line][nk], nk = M / 2 + 1.
__global__ __launch_bounds__(kFftThreads) void pm_fft_real_kernel(Fft f, const double* __restrict__ rho, int n,
                                                                  int64_t n_lines, double2* out) {
  __shared__ double2 b[kFftSlots];
  const int64_t l0 = (int64_t)blockIdx.x * 2 * f.L;
#pragma unroll
  for (int r = 0; r < kFftMine; ++r) {
    const int e = threadIdx.x + r * kFftThreads, p = e & (f.M - 1), line = e >> f.logM;
    const int64_t l = l0 + 2 * line;
    double2 v = make_double2(0.0, 0.0);
    if (p < n) {
      if (l < n_lines) v.x = rho[l * n + p];
      if (l + 1 < n_lines) v.y = rho[(l + 1) * n + p];
    }
    b[fft_at(f, p, line)] = v;
  }
  __syncthreads();
  fft_forward(f, b);
  const int nk = f.M / 2 + 1;
  for (int e = threadIdx.x; e < nk * f.L; e += kFftThreads) {
    const int line = e / nk, k = e - line * nk;
    const int64_t l = l0 + 2 * line;
    const double2 z = b[fft_at(f, fft_rev(f, k), line)], y = b[fft_at(f, fft_rev(f, (f.M - k) & (f.M - 1)), line)];
    if (l < n_lines) out[l * nk + k] = make_double2(0.5 * (z.x + y.x), 0.5 * (z.y - y.y));
    if (l + 1 < n_lines) out[(l + 1) * nk + k] = make_double2(0.5 * (z.y + y.y), 0.5 * (y.x - z.x));
  }
}

// Forward along the middle axis: in [planes][n_in][nk] -> out [planes][M][nk] (in place where n_in = M).
__global__ __launch_bounds__(kFftThreads) void pm_fft_mid_kernel(Fft f, const double2* in, int n_in, int nk,
                                                                 double2* out) {
  __shared__ double2 b[kFftSlots];
  const FftTile tile = fft_tile();
  const int k0 = tile.x * f.L;
  const int64_t plane = tile.y;
#pragma unroll
  for (int r = 0; r < kFftMine; ++r) {
    const int e = threadIdx.x + r * kFftThreads, line = e & (f.L - 1), p = e >> f.logL, k = k0 + line;
    b[fft_at(f, p, line)] = p < n_in && k < nk ? in[(plane * n_in + p) * nk + k] : make_double2(0.0, 0.0);
  }
  __syncthreads();
  fft_forward(f, b);
#pragma unroll
  for (int r = 0; r < kFftMine; ++r) {
    const int e = threadIdx.x + r * kFftThreads, line = e & (f.L - 1), p = e >> f.logL, k = k0 + line;
    if (k < nk) out[(plane * f.M + p) * nk + k] = b[fft_at(f, fft_rev(f, p), line)];
  }
}

// The Plummer kernels of eq. psi and eq. derivs on one octant of displacements, value phi + i len d/dx,
// even in the last two axes: mirrored and transformed along the last one, c [i][j][k], i, j, k <= n.
// (Displacement n is met by no pair of nodes: the odd part is 0 there.)
// len, a power of two, brings d/dx to phi's size: the two share their rounding, which without it is that of
// the larger for both, i.e. depends on the unit of length (phi off by 5e-13 of its largest value at h = 1e-5, the
// derivatives by 3e-14 at h = 20).
__global__ __launch_bounds__(kFftThreads) void pm_kernel_last_kernel(Fft f, int n, double h, double eps2, double G,
                                                                     double len, double2* c) {
  __shared__ double2 b[kFftSlots];
  const int m = n + 1;
  const int64_t l0 = (int64_t)blockIdx.x * f.L, n_lines = (int64_t)m * m;
#pragma unroll
  for (int r = 0; r < kFftMine; ++r) {
    const int e = threadIdx.x + r * kFftThreads, p = e & (f.M - 1), line = e >> f.logM;
    const int64_t l = l0 + line;
    double2 v = make_double2(0.0, 0.0);
    if (l < n_lines) {
      const int i = (int)(l / m), j = (int)(l - (int64_t)i * m), k = p <= n ? p : f.M - p;
      const double dx = i * h, dy = j * h, dz = k * h;
      const double r2 = dx * dx + dy * dy + dz * dz + eps2;
      const double k1 = r2 > 0.0 ? 1.0 / sqrt(r2) : 0.0;
      v = make_double2(-G * k1, i < n ? len * (G * dx * (k1 * k1 * k1)) : 0.0);
    }
    b[fft_at(f, p, line)] = v;
  }
  __syncthreads();
  fft_forward(f, b);
  for (int e = threadIdx.x; e < m * f.L; e += kFftThreads) {
    const int line = e / m, k = e - line * m;
    if (l0 + line < n_lines) c[(l0 + line) * m + k] = b[fft_at(f, fft_rev(f, k), line)];
  }
}

// The same along the middle axis, in place.
__global__ __launch_bounds__(kFftThreads) void pm_kernel_mid_kernel(Fft f, int n, double2* c) {
  __shared__ double2 b[kFftSlots];
  const FftTile tile = fft_tile();
  const int m = n + 1, k0 = tile.x * f.L;
  const int64_t plane = tile.y;
#pragma unroll
  for (int r = 0; r < kFftMine; ++r) {
    const int e = threadIdx.x + r * kFftThreads, line = e & (f.L - 1), p = e >> f.logL, k = k0 + line;
    b[fft_at(f, p, line)] = k < m ? c[(plane * m + (p <= n ? p : f.M - p)) * m + k] : make_double2(0.0, 0.0);
  }
  __syncthreads();
  fft_forward(f, b);
#pragma unroll
  for (int r = 0; r < kFftMine; ++r) {
    const int e = threadIdx.x + r * kFftThreads, line = e & (f.L - 1), p = e >> f.logL, k = k0 + line;
    if (k < m && p <= n) c[(plane * m + p) * m + k] = b[fft_at(f, fft_rev(f, p), line)];
  }
}

// The same along the first axis, where d/dx is odd: phi + i len d/dx transforms to P + len S, P even and S
// odd, both real (the transform of d/dx is -i S).  ps [i][j][k] = (P, S); sz [j][k][i] = S(i; j, k), i.e.
// the kernel of the axis in the last place.  scale: 1 / M^3, a power of two; inv_len: 1 / len.
__global__ __launch_bounds__(kFftThreads) void pm_kernel_first_kernel(Fft f, int n, const double2* c, double scale,
                                                                      double inv_len, double2* ps, double* sz) {
  __shared__ double2 b[kFftSlots];
  const FftTile tile = fft_tile();
  const int m = n + 1, k0 = tile.x * f.L;
  const int64_t j = tile.y, mm = (int64_t)m * m;
#pragma unroll
  for (int r = 0; r < kFftMine; ++r) {
    const int e = threadIdx.x + r * kFftThreads, line = e & (f.L - 1), p = e >> f.logL, k = k0 + line;
    double2 v = make_double2(0.0, 0.0);
    if (k < m) {
      v = c[(p <= n ? p : f.M - p) * mm + j * m + k];
      if (p > n) v.y = -v.y;
    }
    b[fft_at(f, p, line)] = v;
  }
  __syncthreads();
  fft_forward(f, b);
  for (int e = threadIdx.x; e < m * f.L; e += kFftThreads) {
    const int line = e & (f.L - 1), i = e >> f.logL, k = k0 + line;
    if (k >= m) continue;
    const double a = b[fft_at(f, fft_rev(f, i), line)].x, z = b[fft_at(f, fft_rev(f, (f.M - i) & (f.M - 1)), line)].x;
    const double S = 0.5 * scale * (a - z) * inv_len;
    ps[i * mm + j * m + k] = make_double2(0.5 * scale * (a + z), S);
    sz[(j * m + k) * m + i] = S;
  }
}

// Where a product's four results go: phi and its three derivatives.
struct FourOut {
  double2* q[4];
};

// Forward along the first axis (n_in planes of the masses, [i][j][k]), times the four transforms, and back
// along that axis: out.q[i][j][k] for i < n_out.  PERIODIC: the continuum Green's function of Poisson's
// equation, phi_k = -4 pi G rho_k / k^2 (rho = mass / h^3, k = 0 removed, which also removes the mean density)
// and i k_j phi_k (whose n / 2 plane has no real part); frequencies in the FFT's order, index i means
// i / (n h) for i < n/2 and (i - n) / (n h) otherwise.
template <bool PERIODIC>
__global__ __launch_bounds__(kFftThreads, 3) void pm_product_kernel(Fft f, const double2* __restrict__ in, int n_in,
                                                                 int n_out, int nk, const double2* __restrict__ ps,
                                                                 const double* __restrict__ sz, double w, double green,
                                                                 FourOut out) {
  __shared__ double2 b[kFftSlots];
  const FftTile tile = fft_tile();
  const int M = f.M, m = M / 2 + 1, k0 = tile.x * f.L;
  const int64_t j = tile.y, mm = (int64_t)m * m, plane = (int64_t)gridDim.y * nk;
#pragma unroll
  for (int r = 0; r < kFftMine; ++r) {
    const int e = threadIdx.x + r * kFftThreads, line = e & (f.L - 1), p = e >> f.logL, k = k0 + line;
    b[fft_at(f, p, line)] = p < n_in && k < nk ? in[p * plane + j * nk + k] : make_double2(0.0, 0.0);
  }
  __syncthreads();
  fft_forward(f, b);
  double2 a[kFftMine];
#pragma unroll
  for (int r = 0; r < kFftMine; ++r) {
    const int e = threadIdx.x + r * kFftThreads;
    a[r] = b[fft_at(f, e >> f.logL, e & (f.L - 1))];
  }
  const int aj = j <= M / 2 ? (int)j : M - (int)j;
#pragma unroll 1
  for (int q = 0; q < 4; ++q) {
    int tid = threadIdx.x;
    // the addresses are formed anew for each result: kept for all four they take 100 registers, and two
    // wavefronts per SIMD instead of three (3.35 -> 2.2 ms, 256^3 nodes, with places found by shifts)
    asm("" : "+v"(tid));
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kFftMine; ++r) {
      const int e = tid + r * kFftThreads, line = e & (f.L - 1), k = k0 + line, i = fft_freq(f, e >> f.logL);
      double2 v = make_double2(0.0, 0.0);
      if (k < nk) {
        const int ai = i <= M / 2 ? i : M - i;
        if constexpr (PERIODIC) {
          const double kx = (i < M / 2 ? i : i - M) * w, ky = ((int)j < M / 2 ? (int)j : (int)j - M) * w, kz = (k < M / 2 ? k : k - M) * w;
          const double k2 = kx * kx + ky * ky + kz * kz;
          const double g = k2 > 0.0 ? green / k2 : 0.0;
          if (q == 0) {
            v = make_double2(g * a[r].x, g * a[r].y);
          } else {
            const int iq = q == 1 ? ai : (q == 2 ? aj : k);
            const double kq = (2 * iq == M) ? 0.0 : (q == 1 ? kx : (q == 2 ? ky : kz));
            v = make_double2(-kq * (g * a[r].y), kq * (g * a[r].x));
          }
        } else {
          if (q == 0) {
            const double P = ps[ai * mm + (int64_t)aj * m + k].x;
            v = make_double2(P * a[r].x, P * a[r].y);
          } else {
            double S;
            if (q == 1) S = i <= M / 2 ? ps[ai * mm + (int64_t)aj * m + k].y : -ps[ai * mm + (int64_t)aj * m + k].y;
            else if (q == 2) S = j <= M / 2 ? ps[aj * mm + (int64_t)ai * m + k].y : -ps[aj * mm + (int64_t)ai * m + k].y;
            else S = sz[ai * mm + (int64_t)aj * m + k];
            v = make_double2(S * a[r].y, -S * a[r].x);   // -i S a
          }
        }
      }
      b[fft_at(f, e >> f.logL, line)] = v;
    }
    __syncthreads();
    fft_inverse(f, b);
    double2* o = out.q[q];
#pragma unroll
    for (int r = 0; r < kFftMine; ++r) {
      const int e = tid + r * kFftThreads, line = e & (f.L - 1), p = e >> f.logL, k = k0 + line;
      if (p < n_out && k < nk) o[p * plane + j * nk + k] = b[fft_at(f, p, line)];
    }
  }
}

// Back along the middle axis, in place: [i][M][nk], of which the first n_out rows are kept.
__global__ __launch_bounds__(kFftThreads) void pm_ifft_mid_kernel(Fft f, FourOut io, int nk, int n_out) {
  __shared__ double2 b[kFftSlots];
  const FftTile tile = fft_tile();
  const int k0 = tile.x * f.L;
  double2* o = io.q[tile.z] + (int64_t)tile.y * f.M * nk;
#pragma unroll
  for (int r = 0; r < kFftMine; ++r) {
    const int e = threadIdx.x + r * kFftThreads, line = e & (f.L - 1), p = e >> f.logL, k = k0 + line;
    b[fft_at(f, fft_rev(f, p), line)] = k < nk ? o[(int64_t)p * nk + k] : make_double2(0.0, 0.0);
  }
  __syncthreads();
  fft_inverse(f, b);
#pragma unroll
  for (int r = 0; r < kFftMine; ++r) {
    const int e = threadIdx.x + r * kFftThreads, line = e & (f.L - 1), p = e >> f.logL, k = k0 + line;
    if (k < nk && p < n_out) o[(int64_t)p * nk + k] = b[fft_at(f, p, line)];
  }
}

// Back along the last axis to real values, two lines of one quantity (blockIdx.z) as one complex line (neighbours
// of one unit: they share their rounding): lines (i, j), j < n, of planes of `rows` rows, to
// fields[q][(i n + j) n + k], k < n.
__global__ __launch_bounds__(kFftThreads) void pm_ifft_real_kernel(Fft f, FourOut in, int rows, int n, int nk,
                                                                   double* fields) {
  __shared__ double2 b[kFftSlots];
  const int64_t l0 = (int64_t)blockIdx.x * 2 * f.L, n_lines = (int64_t)n * n;   // (an even number)
  const double2* __restrict__ X = in.q[blockIdx.z];
#pragma unroll
  for (int r = 0; r < kFftMine; ++r) {
    const int e = threadIdx.x + r * kFftThreads, k = e & (f.M - 1), line = e >> f.logM;
    const int64_t l = l0 + 2 * line;
    double2 v = make_double2(0.0, 0.0);
    if (l < n_lines) {
      const int64_t i = l / n, j = l - i * n;
      const int64_t at = (i * rows + j) * nk + (k < nk ? k : f.M - k);
      const double2 x = X[at], y = X[at + nk];
      v = k < nk ? make_double2(x.x - y.y, x.y + y.x) : make_double2(x.x + y.y, y.x - x.y);   // x + i y, conj x + i conj y
    }
    b[fft_at(f, fft_rev(f, k), line)] = v;
  }
  __syncthreads();
  fft_inverse(f, b);
  double* o = fields + blockIdx.z * n_lines * n;
#pragma unroll
  for (int r = 0; r < kFftMine; ++r) {
    const int e = threadIdx.x + r * kFftThreads, k = e & (f.M - 1), line = e >> f.logM;
    const int64_t l = l0 + 2 * line;
    if (l < n_lines && k < n) {
      const double2 v = b[fft_at(f, k, line)];
      o[l * n + k] = v.x;
      o[(l + 1) * n + k] = v.y;
    }
  }
}

// Spline second derivatives along each contiguous x^3 line:
//   y2[k-1] + 4 y2[k] + y2[k+1] = r[k] = 6 (y[k+1] - 2 y[k] + y[k-1]) / h^2,
// natural (y2 = 0 at both ends) or periodic (indices mod n), by elimination:
//   c[k] = w[k] (r[k] - c[k-1]),  y2[k] = c[k] - w[k] y2[k+1],
// w[k] = 1 / (4 - w[k-1]) from w[1] = 1/4 on (natural), w = 2 - sqrt 3, its limit (periodic; the cyclic
// matrix is the product of the two recursions' exactly).  Both forget a wrong start at that rate per step, 5e-19
// over kSplineRun = 32 steps, so a line is cut into chunks of eight points (of four, a line of four), one to a thread,
// which starts its recursions 32 points away: lines pass through LDS once and HBM is read and written coalesced.
// Bound: HBM and the 40 steps of each chain.  256^3 nodes: 0.41 ms (2.6 TB/s); a thread per line, two passes
// over HBM at a stride of a line with one step's loads in flight, 1.10.
constexpr int kSplineElems = 2048;
constexpr int kSplineThreads = 256;
constexpr int kSplineRun = 32;

template <bool PERIODIC, int CHUNK>
__global__ __launch_bounds__(kSplineThreads) void pm_spline_z_kernel(const double* __restrict__ F, double* F2, int n,
                                                                     double h, int64_t n_lines) {
  constexpr int kSlots = kSplineElems + kSplineElems / CHUNK;   // (a gap a chunk: chunks start on different banks)
  __shared__ double y[kSlots], cs[kSlots], ws[kSplineRun + CHUNK];
  const double limit = 0.26794919243112270647;   // 2 - sqrt 3
  if (threadIdx.x == 0) {
    double w = 0.0;
    for (int k = 0; k < kSplineRun + CHUNK; ++k) {
      ws[k] = PERIODIC || k >= kSplineRun ? limit : w;
      w = 1.0 / (4.0 - w);
    }
  }
  const int64_t lines = kSplineElems / n, first = (int64_t)blockIdx.x * lines;
  const int64_t left = (n_lines - first) * n;
  const int count = left < lines * n ? (int)left : (int)lines * n;
  for (int e = threadIdx.x; e < count; e += kSplineThreads) y[e + e / CHUNK] = F[first * n + e];
  __syncthreads();
  const double s = 6.0 / (h * h);
  for (int e0 = threadIdx.x * CHUNK; e0 < count; e0 += kSplineThreads * CHUNK) {
    const int k0 = e0 & (n - 1), l0 = e0 - k0;
    auto slot = [&](int g) { const int e = l0 + (PERIODIC ? g & (n - 1) : g); return e + e / CHUNK; };
    int g = k0 - kSplineRun;
    if (!PERIODIC && g < 0) g = 0;
    double c = 0.0, yb = y[slot(g)], ya = PERIODIC ? y[slot(g - CHUNK) + CHUNK - 1] : (g > 0 ? y[slot(g - CHUNK) + CHUNK - 1] : yb);
    for (; g <= k0; g += CHUNK) {
      const int at = slot(g), next = PERIODIC || g + CHUNK < n ? slot(g + CHUNK) : at;   // (c[n - 1] is not used)
      const double* w = ws + (PERIODIC || g > kSplineRun ? kSplineRun : g);
      const bool own = g == k0;
#pragma unroll
      for (int i = 0; i < CHUNK; ++i) {
        const double yc = i + 1 < CHUNK ? y[at + i + 1] : y[next];
        const double r = s * (yc - 2.0 * yb + ya);
        c = (r - c) * (PERIODIC ? limit : w[i]);
        if (own) cs[at + i] = c;
        ya = yb;
        yb = yc;
      }
    }
  }
  __syncthreads();
  for (int e0 = threadIdx.x * CHUNK; e0 < count; e0 += kSplineThreads * CHUNK) {
    const int k0 = e0 & (n - 1), l0 = e0 - k0;
    auto slot = [&](int g) { const int e = l0 + (PERIODIC ? g & (n - 1) : g); return e + e / CHUNK; };
    int g = k0 + kSplineRun;
    if (!PERIODIC && g > n - CHUNK) g = n - CHUNK;
    double v = 0.0;
    for (; g >= k0; g -= CHUNK) {
      const int at = slot(g);
      const double* w = ws + (PERIODIC || g > kSplineRun ? kSplineRun : g);
      const bool own = g == k0;
#pragma unroll
      for (int i = CHUNK - 1; i >= 0; --i) {
        v = cs[at + i] - (PERIODIC ? limit : w[i]) * v;
        if (!PERIODIC && ((i == 0 && g == 0) || (i == CHUNK - 1 && g == n - CHUNK))) v = 0.0;   // the ends
        if (own) y[at + i] = v;
      }
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < count; e += kSplineThreads) F2[first * n + e] = y[e + e / CHUNK];
}

template <bool PERIODIC>
hipError_t launch_spline_z(const double* F, double* F2, int n, double h, int64_t n_lines, hipStream_t s) {
  const dim3 grid((unsigned)((n_lines + kSplineElems / n - 1) / (kSplineElems / n)));
  if (n < 8)
    hipLaunchKernelGGL((pm_spline_z_kernel<PERIODIC, 4>), grid, dim3(kSplineThreads), 0, s, F, F2, n, h, n_lines);
  else
    hipLaunchKernelGGL((pm_spline_z_kernel<PERIODIC, 8>), grid, dim3(kSplineThreads), 0, s, F, F2, n, h, n_lines);
  return hipGetLastError();
}

// ------------------------------------------------------------------ App. B evaluation
// The interpolation is linear in the grid values, so each point needs only its weights: four
// along x^3 (two values and two second derivatives, shared by every node of the window), and
// 2 NI along each of x^1, x^2.  A natural spline through the m = 2 NI window nodes has second
// derivatives y2 = C v / h^2, C constant; in the segment [node kl, node kl + 1], A = node_{kl+1} - u,
// B = 1 - A, its value is  A v_kl + B v_{kl+1} + ((A^3 - A) y2_kl + (B^3 - B) y2_{kl+1}) h^2 / 6.
template <int NI>
struct SplineMatrix {
  static constexpr int m = 2 * NI;
  double c[m][m];   // C / 6: row k gives y2_k h^2 / 6
  constexpr SplineMatrix() : c{} {
    // y2[k-1] + 4 y2[k] + y2[k+1] = 6 (v[k+1] - 2 v[k] + v[k-1]) / h^2, y2 = 0 at both ends
    double cp[m] = {};
    for (int k = 1; k < m - 1; ++k) {
      cp[k] = 1.0 / (4.0 - (k > 1 ? cp[k - 1] : 0.0));
      for (int j = 0; j < m; ++j) {
        const double r = (j == k + 1 || j == k - 1) ? 1.0 : (j == k ? -2.0 : 0.0);
        c[k][j] = (r - (k > 1 ? c[k - 1][j] : 0.0)) * cp[k];
      }
    }
    for (int k = m - 3; k >= 1; --k)
      for (int j = 0; j < m; ++j) c[k][j] -= cp[k] * c[k + 1][j];
  }
};

// Weights of the 2 NI nodes node0, node0 + 1, ... at u (in node units).
template <int NI>
__device__ __forceinline__ void spline_weights(int node0, double u, double (&w)[2 * NI]) {
  constexpr int m = 2 * NI;
  constexpr SplineMatrix<NI> C{};
  int kl = (int)floor(u) - node0;
  kl = kl < 0 ? 0 : (kl > m - 2 ? m - 2 : kl);
  const double A = (double)(node0 + kl + 1) - u, B = 1.0 - A;
  const double a3 = A * A * A - A, b3 = B * B * B - B;
#pragma unroll
  for (int a = 0; a < m; ++a) w[a] = (a == kl ? A : 0.0) + (a == kl + 1 ? B : 0.0);
#pragma unroll
  for (int k = 1; k < m - 1; ++k) {
    const double p = (k == kl ? a3 : 0.0) + (k == kl + 1 ? b3 : 0.0);
#pragma unroll
    for (int a = 0; a < m; ++a) w[a] = fma(C.c[k][a], p, w[a]);
  }
}

__device__ __forceinline__ int window_start(double u, int n, int NI) {
  int k = (int)floor(u);
  k = k < 0 ? 0 : (k > n - 2 ? n - 2 : k);
  int st = k - NI + 1;
  st = st < 0 ? 0 : (st > n - 2 * NI ? n - 2 * NI : st);
  return st;
}

struct PmGrid {
  int n;
  double ox, oy, oz, h;
  int periodic;
  double ih;   // 1 / h
};

// (p - o) / h with ih = 1 / h correctly rounded: a quotient corrected by its own remainder, which for these
// magnitudes is the correctly rounded one (a node's own position gives its integer) in three operations
// instead of the eleven of a division that also scales its operands.
__device__ __forceinline__ double node_units(double p, double o, double h, double ih) {
  const double d = p - o, q = d * ih;
  return fma(fma(-q, h, d), ih, q);
}

// u of a periodic axis brought into [0, n]: fmod's value, then + n for negative ones.
__device__ __forceinline__ double into_box(double u, double dn) {
  if (!(u > -dn && u < dn)) u = fmod(u, dn);
  return u < 0.0 ? u + dn : u;
}

// What a point asks of a grid: its window (first nodes and the x^3 segment) and its weights.
template <int NI>
struct PmPoint {
  int wx, wy, kz;        // kz: segment [kz, kz + 1]; periodic nodes are taken modulo n
  double cz[4];          // of the values at kz and kz + 1, then of their second derivatives
  double x[2 * NI], y[2 * NI];

  // false: no field there (off an isolated grid's nodes, or no finite position)
  __device__ __forceinline__ bool set(const PmGrid& g, double px, double py, double pz) {
    double ux = node_units(px, g.ox, g.h, g.ih), uy = node_units(py, g.oy, g.h, g.ih), uz = node_units(pz, g.oz, g.h, g.ih);
    if (g.periodic) {
      const double dn = (double)g.n;
      ux = into_box(ux, dn);
      uy = into_box(uy, dn);
      uz = into_box(uz, dn);
      if (!(isfinite(ux) && isfinite(uy) && isfinite(uz))) return false;
      wx = (int)floor(ux) - NI + 1;
      wy = (int)floor(uy) - NI + 1;
      kz = (int)floor(uz);
    } else {
      const double top = (double)(g.n - 1);
      if (!(ux >= 0.0 && uy >= 0.0 && uz >= 0.0 && ux <= top && uy <= top && uz <= top)) return false;
      wx = window_start(ux, g.n, NI);
      wy = window_start(uy, g.n, NI);
      kz = (int)floor(uz);
      kz = kz > g.n - 2 ? g.n - 2 : kz;
    }
    const double A = (double)(kz + 1) - uz, B = 1.0 - A, h6 = g.h * g.h * (1.0 / 6.0);
    cz[0] = A;
    cz[1] = B;
    cz[2] = (A * A * A - A) * h6;
    cz[3] = (B * B * B - B) * h6;
    spline_weights<NI>(wx, ux, x);
    spline_weights<NI>(wy, uy, y);
    return true;
  }
};

// Two neighbours along x^3 in one load (8-byte aligned).
typedef double double2u __attribute__((ext_vector_type(2), aligned(8)));

// (value, next value) of node row i, j of a grid quantity at segment kz; n is a power of two.
__device__ __forceinline__ double2u load_pair(const double* __restrict__ F, int n, int periodic, int i, int j, int kz) {
  if (periodic) {
    i &= n - 1;
    j &= n - 1;
    kz &= n - 1;
  }
  const double* at = F + ((int64_t)i * n + j) * n + kz;
  if (kz + 1 < n) return *reinterpret_cast<const double2u*>(at);
  return double2u{at[0], at[1 - n]};   // the last node of a periodic line and its first
}

// One point on its own lane (arbitrary points).
template <int NI>
__device__ __forceinline__ void pm_field(const PmGrid& g, const double* __restrict__ fields, double x, double y,
                                         double z, double& phi, double& gx, double& gy, double& gz) {
  phi = gx = gy = gz = 0.0;
  PmPoint<NI> p;
  if (!p.set(g, x, y, z)) return;
  const int64_t n3 = (int64_t)g.n * g.n * g.n;
  double out[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    double s = 0.0;
#pragma unroll
    for (int b = 0; b < 2 * NI; ++b) {
      double w = 0.0;
#pragma unroll
      for (int a = 0; a < 2 * NI; ++a) {
        const double2u f = load_pair(fields + q * n3, g.n, g.periodic, p.wx + a, p.wy + b, p.kz);
        const double2u f2 = load_pair(fields + (q + 4) * n3, g.n, g.periodic, p.wx + a, p.wy + b, p.kz);
        w = fma(p.x[a], p.cz[0] * f[0] + p.cz[1] * f[1] + (p.cz[2] * f2[0] + p.cz[3] * f2[1]), w);
      }
      s = fma(p.y[b], w, s);
    }
    out[q] = s;
  }
  phi = out[0];
  gx = out[1];
  gy = out[2];
  gz = out[3];
}

// The same with the splines solved in place, for windows of six and eight nodes a side: their weights and
// loads in pairs take up to four times as long there (10^6 points of a 128^3 grid in cell order, six a side 1.5 against
// 3.2 ms, eight 1.9 against 7.3; in random order 5.0 against 6.3 and 8.5 against 12.0), where those of two and four a side
// are the faster (0.39 against 0.32, 0.89 against 0.67).
__device__ __forceinline__ double spline_eval(double yk, double yk1, double y2k, double y2k1, double A, double h) {
  const double B = 1.0 - A;
  return A * yk + B * yk1 + ((A * A * A - A) * y2k + (B * B * B - B) * y2k1) * (h * h) / 6.0;
}

// Natural spline through m = 2 NI values at unit-spaced nodes node0 + a (spacing h),
// evaluated at u (in node units).
template <int NI>
__device__ __forceinline__ double local_spline(const double (&v)[2 * NI], int node0, double u, double h) {
  constexpr int m = 2 * NI;
  double y2[m];
  y2[0] = 0.0;
  y2[m - 1] = 0.0;
  if constexpr (m >= 3) {
    const double s = 6.0 / (h * h);
    double cp[m];
    double c = 0.0, d = 0.0;
#pragma unroll
    for (int k = 1; k < m - 1; ++k) {
      c = 1.0 / (4.0 - (k > 1 ? c : 0.0));
      cp[k] = c;
      d = (s * (v[k + 1] - 2.0 * v[k] + v[k - 1]) - (k > 1 ? d : 0.0)) * c;
      y2[k] = d;
    }
#pragma unroll
    for (int k = m - 3; k >= 1; --k) y2[k] = y2[k] - cp[k] * y2[k + 1];
  }
  int kl = (int)floor(u) - node0;
  kl = kl < 0 ? 0 : (kl > m - 2 ? m - 2 : kl);
  const double A = (double)(node0 + kl + 1) - u;
  double yk = v[0], yk1 = v[1], s2k = y2[0], s2k1 = y2[1];
#pragma unroll
  for (int a = 1; a < m - 1; ++a)
    if (a == kl) {
      yk = v[a];
      yk1 = v[a + 1];
      s2k = y2[a];
      s2k1 = y2[a + 1];
    }
  return spline_eval(yk, yk1, s2k, s2k1, A, h);
}

__device__ __forceinline__ int wrap(int i, int n) { return ((i % n) + n) % n; }

// App. B on a periodic grid: the point is brought into the box (fmod, then + n
// for negative values), the x^3 segment and the x^1, x^2 windows are taken
// modulo n; the local splines see the unwrapped window nodes.
template <int NI>
__device__ __forceinline__ void pm_splines_periodic(const PmGrid& g, const double* __restrict__ fields, double x, double y, double z,
                                  double& phi, double& gx, double& gy, double& gz) {
  const int n = g.n;
  const double dn = (double)n;
  double ux = fmod((x - g.ox) / g.h, dn), uy = fmod((y - g.oy) / g.h, dn), uz = fmod((z - g.oz) / g.h, dn);
  phi = gx = gy = gz = 0.0;
  if (!(isfinite(ux) && isfinite(uy) && isfinite(uz))) return;
  if (ux < 0.0) ux += dn;
  if (uy < 0.0) uy += dn;
  if (uz < 0.0) uz += dn;
  const int fx = (int)floor(ux), fy = (int)floor(uy), fz = (int)floor(uz);
  const int wx = fx - NI + 1, wy = fy - NI + 1;
  const int kz0 = wrap(fz, n), kz1 = wrap(fz + 1, n);
  const double Az = (double)(fz + 1) - uz;
  const int64_t n3 = (int64_t)n * n * n;
  double out[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double* F = fields + q * n3;
    const double* F2 = fields + (q + 4) * n3;
    double w[2 * NI];
#pragma unroll
    for (int b = 0; b < 2 * NI; ++b) {
      const int j = wrap(wy + b, n);
      double v[2 * NI];
#pragma unroll
      for (int a = 0; a < 2 * NI; ++a) {
        const int64_t row = ((int64_t)wrap(wx + a, n) * n + j) * n;
        v[a] = spline_eval(F[row + kz0], F[row + kz1], F2[row + kz0], F2[row + kz1], Az, g.h);
      }
      w[b] = local_spline<NI>(v, wx, ux, g.h);
    }
    out[q] = local_spline<NI>(w, wy, uy, g.h);
  }
  phi = out[0];
  gx = out[1];
  gy = out[2];
  gz = out[3];
}

// The four grid quantities at (x, y, z): phi and its gradient.
template <int NI>
__device__ __forceinline__ void pm_splines(const PmGrid& g, const double* __restrict__ fields, double x, double y, double z, double& phi,
                         double& gx, double& gy, double& gz) {
  if (g.periodic) {
    pm_splines_periodic<NI>(g, fields, x, y, z, phi, gx, gy, gz);
    return;
  }
  const int n = g.n;
  const double ux = (x - g.ox) / g.h, uy = (y - g.oy) / g.h, uz = (z - g.oz) / g.h;
  phi = gx = gy = gz = 0.0;
  if (!(ux >= 0.0 && uy >= 0.0 && uz >= 0.0 && ux <= n - 1 && uy <= n - 1 && uz <= n - 1)) return;
  const int wx = window_start(ux, n, NI), wy = window_start(uy, n, NI);
  int kz = (int)floor(uz);
  kz = kz > n - 2 ? n - 2 : kz;
  const double Az = (double)(kz + 1) - uz;
  const int64_t n3 = (int64_t)n * n * n;
  double out[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double* F = fields + q * n3;
    const double* F2 = fields + (q + 4) * n3;
    double w[2 * NI];
#pragma unroll
    for (int b = 0; b < 2 * NI; ++b) {
      double v[2 * NI];
#pragma unroll
      for (int a = 0; a < 2 * NI; ++a) {
        const int64_t at = ((int64_t)(wx + a) * n + (wy + b)) * n + kz;
        v[a] = spline_eval(F[at], F[at + 1], F2[at], F2[at + 1], Az, g.h);
      }
      w[b] = local_spline<NI>(v, wx, ux, g.h);
    }
    out[q] = local_spline<NI>(w, wy, uy, g.h);
  }
  phi = out[0];
  gx = out[1];
  gy = out[2];
  gz = out[3];
}

// A node row's value at the point's x^3: two values and two second derivatives.  (Explicit, so that every way to sum a
// window gives the same bits.)
__device__ __forceinline__ double along_z(const double (&c)[4], double f0, double f1, double g0, double g1) {
  return fma(c[0], f0, fma(c[1], f1, fma(c[2], g0, c[3] * g1)));
}

// A ray on its own lane: its nodes, loaded by itself, ROWS rows of the window (along x^2, of one quantity after the
// other: the eight grids lie a power of two apart, so that their lines share the sets of a cache) in flight at a
// time.  PAIR: the two nodes of the x^3 segment are neighbours, which makes one load of them (false where some lane's
// segment wraps round a periodic line).  With a branch at every pair for the one that wraps, each load waited for the
// one before.
template <int NI, int ROWS, bool PAIR>
__device__ __forceinline__ void pm_gather(const PmPoint<NI>& p, int n, int periodic, const double* __restrict__ fields,
                                          double (&out)[4]) {
  constexpr int m = 2 * NI;
  static_assert(4 * m % ROWS == 0, "whole batches");
  const int64_t n3 = (int64_t)n * n * n;
  const int wrap = periodic ? n - 1 : -1;
  const int k0 = p.kz & wrap, next = PAIR ? 1 : ((p.kz + 1) & wrap) - k0;
  // where a row starts: the parts of its two indices (n <= 512: below 2^27)
  unsigned at_x[m], at_y[m];
#pragma unroll
  for (int a = 0; a < m; ++a) {
    at_x[a] = (unsigned)((p.wx + a) & wrap) * (unsigned)(n * n) + (unsigned)k0;
    at_y[a] = (unsigned)((p.wy + a) & wrap) * (unsigned)n;
  }
  // `count` rows (quantity, index along x^1) from the quantity at `first` on
  auto rows = [&](const double* first, int count, auto& sum) {
#pragma unroll
    for (int r0 = 0; r0 < count; r0 += ROWS) {
      double v[ROWS][m][4];
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        const int q = (r0 + r) / m, a = (r0 + r) % m;
#pragma unroll
        for (int b = 0; b < m; ++b) {
          const double *f = first + q * n3 + (at_x[a] + at_y[b]), *f2 = f + 4 * n3;
          v[r][b][0] = f[0];
          v[r][b][1] = f[next];
          v[r][b][2] = f2[0];
          v[r][b][3] = f2[next];
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        const int q = (r0 + r) / m, a = (r0 + r) % m;
        double w = 0.0;
#pragma unroll
        for (int b = 0; b < m; ++b) w = fma(p.y[b], along_z(p.cz, v[r][b][0], v[r][b][1], v[r][b][2], v[r][b][3]), w);
        sum[q] = fma(p.x[a], w, sum[q]);
      }
    }
  };
#pragma unroll
  for (int q = 0; q < 4; ++q) out[q] = 0.0;
  if constexpr (NI < 4) {
    rows(fields, 4 * m, out);
  } else {   // (unrolled, the quantities' addresses are all kept, and spilled)
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
      double s[1] = {0.0};
      rows(fields + q * n3, m, s);
#pragma unroll
      for (int t = 0; t < 4; ++t) out[t] = q == t ? s[0] : out[t];
    }
  }
}

// The same for the lanes with a point of a wavefront all of whose lanes call it.
template <int NI, int ROWS>
__device__ __forceinline__ void pm_gather_lanes(bool want, const PmPoint<NI>& p, int n, int periodic,
                                                const double* __restrict__ fields, double (&out)[4]) {
  const bool pair = !periodic || (p.kz & (n - 1)) + 1 < n;
  if (__all(!want || pair)) {
    if (want) pm_gather<NI, ROWS, true>(p, n, periodic, fields, out);
  } else if (want) {
    pm_gather<NI, ROWS, false>(p, n, periodic, fields, out);
  }
}

// The rays of a wavefront (seven bundles, lane 9 b + k = ray k of bundle b; lane 63 idle).  The
// nine rays of a bundle lie parsecs apart and cells are kiloparsecs wide, so they nearly always
// ask for the same window: its nodes (four values each) are fetched once per bundle, a ninth by
// each lane, into LDS, and stay there until a ray asks for another window or segment.  SAMEZ: the rays
// share x^3 (the trace in z), so the m^2 values along x^3 of each quantity (m = 2 NI) are formed once
// per bundle too.  A bundle that straddles cells takes one round per window.
// Up to NI = 3 the four quantities of a window are kept (4.6 KB a bundle); for NI = 4 that would
// leave half of the SIMDs without a wavefront, and the quantities pass one at a time, unkept.
// Bound: issue and latency of FP64 operations at one to two wavefronts per SIMD.  One ray per lane
// with its own loads fetched the same lines at every stage (about 130 MB a stage for a band of 7168
// bundles, 16 B used of each 128 B line) and solved 4 (m + 1) tridiagonal systems: 85.4 ms for that band
// through 2236 steps against 19.5, and 162 ms against 37.1 for 8192 bundles through 14 periodic 128^3
// meshes in lambda (21.5 and 43.8 when every stage elected a leader instead of comparing with the kept window).
// The fetch shared by the bundle but not kept: 57 and 65 ms.
template <int NI, bool SAMEZ>
struct PmWave {
  static constexpr int m = 2 * NI;
  static constexpr bool KEEP = NI <= 3;
  static constexpr int QG = KEEP ? 4 : 1;               // quantities at a time
  static constexpr int kNodes = QG * m * m;
  static constexpr int kRounds = (kNodes + 8) / 9;      // of a bundle's nine lanes
  static constexpr int kRaw = 4 * kNodes + 2;           // + 2: the bundles' reads start in different banks
  static constexpr bool SLOPE = !SAMEZ && NI <= 2;      // (for NI = 3 the slopes would cost a wavefront per unit)
  static constexpr int kVal = SAMEZ ? (KEEP ? kNodes + 2 : 0) : (SLOPE ? 2 * kNodes + 2 : 0);
  static constexpr int kDoubles = 7 * (kRaw + kVal);

  // What the bundle's raw area holds (the same on its nine lanes).
  int tag_g = -1, tag_x = 0, tag_y = 0, tag_z = 0;

  // Every lane of the wavefront calls this; want: the lane has a field to look up; gi names the grid.
  __device__ __forceinline__ void eval(double* lds, int lane, bool want, int gi, const PmGrid& g,
                                       const double* fields, double x, double y, double z, double& phi,
                                       double& gx, double& gy, double& gz) {
    phi = gx = gy = gz = 0.0;
    if (!__any(want)) return;
    PmPoint<NI> p{};
    want = want && p.set(g, x, y, z);
    if (!__any(want)) return;   // (an isolated grid fills little of a ray's way)
    const int seg = lane < 63 ? lane / 9 : 6, k9 = lane - 9 * seg;
    double* raw = lds + seg * kRaw;
    double* val = lds + 7 * kRaw + seg * kVal;
    double out[4] = {0.0, 0.0, 0.0, 0.0};
    // nearly always: every bundle holds what its rays ask for
    if (KEEP && __all(!want || (tag_g == gi && tag_x == p.wx && tag_y == p.wy && tag_z == p.kz))) {
      combine(raw, val, seg, k9, want, p, g.h, out);
      lds_sync();
      phi = out[0];
      gx = out[1];
      gy = out[2];
      gz = out[3];
      return;
    }
    bool pending = want;
    for (;;) {
      const unsigned long long all = __ballot(pending);
      if (all == 0) break;
      const unsigned mine = (unsigned)(all >> (9 * seg)) & 0x1ffu;
      const int lead = 9 * seg + (mine ? __ffs(mine) - 1 : 0);
      const int lgi = __shfl(gi, lead), lwx = __shfl(p.wx, lead), lwy = __shfl(p.wy, lead), lkz = __shfl(p.kz, lead);
      const bool take = pending && gi == lgi && p.wx == lwx && p.wy == lwy && p.kz == lkz;
      const bool load = mine && k9 < 9 && !(KEEP && tag_g == lgi && tag_x == lwx && tag_y == lwy && tag_z == lkz);
      if (__any(load)) {
        const int ln = __shfl(g.n, lead), lper = __shfl(g.periodic, lead);
        const double* lf = reinterpret_cast<const double*>(__shfl((unsigned long long)fields, lead));
        if (KEEP) {
          if (load) {
            fetch(raw, 0, k9, lf, ln, lper, lwx, lwy, lkz);
            tag_g = lgi;
            tag_x = lwx;
            tag_y = lwy;
            tag_z = lkz;
          }
          lds_sync();
        } else {
          for (int q = 0; q < 4; ++q) {
            if (load) fetch(raw, q, k9, lf, ln, lper, lwx, lwy, lkz);
            lds_sync();
            combine(raw, val, seg, k9, take, p, g.h, out + q);
            lds_sync();
          }
        }
      }
      if (KEEP) {
        combine(raw, val, seg, k9, take, p, g.h, out);
        lds_sync();
      }
      pending = pending && !take;
    }
    phi = out[0];
    gx = out[1];
    gy = out[2];
    gz = out[3];
  }

 private:
  // This lane's ninth of the nodes of QG quantities from q0 on.
  __device__ __forceinline__ static void fetch(double* raw, int q0, int k9, const double* f, int n, int periodic, int wx,
                                               int wy, int kz) {
    const int64_t n3 = (int64_t)n * n * n;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const int t = k9 + 9 * r;
      if (t < kNodes) {
        const int q = q0 + t / (m * m), a = (t / m) % m, b = t % m;
        const double2u v = load_pair(f + q * n3, n, periodic, wx + a, wy + b, kz);
        const double2u v2 = load_pair(f + (q + 4) * n3, n, periodic, wx + a, wy + b, kz);
        raw[4 * t] = v[0];
        raw[4 * t + 1] = v[1];
        raw[4 * t + 2] = v2[0];
        raw[4 * t + 3] = v2[1];
      }
    }
  }

  // The interpolated quantities of the lanes that take this round's window.
  __device__ __forceinline__ static void combine(const double* raw, double* val, int seg, int k9, bool take,
                                                 const PmPoint<NI>& p, double h, double* out) {
    if constexpr (SAMEZ && KEEP) {
      // all rays of the wavefront are at one height of one grid
      const int one = __ffsll(__ballot(take)) - 1;
      if (one < 0) return;
      double c[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) c[i] = read_lane(p.cz[i], one);
      if (k9 < 9) {
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
          const int t = k9 + 9 * r;
          if (t < kNodes)
            val[t] = along_z(c, raw[4 * t], raw[4 * t + 1], raw[4 * t + 2], raw[4 * t + 3]);
        }
      }
      lds_sync();
      const double unit[1] = {1.0};
      if (take) weigh<1>(val, unit, p, out);
    } else if constexpr (!SLOPE) {
      if (take) weigh<4>(raw, p.cz, p, out);
    } else {
      // The heights of a bundle's rays differ by far less than a node spacing: value and slope along x^3 at one
      // of them serve all, where the next term, d^2 / 2 times a second difference, is below the rounding of
      // the value (d: the difference in spacings).
      const unsigned takers = (unsigned)(__ballot(take) >> (9 * seg)) & 0x1ffu;
      const int lead = 9 * seg + (takers ? __ffs(takers) - 1 : 0);
      const double A = __shfl(p.cz[0], lead), B = 1.0 - A, d = p.cz[0] - A;
      if (__all(!take || fabs(d) < 0x1p-27)) {
        const double hl = __shfl(h, lead), h6 = hl * hl * (1.0 / 6.0);
        const double c2 = (A * A * A - A) * h6, c3 = (B * B * B - B) * h6;
        const double s2 = (3.0 * A * A - 1.0) * h6, s3 = (1.0 - 3.0 * B * B) * h6;   // d/dA; of A and B: 1, -1
        if (k9 < 9) {
#pragma unroll
          for (int r = 0; r < kRounds; ++r) {
            const int t = k9 + 9 * r;
            if (t < kNodes) {
              const double f0 = raw[4 * t], f1 = raw[4 * t + 1], g0 = raw[4 * t + 2], g1 = raw[4 * t + 3];
              val[2 * t] = A * f0 + B * f1 + (c2 * g0 + c3 * g1);
              val[2 * t + 1] = (f0 - f1) + (s2 * g0 + s3 * g1);
            }
          }
        }
        lds_sync();
        const double two[2] = {1.0, d};
        if (take) weigh<2>(val, two, p, out);
      } else if (take) {
        weigh<4>(raw, p.cz, p, out);
      }
    }
  }

  // Sums over the window of C values a node, weighted by c (its first is 1 for fewer than four).
  template <int C>
  __device__ __forceinline__ static void weigh(const double* v, const double (&c)[C], const PmPoint<NI>& p, double* out) {
#pragma unroll
    for (int q = 0; q < QG; ++q) {
      double s = 0.0;
#pragma unroll
      for (int a = 0; a < m; ++a) {
        double w = 0.0;
#pragma unroll
        for (int b = 0; b < m; ++b) {
          const double* t = v + C * ((q * m + a) * m + b);
          if constexpr (C == 1) w = fma(p.y[b], t[0], w);
          else if constexpr (C == 2) w = fma(p.y[b], fma(c[1], t[1], t[0]), w);
          else w = fma(p.y[b], along_z(c, t[0], t[1], t[2], t[3]), w);
        }
        s = fma(p.x[a], w, s);
      }
      out[q] = s;
    }
  }

  // lane's value of v (lane: the same on all lanes), through scalar registers
  __device__ __forceinline__ static double read_lane(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
  }

  // LDS of one wavefront: its own stores are visible to its lanes after this
  __device__ __forceinline__ static void lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
};

// The rays of a wavefront whose bundles are wider than cells: every ray loads its own nodes.
template <int NI>
struct PmLanes {
  __device__ __forceinline__ void eval(double*, int, bool want, int, const PmGrid& g, const double* fields, double x, double y,
                                       double z, double& phi, double& gx, double& gy, double& gz) {
    phi = gx = gy = gz = 0.0;
    if (!__any(want)) return;
    PmPoint<NI> p{};
    double out[4] = {0.0, 0.0, 0.0, 0.0};
    want = want && p.set(g, x, y, z);
    pm_gather_lanes<NI, NI == 1 ? 8 : (NI == 4 ? 1 : 2)>(want, p, g.n, g.periodic, fields, out);
    phi = out[0];
    gx = out[1];
    gy = out[2];
    gz = out[3];
  }
};

// Whether some bundle of the wavefront becomes wide on straight lines to z_end: a ray more than a twentieth of a
// node spacing h (for windows of two nodes a side, whose loads are few, a thousandth) away from its anchor.  Its rays
// then ask for different windows at many stages, and a round of fetching for each takes longer than a load of every ray's own nodes: the wavefront takes that way from the start.
// Both give a ray the same bits in z.  4096 bundles through a periodic 128^3 mesh, four nodes a side, 40 steps in z, rings of a
// fifteenth, two thirds and seven spacings: shared 2.3, 4.6, 11.2 ms, own nodes 1.6, 2.2, 8.5; of a 150th 1.9 and 2.9.
template <int NI>
__device__ __forceinline__ bool wide_bundles(int lane, bool valid, const double* rays, int64_t N, int64_t ri, double z_end,
                                             double h) {
  const int anchor = lane < 63 ? lane - lane % 9 : 54;
  const double x = rays[N + ri], y = rays[2 * N + ri], l = fabs(z_end - rays[3 * N + ri]);
  const double ik = 1.0 / rays[7 * N + ri], sx = rays[5 * N + ri] * ik, sy = rays[6 * N + ri] * ik;
  const double dx = fabs(x - __shfl(x, anchor)) + fabs(sx - __shfl(sx, anchor)) * l;
  const double dy = fabs(y - __shfl(y, anchor)) + fabs(sy - __shfl(sy, anchor)) * l;
  const double limit = (NI == 1 ? 0.001 : 0.05) * h;
  return __any(valid && (dx > limit || dy > limit));
}

template <int NI>
__global__ __launch_bounds__(256) void pm_eval_kernel(PmGrid g, const double* __restrict__ fields, int64_t np,
                                                      const double* __restrict__ pts, double* phi, double* grad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= np) return;
  double p, gx, gy, gz;
  if constexpr (NI <= 2) pm_field<NI>(g, fields, pts[i], pts[np + i], pts[2 * np + i], p, gx, gy, gz);
  else pm_splines<NI>(g, fields, pts[i], pts[np + i], pts[2 * np + i], p, gx, gy, gz);
  phi[i] = p;
  grad[i] = gx;
  grad[np + i] = gy;
  grad[2 * np + i] = gz;
}

// ------------------------------------------------------------------ trace through the PM field
// One ray per lane, seven bundles per wavefront and workgroup (small workgroups spread a band of
// some thousand bundles evenly over the 1024 SIMDs); the same RK4 in z, Christoffel contraction and
// flags as the direct-sum trace kernel, with the field of step s taken from grid
// step_grid[s] (none for -1): one isolated grid for a lens, one periodic grid
// per box replica for a light cone.
template <int NI, class Mesh>
__device__ __forceinline__ void pm_trace_rays(Mesh mesh, double* lds, const DevCosmo& cz, const DevPmGrid* __restrict__ grids,
                                              const int32_t* __restrict__ step_grid, const double* __restrict__ nodes,
                                              int32_t step_begin, int32_t step_end, double* rays, int64_t N, int64_t ri,
                                              bool valid, uint8_t* flags) {
  const int lane = threadIdx.x;
  State Y{rays[ri], rays[N + ri], rays[2 * N + ri], rays[4 * N + ri], rays[5 * N + ri], rays[6 * N + ri],
          rays[7 * N + ri]};
  double zpos = rays[3 * N + ri];
  uint8_t flag = 0;
  bool live = valid;
  int cur = -1;
  PmGrid g{0, 0.0, 0.0, 0.0, 1.0, 0, 1.0};
  const double* fields = nullptr;
  double Z1 = nodes[step_begin];
  for (int s = step_begin; s < step_end && __any(live); ++s) {
    const double Z0 = Z1;
    Z1 = nodes[s + 1];
    const double h = Z1 - Z0, hh = 0.5 * h;
    const int gi = step_grid[s];
    if (gi >= 0 && gi != cur) {
      const DevPmGrid d = grids[gi];
      g = PmGrid{d.n, d.origin[0], d.origin[1], d.origin[2], d.h, d.periodic, 1.0 / d.h};
      fields = d.fields;
      cur = gi;
    }
    State acc{}, Ys{}, k;
    double psi;
#pragma unroll 1
    for (int stage = 0; stage < 4; ++stage) {
      const State& Yin = (stage == 0) ? Y : Ys;
      const double zs = (stage == 0) ? Z0 : ((stage == 3) ? Z1 : Z0 + hh);
      double phi, gx, gy, gz;
      mesh.eval(lds, lane, live && gi >= 0, gi, g, fields, Yin.x, Yin.y, zs, phi, gx, gy, gz);
      k = rhs(cz, Yin, phi, gx, gy, gz, psi);
      if (stage == 0) {
        if (live && fabs(psi) > 1e-2) flag |= 4;
        acc = k;
        Ys = axpy(Y, hh, k);
      } else if (stage == 1) {
        acc = axpy(acc, 2.0, k);
        Ys = axpy(Y, hh, k);
      } else if (stage == 2) {
        acc = axpy(acc, 2.0, k);
        Ys = axpy(Y, h, k);
      } else {
        acc = axpy(acc, 1.0, k);
      }
    }
    if (live) {
      const State Yn = axpy(Y, h / 6.0, acc);
      const bool finite = isfinite(Yn.t) && isfinite(Yn.x) && isfinite(Yn.y) && isfinite(Yn.kt) && isfinite(Yn.kx) &&
                          isfinite(Yn.ky) && isfinite(Yn.kz);
      if (!finite) {
        flag |= 1;
        live = false;
      } else if (!(Yn.kz > 0.0)) {
        flag |= 2;
        live = false;
      } else {
        Y = Yn;
        zpos = Z1;
      }
    }
  }
  if (!valid) return;
  rays[ri] = Y.t;
  rays[N + ri] = Y.x;
  rays[2 * N + ri] = Y.y;
  rays[3 * N + ri] = zpos;
  rays[4 * N + ri] = Y.kt;
  rays[5 * N + ri] = Y.kx;
  rays[6 * N + ri] = Y.ky;
  rays[7 * N + ri] = Y.kz;
  if (flags && flag) flags[ri] |= flag;
}

template <int NI>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(NI == 3 ? 1 : 2, NI == 3 ? 1 : 2))) void pm_trace_kernel(
    DevCosmo cz, const DevPmGrid* __restrict__ grids, const int32_t* __restrict__ step_grid,
    const double* __restrict__ nodes, int32_t step_begin, int32_t step_end, double h_min, double* rays, int64_t N,
    uint8_t* flags) {
  __shared__ double lds[PmWave<NI, true>::kDoubles];
  const int64_t at = (int64_t)blockIdx.x * 63 + threadIdx.x;
  const bool valid = threadIdx.x < 63 && at < N;
  const int64_t ri = valid ? at : N - 1;
  if (wide_bundles<NI>(threadIdx.x, valid, rays, N, ri, nodes[step_end], h_min))
    pm_trace_rays<NI>(PmLanes<NI>{}, lds, cz, grids, step_grid, nodes, step_begin, step_end, rays, N, ri, valid, flags);
  else
    pm_trace_rays<NI>(PmWave<NI, true>{}, lds, cz, grids, step_grid, nodes, step_begin, step_end, rays, N, ri, valid, flags);
}

// The paper's own integrator (Sec. 3.4, eq. RKstepsize): classical RK4 in the
// affine parameter with the fixed step f_RK h / kz_0 (h: the Fourier-grid
// spacing, kz_0: the ray's dz/dlambda at the start), repeated until z reaches
// chi_s; the step that overshoots is replaced by the linear interpolation
// between the previous and the current state at z = chi_s.  One ray per
// lane, seven bundles per wavefront as in pm_trace_kernel; a ray that has not
// reached chi_s after max_steps is flagged 8.  The
// field is a functor of the evaluation point: one grid everywhere, or the grid
// of the slab along x^3 that holds the point (Sec. 5.2's stack of cubes).
struct State8 {
  double t, x, y, z, kt, kx, ky, kz;
};

__device__ __forceinline__ State8 axpy8(const State8& Y, double h, const State8& k) {
  return State8{Y.t + h * k.t,   Y.x + h * k.x,   Y.y + h * k.y,   Y.z + h * k.z,
                Y.kt + h * k.kt, Y.kx + h * k.kx, Y.ky + h * k.ky, Y.kz + h * k.kz};
}

// Picks the grid of height z for one lane: false where there is none.  g, fields and gi
// keep the last grid picked.
struct OneGrid {
  PmGrid grid;
  const double* data;
  __device__ __forceinline__ bool pick(double, int& gi, PmGrid& g, const double*& fields, double&, double&) const {
    gi = 0;
    g = grid;
    fields = data;
    return true;
  }
};

// bounds [n_slabs + 1] strictly increasing; slab k = [bounds[k], bounds[k + 1])
// takes grid slab_grid[k] (none for -1); no field outside [bounds[0],
// bounds[n_slabs]) (a NaN z included).  lo, hi: the slab that the lane was in last.
struct SlabGrids {
  const DevPmGrid* grids;
  const double* bounds;
  const int32_t* slab_grid;
  int32_t n_slabs;
  __device__ __forceinline__ bool pick(double z, int& gi, PmGrid& g, const double*& fields, double& lo,
                                       double& hi) const {
    if (z >= lo && z < hi) return gi >= 0;
    if (!(z >= bounds[0] && z < bounds[n_slabs])) return false;
    int a = 0, b = n_slabs;   // bounds[a] <= z < bounds[b]
    while (b - a > 1) {
      const int mid = (a + b) >> 1;
      if (z >= bounds[mid])
        a = mid;
      else
        b = mid;
    }
    lo = bounds[a];
    hi = bounds[a + 1];
    gi = slab_grid[a];
    if (gi < 0) return false;
    const DevPmGrid d = grids[gi];
    g = PmGrid{d.n, d.origin[0], d.origin[1], d.origin[2], d.h, d.periodic, 1.0 / d.h};
    fields = d.fields;
    return true;
  }
};

template <int NI, class Grids, class Mesh>
__device__ __forceinline__ void pm_trace_rays_lambda(Mesh mesh, double* lds, const DevCosmo& cz, const Grids& grids, double h_rk,
                                                     double chi_s, double f_rk, int32_t max_steps, double* rays, int64_t N,
                                                     int64_t ri, bool valid, uint8_t* flags, int32_t* steps_out) {
  const int lane = threadIdx.x;
  State8 Y{rays[ri],         rays[N + ri],     rays[2 * N + ri], rays[3 * N + ri],
           rays[4 * N + ri], rays[5 * N + ri], rays[6 * N + ri], rays[7 * N + ri]};
  const double dl = f_rk * h_rk / Y.kz;
  uint8_t flag = 0;
  bool done = !valid || !(Y.z < chi_s);
  int32_t steps = 0;
  int gi = -1;
  PmGrid g{4, 0.0, 0.0, 0.0, 1.0, 0, 1.0};
  const double* fields = nullptr;
  double lo = 1.0, hi = 0.0;   // no slab yet
  for (int32_t s = 0; s < max_steps && __any(!done); ++s) {
    State8 sum{}, Ys = Y;
#pragma unroll 1
    for (int stage = 0; stage < 4; ++stage) {
      double phi, gx, gy, gz, psi, At, Ax, Ay, Az;
      const bool want = !done && grids.pick(Ys.z, gi, g, fields, lo, hi);
      mesh.eval(lds, lane, want, gi, g, fields, Ys.x, Ys.y, Ys.z, phi, gx, gy, gz);
      accel(cz, Ys.t, Ys.kt, Ys.kx, Ys.ky, Ys.kz, phi, gx, gy, gz, psi, At, Ax, Ay, Az);
      const State8 k{Ys.kt, Ys.kx, Ys.ky, Ys.kz, -At, -Ax, -Ay, -Az};
      if (stage == 0) {
        if (!done && fabs(psi) > 1e-2) flag |= 4;
        sum = k;
      } else {
        sum = axpy8(sum, stage == 3 ? 1.0 : 2.0, k);
      }
      Ys = axpy8(Y, stage == 2 ? dl : 0.5 * dl, k);
    }
    if (done) continue;
    ++steps;
    const State8 Yn = axpy8(Y, dl / 6.0, sum);
    const bool finite = isfinite(Yn.t) && isfinite(Yn.x) && isfinite(Yn.y) && isfinite(Yn.z) && isfinite(Yn.kt) &&
                        isfinite(Yn.kx) && isfinite(Yn.ky) && isfinite(Yn.kz);
    if (!finite) {
      flag |= 1;
      done = true;
    } else if (!(Yn.kz > 0.0)) {
      flag |= 2;
      done = true;
    } else if (Yn.z >= chi_s) {
      const double w = (chi_s - Y.z) / (Yn.z - Y.z);
      Y = State8{Y.t + w * (Yn.t - Y.t),     Y.x + w * (Yn.x - Y.x),     Y.y + w * (Yn.y - Y.y),
                 Y.z + w * (Yn.z - Y.z),     Y.kt + w * (Yn.kt - Y.kt),  Y.kx + w * (Yn.kx - Y.kx),
                 Y.ky + w * (Yn.ky - Y.ky), Y.kz + w * (Yn.kz - Y.kz)};
      done = true;
    } else {
      Y = Yn;
    }
  }
  if (!valid) return;
  if (!done) flag |= 8;
  rays[ri] = Y.t;
  rays[N + ri] = Y.x;
  rays[2 * N + ri] = Y.y;
  rays[3 * N + ri] = Y.z;
  rays[4 * N + ri] = Y.kt;
  rays[5 * N + ri] = Y.kx;
  rays[6 * N + ri] = Y.ky;
  rays[7 * N + ri] = Y.kz;
  if (flags && flag) flags[ri] |= flag;
  if (steps_out) steps_out[ri] = steps;
}

template <int NI, class Grids>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void pm_trace_lambda_kernel(
    DevCosmo cz, Grids grids, double h_rk, double chi_s, double f_rk, int32_t max_steps, double* rays, int64_t N,
    uint8_t* flags, int32_t* steps_out) {
  __shared__ double lds[PmWave<NI, false>::kDoubles];
  const int64_t at = (int64_t)blockIdx.x * 63 + threadIdx.x;
  const bool valid = threadIdx.x < 63 && at < N;
  const int64_t ri = valid ? at : N - 1;
  if (wide_bundles<NI>(threadIdx.x, valid, rays, N, ri, chi_s, h_rk))
    pm_trace_rays_lambda<NI>(PmLanes<NI>{}, lds, cz, grids, h_rk, chi_s, f_rk, max_steps, rays, N, ri, valid, flags, steps_out);
  else
    pm_trace_rays_lambda<NI>(PmWave<NI, false>{}, lds, cz, grids, h_rk, chi_s, f_rk, max_steps, rays, N, ri, valid, flags,
                             steps_out);
}

inline unsigned blocks_for(int64_t count, int threads) { return (unsigned)((count + threads - 1) / threads); }

}  // namespace

const void* trace_ray_fn() { return (const void*)&trace_few_kernel<kRayPlanRays, 1, 1, kRayPlanTile>; }

hipError_t launch_trace_ray(const TraceParams& p, int grid, hipStream_t s) {
  hipLaunchKernelGGL((trace_few_kernel<kRayPlanRays, 1, 1, kRayPlanTile>), dim3(grid), dim3(64), 0, s, p);
  return hipGetLastError();
}

int64_t pm_workspace_bytes(int n, int periodic) {
  const int64_t M = periodic ? (int64_t)n : 2 * (int64_t)n;
  return 2 * M * M * M * (int64_t)sizeof(double2) + (M / 2) * (int64_t)sizeof(double2);
}

// Workspace (32 M^3 bytes and M / 2 twiddles), in points of 16 B.  Isolated, m = n + 1 = M / 2 + 1:
//   [4][n][M][m] results | [n][M][m] masses after two axes | kernels (P, S) [m][m][m] | S by the last axis
// with the masses, their transform along one axis and the kernels' transforms on the way in the results' place;
// fullest at n = 4, where it takes 988 of 1,024 points.  Periodic, m = n / 2 + 1: two results; the other two lie
// in the fields' second-derivative grids and the masses [n][n][m] in their first four, which are written later.
hipError_t launch_pm_build(const double* xyzm, int64_t np, double eps, const double origin[3], double h, int n,
                           int periodic, double G, double* fields, void* workspace, hipStream_t s) {
  const int M = periodic ? n : 2 * n;
  const int64_t M3 = (int64_t)M * M * M, n3 = (int64_t)n * n * n;
  double2* ws = static_cast<double2*>(workspace);
  double2* tw = ws + 2 * M3;
  const Fft f = make_fft(M, tw);
  const int nk = M / 2 + 1;
  const int64_t half = (int64_t)n * M * nk;   // one result, or the masses after two axes
  const dim3 threads(kFftThreads);
  const unsigned batches = blocks_for(nk, f.L);   // of the last axis's points, f.L at a time
  FourOut out;
  double2 *mass, *last;        // after two axes, after one
  double* rho;
  if (periodic) {
    // (fields may be 8-byte aligned; both places have a point to spare)
    auto aligned = [](double* p) { return reinterpret_cast<double2*>((reinterpret_cast<uintptr_t>(p) + 15) & ~(uintptr_t)15); };
    mass = last = aligned(fields);
    out.q[0] = ws;
    out.q[1] = ws + half;
    out.q[2] = aligned(fields + 4 * n3);
    out.q[3] = out.q[2] + half;
    rho = reinterpret_cast<double*>(ws);
  } else {
    for (int q = 0; q < 4; ++q) out.q[q] = ws + q * half;
    mass = ws + 4 * half;
    rho = reinterpret_cast<double*>(ws);
    last = ws + (n3 + 1) / 2;
  }
  hipLaunchKernelGGL(pm_twiddle_kernel, dim3(blocks_for(M / 2, 256)), dim3(256), 0, s, tw, M);
  double2* ps = nullptr;
  double* sz = nullptr;
  if (!periodic) {
    ps = mass + half;
    const int64_t mm = (int64_t)nk * nk;
    double2* c = ws;
    // phi / (d phi / dx) in the root mean square over the grid, from e = the larger of spacing and softening to R =
    // its side: 1/r over it falls to 1/R, x/r^3 to 1/sqrt(e R^3), and for a softening beyond the side to R/e^2
    const double e = h > eps ? h : eps, R = n * h;
    const double ratio = sqrt(e) * sqrt(R) * (e > R ? (e / R) * sqrt(e / R) : 1.0);
    const double len = ratio > 1e-100 && ratio < 1e100 ? exp2(rint(log2(ratio))) : 1.0;
    sz = reinterpret_cast<double*>(ps + mm * nk);
    hipLaunchKernelGGL(pm_kernel_last_kernel, dim3(blocks_for(mm, f.L)), threads, 0, s, f, n, h, eps * eps, G, len, c);
    hipLaunchKernelGGL(pm_kernel_mid_kernel, dim3(batches, nk), threads, 0, s, f, n, c);
    hipLaunchKernelGGL(pm_kernel_first_kernel, dim3(batches, nk), threads, 0, s, f, n, (const double2*)c,
                       1.0 / (double)M3, 1.0 / len, ps, sz);
  }
  hipLaunchKernelGGL(pm_clear_kernel, dim3(blocks_for(n3, 256)), dim3(256), 0, s, rho, n3);
  if (np > 0 && n <= kCicSmall)
    hipLaunchKernelGGL(pm_cic_small_kernel, dim3(np < 64 * kCicThreads ? blocks_for(np, kCicThreads) : 64u), dim3(kCicThreads), 0,
                       s, xyzm, np, origin[0], origin[1], origin[2], h, n, periodic, rho);
  else if (np > 0)
    hipLaunchKernelGGL(pm_cic_kernel, dim3(blocks_for(np, 256)), dim3(256), 0, s, xyzm, np, origin[0], origin[1],
                       origin[2], h, n, periodic, rho);
  const int64_t lines = (int64_t)n * n;
  hipLaunchKernelGGL(pm_fft_real_kernel, dim3(blocks_for(lines, 2 * f.L)), threads, 0, s, f, (const double*)rho, n, lines,
                     last);
  hipLaunchKernelGGL(pm_fft_mid_kernel, dim3(batches, n), threads, 0, s, f, (const double2*)last, n, nk, mass);
  if (periodic)
    hipLaunchKernelGGL(pm_product_kernel<true>, dim3(batches, M), threads, 0, s, f, (const double2*)mass, n, n, nk,
                       (const double2*)nullptr, (const double*)nullptr, 2.0 * M_PI / (n * h),
                       -4.0 * M_PI * G / (h * h * h) / (double)M3, out);
  else
    hipLaunchKernelGGL(pm_product_kernel<false>, dim3(batches, M), threads, 0, s, f, (const double2*)mass, n, n, nk,
                       (const double2*)ps, (const double*)sz, 0.0, 0.0, out);
  hipLaunchKernelGGL(pm_ifft_mid_kernel, dim3(batches, n, 4), threads, 0, s, f, out, nk, n);
  hipLaunchKernelGGL(pm_ifft_real_kernel, dim3(blocks_for(lines, 2 * f.L), 1, 4), threads, 0, s, f, out, M, n, nk, fields);
  const double* values = fields;
  if (periodic) return launch_spline_z<true>(values, fields + 4 * n3, n, h, 4 * lines, s);
  return launch_spline_z<false>(values, fields + 4 * n3, n, h, 4 * lines, s);
}

hipError_t launch_pm_eval(const double origin[3], double h, int n, int periodic, const double* fields, int n_int, int64_t np,
                          const double* pts, double* phi, double* grad, hipStream_t s) {
  const PmGrid g{n, origin[0], origin[1], origin[2], h, periodic, 1.0 / h};
  const dim3 grid(blocks_for(np, 256)), block(256);
  switch (n_int) {
    case 1: hipLaunchKernelGGL(pm_eval_kernel<1>, grid, block, 0, s, g, fields, np, pts, phi, grad); break;
    case 2: hipLaunchKernelGGL(pm_eval_kernel<2>, grid, block, 0, s, g, fields, np, pts, phi, grad); break;
    case 3: hipLaunchKernelGGL(pm_eval_kernel<3>, grid, block, 0, s, g, fields, np, pts, phi, grad); break;
    default: hipLaunchKernelGGL(pm_eval_kernel<4>, grid, block, 0, s, g, fields, np, pts, phi, grad); break;
  }
  return hipGetLastError();
}

hipError_t launch_pm_trace(DevCosmo c, const DevPmGrid* grids, const int32_t* step_grid, int n_int,
                           const double* nodes, int32_t step_begin, int32_t step_end, double h_min, double* rays, int64_t n_rays,
                           uint8_t* flags, hipStream_t s) {
  const dim3 grid(blocks_for(n_rays, 63)), block(64);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, s, c, grids, step_grid, nodes, step_begin, step_end, h_min, rays, n_rays,
                       flags);
  };
  switch (n_int) {
    case 1: go(pm_trace_kernel<1>); break;
    case 2: go(pm_trace_kernel<2>); break;
    case 3: go(pm_trace_kernel<3>); break;
    default: go(pm_trace_kernel<4>); break;
  }
  return hipGetLastError();
}

namespace {
template <class Grids>
hipError_t launch_lambda(DevCosmo c, const Grids& grids, double h_rk, int n_int, double chi_s, double f_rk,
                         int32_t max_steps, double* rays, int64_t n_rays, uint8_t* flags, int32_t* steps,
                         hipStream_t s) {
  const dim3 grid(blocks_for(n_rays, 63)), block(64);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, s, c, grids, h_rk, chi_s, f_rk, max_steps, rays, n_rays, flags, steps);
  };
  switch (n_int) {
    case 1: go(pm_trace_lambda_kernel<1, Grids>); break;
    case 2: go(pm_trace_lambda_kernel<2, Grids>); break;
    case 3: go(pm_trace_lambda_kernel<3, Grids>); break;
    default: go(pm_trace_lambda_kernel<4, Grids>); break;
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_pm_trace_lambda(DevCosmo c, const double origin[3], double h, int n, int periodic, const double* fields,
                                  int n_int, double chi_s, double f_rk, int32_t max_steps, double* rays,
                                  int64_t n_rays, uint8_t* flags, int32_t* steps, hipStream_t s) {
  const OneGrid g{PmGrid{n, origin[0], origin[1], origin[2], h, periodic, 1.0 / h}, fields};
  return launch_lambda(c, g, h, n_int, chi_s, f_rk, max_steps, rays, n_rays, flags, steps, s);
}

hipError_t launch_pm_trace_lambda_slabs(DevCosmo c, const DevPmGrid* grids, const double* bounds,
                                        const int32_t* slab_grid, int32_t n_slabs, double h_rk, int n_int,
                                        double chi_s, double f_rk, int32_t max_steps, double* rays, int64_t n_rays,
                                        uint8_t* flags, int32_t* steps, hipStream_t s) {
  const SlabGrids g{grids, bounds, slab_grid, n_slabs};
  return launch_lambda(c, g, h_rk, n_int, chi_s, f_rk, max_steps, rays, n_rays, flags, steps, s);
}

}  // namespace rt
