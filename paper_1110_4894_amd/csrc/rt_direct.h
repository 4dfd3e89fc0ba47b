// Device code of the FP64 direct sum that more than one file of kernels uses: the pair term, the uniform
// cuboid, and the trace kernel for few rays.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include "rt_geodesic.h"
#include "rt_internal.h"

namespace rt {
namespace {

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// FP64 reciprocal square root of a finite x > 0: the hardware estimate r
// (relative error about 2^-24) refined with the second-order expansion of
// (1 - e)^(-1/2), where e = 1 - x r^2:  r (1 + e/2 + 3 e^2/8).  The neglected
// term is 5 e^3 / 16, far below 2^-53.  The input is r^2 + eps^2 of a pair;
// it is zero only for a ray exactly on an unsoftened particle, where the
// field is singular anyway (the result is then NaN and the ray is flagged).
__device__ __forceinline__ double rsqrt_f64(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * r), r, 1.0);
  return fma(r * e, fma(0.375, e, 0.5), r);
}

// ---------------------------------------------------------------------------
// Uniform cuboid of unit density: U = int d^3x'/|p - x'| and dU/dp, from the
// antiderivative of 1/R evaluated at the eight corners (mean-density term of
// Sec. 3.3).  Each corner's three logarithms and three arctangents serve both
// U and its gradient; terms whose coefficient vanishes are skipped, which
// keeps faces, edges and corners finite (the observer sits on a face of the
// first box replica).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double log_w_plus_r(double w, double R, double other2) {
  if (other2 == 0.0) return 0.0;      // every coefficient of this log is zero then
  return (w >= 0.0) ? log(w + R) : log(other2 / (R - w));
}

__device__ __forceinline__ void cuboid_corner(const double lo[3], const double hi[3], int corner, double px, double py,
                                              double pz, double& U, double& gx, double& gy, double& gz) {
  const int i = corner & 1, j = (corner >> 1) & 1, k = (corner >> 2) & 1;
  const double X = (i ? hi[0] : lo[0]) - px, Y = (j ? hi[1] : lo[1]) - py, Z = (k ? hi[2] : lo[2]) - pz;
  // sign = product over the axes of (+1 upper limit, -1 lower limit)
  const double s = ((i + j + k) & 1) ? 1.0 : -1.0;
  const double X2 = X * X, Y2 = Y * Y, Z2 = Z * Z;
  const double R = sqrt(X2 + Y2 + Z2);
  if (R == 0.0) return;
  const double LX = log_w_plus_r(X, R, Y2 + Z2);
  const double LY = log_w_plus_r(Y, R, Z2 + X2);
  const double LZ = log_w_plus_r(Z, R, X2 + Y2);
  const double AX = (X != 0.0) ? atan(Y * Z / (X * R)) : 0.0;
  const double AY = (Y != 0.0) ? atan(Z * X / (Y * R)) : 0.0;
  const double AZ = (Z != 0.0) ? atan(X * Y / (Z * R)) : 0.0;
  const double F = X * Y * LZ + Y * Z * LX + Z * X * LY - 0.5 * (X2 * AX + Y2 * AY + Z2 * AZ);
  U += s * F;
  // the limits move with p (d limit / dp = -1)
  gx -= s * (Y * LZ + Z * LY - X * AX);
  gy -= s * (Z * LX + X * LZ - Y * AY);
  gz -= s * (X * LY + Y * LX - Z * AZ);
}

__device__ __forceinline__ void cuboid_field(const double lo[3], const double hi[3], double px, double py, double pz,
                                             double& U, double& gx, double& gy, double& gz) {
  U = gx = gy = gz = 0.0;
#pragma unroll 1
  for (int corner = 0; corner < 8; ++corner) cuboid_corner(lo, hi, corner, px, py, pz, U, gx, gy, gz);
}

// One pair term of the direct sum.
__device__ __forceinline__ void pair_fp64(const double4 c, double x, double y, double z, double e2, double& a0,
                                          double& a1, double& a2, double& a3) {
  const double ex = c.x - x, ey = c.y - y, ez = c.z - z;
  double r2 = fma(ex, ex, e2);
  r2 = fma(ey, ey, r2);
  r2 = fma(ez, ez, r2);
  const double ri = rsqrt_f64(r2);
  const double mr = c.w * ri;
  a0 += mr;
  const double mr3 = mr * ri * ri;
  a1 = fma(mr3, ex, a1);
  a2 = fma(mr3, ey, a2);
  a3 = fma(mr3, ez, a3);
}

// ---------------------------------------------------------------------------
// Few rays: the trace kernel of launches that cannot fill the chip with a ray per lane.
// A workgroup of NW wavefronts holds R rays (a power of two).  Every lane integrates ray lane % R; for the
// sums a lane takes a share of the particles for K of the rays at once (lane = group + G slot, group g = rays
// g K .. g K + K - 1), so that one read of a particle from LDS serves K pairs and K chains of FP64 operations
// run side by side (FP64 direct sums, rays are independent).  The partial sums meet by lane exchanges (half of
// the rays go to the other half of the slots, until a lane holds one ray) and in LDS, in a fixed order, so that
// all copies of a ray stay identical.  The particles are staged in chunks of C, and a set that fits one chunk stays in
// LDS for as long as the steps use it.  The corners of a cuboid background are split over the copies of a ray.
// Bound: the chain of one stage (sum, reduction, right-hand side) and, beyond some thousand pairs per
// workgroup and stage, FP64 issue of the workgroup's compute unit.  Registers: two wavefronts per SIMD, so
// that the ray state stays in them (the other plans' 128 per lane spill it, and at one or two
// wavefronts per SIMD nothing hides the reloads).
// Measured: a point lens's 1024 bundles through 1225 steps 24.4 -> 3.8 ms (0.8 us a stage); 49 bundles in a halo of
// 3001 particles 103 -> 4.8 ms; 4 steps of 16 bundles, 32768 particles 6.7 -> 0.8 ms; of 896 bundles 6.8 -> 3.3 ms.
// One pair per particle read (K = 1) took 2.9 ms for 448 bundles against 2.0: LDS could not feed the pairs.
// ---------------------------------------------------------------------------
template <int R, int K, int NW, int C>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void trace_few_kernel(TraceParams P) {
  constexpr int G = R / K, ST = 64 / G * NW;              // groups; slots of the workgroup
  constexpr int COPIES = 64 / R;                           // of a ray per wavefront
  constexpr int CW = 8 / COPIES > 0 ? 8 / COPIES : 1;      // wavefronts that take cuboid corners
  static_assert(NW == 1 || CW <= NW, "every corner has a taker");
  __shared__ double px[C], py[C], pz[C], pm[C];
  __shared__ double red[2][NW > 1 ? NW + CW : 1][4][NW > 1 ? R : 1];
  __shared__ int s_item;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int ray = lane & (R - 1), group = lane & (G - 1), lslot = lane / G, slot = wave * (64 / G) + lslot;
  const DevCosmo& cz = P.cosmo;
  int held = -1;            // set whose particles are in LDS
  int64_t held_at = 0;      // from this one on
  int flip = 0;             // half of red in use
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(P.queue, 1);
    __syncthreads();
    const int item = s_item;
    __syncthreads();
    if (item >= P.n_items) break;
    const WorkItem wi = P.items[item];
    const DevField f = P.fields[wi.field];
    const int64_t rend = f.ray_begin + f.n_rays, N = P.n_rays;
    int64_t ri = f.ray_begin + (int64_t)wi.block * R + ray;
    const bool writes = wave == 0 && lane < R && ri < rend;
    if (ri >= rend) ri = rend - 1;
    State Y{P.rays[ri], P.rays[N + ri], P.rays[2 * N + ri], P.rays[4 * N + ri], P.rays[5 * N + ri],
            P.rays[6 * N + ri], P.rays[7 * N + ri]};
    double zpos = P.rays[3 * N + ri];
    uint8_t flag = 0;
    bool live = true;
    const int sb = P.step_begin < 0 ? 0 : P.step_begin;
    const int se = P.step_end > f.n_steps ? f.n_steps : P.step_end;
    for (int s = sb; s < se; ++s) {
      const double Z0 = P.nodes[f.node_off + s], Z1 = P.nodes[f.node_off + s + 1];
      const double h = Z1 - Z0, hh = 0.5 * h;
      const int S = P.step_set[f.step_off + s];
      const int idx = f.set_off + S;
      const DevSet* set = P.sets + (S >= 0 ? idx : 0);
      const int64_t n = S >= 0 ? set->n : 0;
      const double e2 = S >= 0 ? set->eps2 : 0.0;
      const bool background = S >= 0 && set->background;
      const double* __restrict__ src = S >= 0 ? set->p64 : nullptr;
      State acc{}, Ys{}, k;
      double psi;
#pragma unroll 1
      for (int stage = 0; stage < 4; ++stage) {
        const double x = (stage == 0) ? Y.x : Ys.x, y = (stage == 0) ? Y.y : Ys.y;
        const double z = (stage == 0) ? Z0 : ((stage == 3) ? Z1 : Z0 + hh);
        double xs[K], ys[K], sum[K][4];
#pragma unroll
        for (int i = 0; i < K; ++i) {
          xs[i] = K > 1 ? __shfl(x, group * K + i) : x;
          ys[i] = K > 1 ? __shfl(y, group * K + i) : y;
#pragma unroll
          for (int q = 0; q < 4; ++q) sum[i][q] = 0.0;
        }
        for (int64_t c0 = 0; c0 < n; c0 += C) {
          const int cnt = n - c0 < C ? (int)(n - c0) : C;
          if (held != idx || held_at != c0) {
            if (NW > 1) __syncthreads();
            else wave_sync();
            for (int j = threadIdx.x; j < cnt; j += NW * 64) {
              px[j] = src[c0 + j];
              py[j] = src[n + c0 + j];
              pz[j] = src[2 * n + c0 + j];
              pm[j] = src[3 * n + c0 + j];
            }
            if (NW > 1) __syncthreads();
            else wave_sync();
            held = idx;
            held_at = c0;
          }
#pragma unroll 1
          for (int j = NW > 1 ? slot : 0; j < cnt; j += NW > 1 ? ST : 1) {
            const double4 c = make_double4(px[j], py[j], pz[j], pm[j]);
#pragma unroll
            for (int i = 0; i < K; ++i) pair_fp64(c, xs[i], ys[i], z, e2, sum[i][0], sum[i][1], sum[i][2], sum[i][3]);
          }
        }
        double phi, gx, gy, gz;
        if constexpr (NW == 1) {   // no split: the lane's own ray
          phi = -cz.G * sum[0][0];
          gx = -cz.G * sum[0][1];
          gy = -cz.G * sum[0][2];
          gz = -cz.G * sum[0][3];
          if (background) {
            double U, ux, uy, uz;
            cuboid_field(set->lo, set->hi, x, y, z, U, ux, uy, uz);
            phi += cz.G_rho * U;
            gx += cz.G_rho * ux;
            gy += cz.G_rho * uy;
            gz += cz.G_rho * uz;
          }
        } else {
          phi = gx = gy = gz = 0.0;
          if (S >= 0) {
            double(*m)[4][R] = red[flip];
            flip ^= 1;
            // rays: halve what a lane holds until it is one
            int mine = 0;
#pragma unroll
            for (int b = 0; (K >> b) > 1; ++b) {
              const int keep = K >> (b + 1);
              const bool up = (lslot >> b) & 1;
              mine += up ? keep : 0;
#pragma unroll
              for (int i = 0; i < keep; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                  const double send = up ? sum[i][q] : sum[i + keep][q];
                  sum[i][q] = (up ? sum[i + keep][q] : sum[i][q]) + __shfl_xor(send, G << b);
                }
            }
            // the slots that hold the same ray
#pragma unroll
            for (int off = R; off < 64; off <<= 1)
#pragma unroll
              for (int q = 0; q < 4; ++q) sum[0][q] += __shfl_xor(sum[0][q], off);
            if (lane < R) {
#pragma unroll
              for (int q = 0; q < 4; ++q) m[wave][q][group * K + mine] = -cz.G * sum[0][q];
            }
            if (background && wave < CW) {
              double u[4] = {0.0, 0.0, 0.0, 0.0};
              for (int c = wave * COPIES + lane / R; c < 8; c += CW * COPIES)
                cuboid_corner(set->lo, set->hi, c, x, y, z, u[0], u[1], u[2], u[3]);
#pragma unroll
              for (int off = R; off < 64; off <<= 1)
#pragma unroll
                for (int q = 0; q < 4; ++q) u[q] += __shfl_xor(u[q], off);
              if (lane < R) {
#pragma unroll
                for (int q = 0; q < 4; ++q) m[NW + wave][q][ray] = cz.G_rho * u[q];
              }
            }
            __syncthreads();   // (the next stage writes the other half: one barrier per stage)
#pragma unroll
            for (int w = 0; w < NW; ++w) {
              phi += m[w][0][ray];
              gx += m[w][1][ray];
              gy += m[w][2][ray];
              gz += m[w][3][ray];
            }
            if (background) {
#pragma unroll
              for (int w = NW; w < NW + CW; ++w) {
                phi += m[w][0][ray];
                gx += m[w][1][ray];
                gy += m[w][2][ray];
                gz += m[w][3][ray];
              }
            }
          }
        }
        const State& Yin = (stage == 0) ? Y : Ys;
        k = rhs(cz, Yin, phi, gx, gy, gz, psi);
        if (stage == 0) {
          if (fabs(psi) > 1e-2) flag |= 4;
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
        const bool finite = isfinite(Yn.t) && isfinite(Yn.x) && isfinite(Yn.y) && isfinite(Yn.kt) &&
                            isfinite(Yn.kx) && isfinite(Yn.ky) && isfinite(Yn.kz);
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
    if (writes) {
      P.rays[ri] = Y.t;
      P.rays[N + ri] = Y.x;
      P.rays[2 * N + ri] = Y.y;
      P.rays[3 * N + ri] = zpos;
      P.rays[4 * N + ri] = Y.kt;
      P.rays[5 * N + ri] = Y.kx;
      P.rays[6 * N + ri] = Y.ky;
      P.rays[7 * N + ri] = Y.kz;
      if (P.flags && flag) P.flags[ri] |= flag;
    }
  }
}

}  // namespace
}  // namespace rt
