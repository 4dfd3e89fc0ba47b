// Device code shared by the direct-sum and the particle-mesh trace kernels:
// the background a(t) and the geodesic right-hand side in z.  Not part of the
// public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

#include "rt_internal.h"

namespace rt {

// FP64 reciprocal of a finite x != 0: the hardware estimate r (relative error about 2^-23)
// refined to r (1 + e + e^2), e = 1 - x r; the neglected e^3 is far below 2^-53.  Four dependent
// instructions against eleven of the IEEE division, which also scales operands near the ends of
// the exponent range; x = 0 or infinite gives NaN.
__device__ __forceinline__ double recip_f64(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// r^(-1/3) of a normal FP32-range r > 0: an FP32 estimate y refined with the expansion of
// (1 - e)^(-1/3), e = 1 - r y^3:  y (1 + e/3 + 2 e^2/9); |e| < 1e-5, so that the neglected
// 14 e^3/81 stays below 2^-52.
__device__ __forceinline__ double rcbrt_f64(double r) {
  const double y = (double)__builtin_amdgcn_exp2f(__builtin_amdgcn_logf((float)r) * (-1.0f / 3.0f));
  const double e = fma(-(r * y), y * y, 1.0);
  return fma(y * e, fma(2.0 / 9.0, e, 1.0 / 3.0), y);
}

// ---------------------------------------------------------------------------
// Background: a(t) of eq. scalefac2 (t = lookback time), 1/a and da/dt.
// a = (ratio sinh^2 u)^(1/3) comes as r (r^(-1/3))^2, which gives 1/a with it: no division by a.  Both are
// corrected by their own remainders, r - a^3 (with a^2 in two parts) and 1 - a (1/a), and so rounded like a cube
// root and a division (uncorrected, a was off by up to 3.7 x 2^-53).
// The integration of a ray is one chain of dependent FP64 operations per stage, whose length bounds the small
// launches; the corrections lengthen it by six of them (point lens, 4900 stages: 3.70 -> 3.81 ms).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void scale_factor(const DevCosmo& c, double t, double& a, double& inv_a, double& adot) {
  const double rate = 1.5 * c.sqrt_ol * c.H0;
  const double u = rate * (c.t0 - t);
  const double e = exp(u);
  const double ie = recip_f64(e);
  const double sh = 0.5 * (e - ie), ch = 0.5 * (e + ie);
  const double a3 = c.ratio * sh * sh;
  const double y = rcbrt_f64(a3), y2 = y * y, b = a3 * y2;
  const double b2 = b * b, low = fma(b, b, -b2);
  a = fma(fma(-low, b, fma(-b2, b, a3)), y2 * (1.0 / 3.0), b);
  inv_a = fma(y, fma(-a, y, 1.0), y);
  const double inv_a2 = inv_a * inv_a;
  // a^3 = ratio sh^2  =>  3 a^2 da/dt = -2 ratio sh ch rate
  adot = -(2.0 / 3.0) * rate * c.ratio * sh * ch * inv_a2;
}

// ---------------------------------------------------------------------------
// Geodesic right-hand side (Sec. 3.4, eq. geodesiceqn), Christoffel symbols
// differentiated exactly from eq. expandingmetric with psi = phi / a.  The
// z-form (x^3 as independent variable) integrates Y = (t, x, y, kt, kx, ky, kz).
// ---------------------------------------------------------------------------
struct State {
  double t, x, y, kt, kx, ky, kz;
};

// The contraction A^mu = Gamma^mu_ab k^a k^b at lookback time t for wave vector
// (kt, kx, ky, kz), comoving potential phi and gradient g; psi = phi / a(t).
__device__ __forceinline__ void accel(const DevCosmo& c, double t, double kt, double kx, double ky, double kz,
                                      double phi, double gx, double gy, double gz, double& psi, double& At,
                                      double& Ax, double& Ay, double& Az) {
  double a, inv_a, adot;
  scale_factor(c, t, a, inv_a, adot);
  psi = phi * inv_a;
  const double invE = recip_f64(fma(2.0, psi, 1.0));
  const double invF = recip_f64(fma(-2.0, phi, a)) * inv_a;   // 1 / (a^2 - 2 a phi)
  const double gk = gx * kx + gy * ky + gz * kz;
  const double k2 = kx * kx + ky * ky + kz * kz;
  const double kt2 = kt * kt;
  const double hub = adot * (a - phi);
  At = (-adot * psi * inv_a * kt2 + 2.0 * kt * inv_a * gk + hub * k2) * invE;
  const double c1 = kt2 * inv_a, c2 = 2.0 * hub * kt;
  Ax = (gx * c1 + c2 * kx + a * (gx * k2 - 2.0 * kx * gk)) * invF;
  Ay = (gy * c1 + c2 * ky + a * (gy * k2 - 2.0 * ky * gk)) * invF;
  Az = (gz * c1 + c2 * kz + a * (gz * k2 - 2.0 * kz * gk)) * invF;
}

// dY/dz = (dY/dlambda) / k^z.
__device__ __forceinline__ State rhs(const DevCosmo& c, const State& Y, double phi, double gx, double gy, double gz,
                                     double& psi) {
  double At, Ax, Ay, Az;
  accel(c, Y.t, Y.kt, Y.kx, Y.ky, Y.kz, phi, gx, gy, gz, psi, At, Ax, Ay, Az);
  const double iz = recip_f64(Y.kz);
  return State{Y.kt * iz, Y.kx * iz, Y.ky * iz, -At * iz, -Ax * iz, -Ay * iz, -Az * iz};
}

__device__ __forceinline__ State axpy(const State& Y, double h, const State& k) {
  return State{Y.t + h * k.t, Y.x + h * k.x, Y.y + h * k.y, Y.kt + h * k.kt, Y.kx + h * k.kx, Y.ky + h * k.ky,
               Y.kz + h * k.kz};
}

}  // namespace rt
