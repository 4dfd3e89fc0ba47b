"""The device code of the background (csrc/rt_geodesic.h) compiled for the CPU, with the hardware's estimates
replaced by their exact values off by as much as their stated error: a(t) and 1/a keep the rounding of a
correctly rounded cube root and division.

Bounds, relative: a ends in one rounding, at most 2^-53, of a correction whose own error is of second order (2^-100);
1/a takes a's error and one rounding more."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdio>
#include <random>
#include <quadmath.h>
#undef __device__
#undef __forceinline__
#define __device__
#define __forceinline__ inline
using std::exp;
using std::fma;
static std::mt19937_64 gen(7);
static double off(double rel) { return 1.0 + rel * std::uniform_real_distribution<double>(-1.0, 1.0)(gen); }
static double rcp_estimate(double x) { return (double)(float)(1.0 / x * off(0x1p-24)); }
static float log2_estimate(float x) { return (float)(std::log2((double)x) * off(0x1p-23)); }
static float exp2_estimate(float x) { return (float)(std::exp2((double)x) * off(0x1p-23)); }
#define __builtin_amdgcn_rcp rcp_estimate
#define __builtin_amdgcn_logf log2_estimate
#define __builtin_amdgcn_exp2f exp2_estimate
#include "rt_geodesic.h"

int main() {
  const double om = 0.3, ol = 0.7;
  rt::DevCosmo c{};
  c.H0 = 70.0 / 299792.458;
  c.sqrt_ol = std::sqrt(ol);
  c.ratio = om / ol;
  c.t0 = 2.0 / (3.0 * c.H0 * c.sqrt_ol) * std::asinh(std::sqrt(ol / om));
  double worst[3] = {0.0, 0.0, 0.0};
  for (int i = 0; i < 200000; ++i) {
    const double t = c.t0 * std::uniform_real_distribution<double>(0.0, 0.999)(gen);
    double a, inv_a, adot;
    const std::mt19937_64 before = gen;
    rt::scale_factor(c, t, a, inv_a, adot);
    const std::mt19937_64 after = gen;
    gen = before;   // the same estimate of exp(-u)
    const double e = exp(1.5 * c.sqrt_ol * c.H0 * (c.t0 - t)), ie = rt::recip_f64(e), sh = 0.5 * (e - ie);
    gen = after;
    const double a3 = c.ratio * sh * sh;
    const __float128 root = cbrtq((__float128)a3);
    worst[0] = std::fmax(worst[0], (double)(fabsq((__float128)a - root) / root) * 0x1p53);
    worst[1] = std::fmax(worst[1], (double)fabsq((__float128)inv_a * root - 1) * 0x1p53);
    worst[2] = std::fmax(worst[2], (double)fabsq((__float128)ie * (__float128)e - 1) * 0x1p53);
  }
  std::printf("%.6f %.6f %.6f\n", worst[0], worst[1], worst[2]);
  return 0;
}
"""


def test_scale_factor_is_rounded_once(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("no g++ or no HIP headers")
    src, exe = tmp_path / "rounding.cpp", tmp_path / "rounding"
    src.write_text(SOURCE)
    subprocess.run([gxx, "-O1", "-std=gnu++17", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_1110_4894_amd", "csrc"), str(src), "-o", str(exe), "-lquadmath"],
                   check=True)
    a, inv_a, recip = map(float, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert a <= 1.001
    assert inv_a <= 2.001
    assert recip <= 1.001
