"""The FP64 Jacobi rotation carries working accuracy: the scalar functions of
csrc/rotation.hpp are compiled for the host, with the hardware's approximations
of reciprocal and reciprocal root replaced by correctly rounded values cut to 23
bits, and compared with extended precision over products from 1e-16 to 1 of the
norms and squared norms, scaled as the solver scales them, from 1 down to
1e-270.  Each quotient, root and product rounds once: 8 ulp asserted for the
tangent, 4 for the cosine and for how far cosine and sine are from a unit
vector, 2 for 1 / sqrt(x).  Equal norms take either sign."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2608_11091_amd", "csrc")

HOST = r"""
#include <cmath>
#include <cstdio>
#include <random>
#define __device__
#define __forceinline__ inline
static double cut(double x) {
  int e;
  const double m = std::frexp(x, &e);
  return std::ldexp(std::floor(std::ldexp(m, 23)), e - 23);
}
static double __builtin_amdgcn_rcp(double x) { return cut(1.0 / x); }
static double __builtin_amdgcn_rsq(double x) { return cut(1.0 / std::sqrt(x)); }
static float __builtin_amdgcn_rcpf(float x) { return 1.0f / x; }
static float __builtin_amdgcn_rsqf(float x) { return float(1.0 / std::sqrt(double(x))); }
#include "rotation.hpp"
int main() {
  std::mt19937_64 g(7);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  double et = 0.0, er = 0.0, co = 0.0, un = 0.0;
  const double ulp = std::ldexp(1.0, -52);
  for (int i = 0; i < 400000; ++i) {
    const double nx = std::ldexp(std::pow(10.0, -135.0 * u(g) * (i & 1)), tk::kJacExp<double>), ny = nx * std::pow(10.0, -135.0 * u(g) * (i & 2) / 2);
    double a = nx, b = ny;
    if (i & 4) std::swap(a, b);
    if (i % 97 == 0) b = a;
    const double d = std::sqrt(a) * std::sqrt(b) * std::pow(10.0, -16.0 * u(g)) * (i & 8 ? -1.0 : 1.0);
    const double t = tk::jac_tan(d, a, b), c = tk::rsq_full(std::fma(t, t, 1.0));
    // (the difference of the norms is an input here: FP64 rounds it once)
    const long double z = (long double)(b - a) / (2.0L * d);
    const long double ref = (std::signbit(z) ? -1.0L : 1.0L) / (fabsl(z) + sqrtl(1.0L + z * z));
    et = std::fmax(et, double(fabsl((b == a ? std::fabs(t) : t) / (b == a ? 1.0L : ref) - 1.0L)) / ulp);
    co = std::fmax(co, double(fabsl(c * sqrtl(1.0L + ref * ref) - 1.0L)) / ulp);
    const double s = t * c;
    un = std::fmax(un, double(fabsl((long double)c * c + (long double)s * s - 1.0L)) / ulp);
    const double x = std::pow(10.0, 300.0 * (u(g) - 0.5));
    er = std::fmax(er, double(fabsl(tk::rsq_full(x) * sqrtl((long double)x) - 1.0L)) / ulp);
  }
  std::printf("%.3f %.3f %.3f %.3f\n", et, co, un, er);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_rotation_has_working_accuracy(tmp_path):
    src, exe = tmp_path / "rot.cpp", tmp_path / "rot"
    src.write_text(HOST)
    subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    tan, cos, unit, rsq = (float(x) for x in out.split())
    print(f"tangent {tan} ulp, cosine {cos}, unit vector {unit}, reciprocal root {rsq}", flush=True)
    assert tan <= 8.0 and cos <= 4.0 and unit <= 4.0 and rsq <= 2.0
