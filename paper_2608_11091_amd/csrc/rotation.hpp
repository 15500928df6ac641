// Scalars of the Jacobi rotations, from the hardware's approximations of
// reciprocal and reciprocal root (1 ulp in FP32, about 24 bits in FP64).
#pragma once

namespace tk {

// 1 / sqrt(x) to working accuracy: the approximation and one step, of third
// order in FP64.  The FP32 step matters: an error of the root is common to a
// whole column and reaches the result once a mode (200 RoundSums of ranks 3 to
// 12: mean error against 64 bits 3-8% below the rotated vectors of a two-sided
// sweep with it, above without).
__device__ __forceinline__ float rsq_full(float x) {
  const float y = __builtin_amdgcn_rsqf(x), h = x * y;
  const float e = fmaf(-fmaf(x, y, -h), y, fmaf(-h, y, 1.0f));
  return fmaf(0.5f * y, e, y);
}
__device__ __forceinline__ double rsq_full(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// Tangent of the rotation that makes columns with dot product d and squared
// norms nx, ny orthogonal: t = sign(z) / (|z| + sqrt(1 + z^2)), z = (ny - nx) / 2d.
// FP64 forms it to working accuracy (what an inexact angle leaves of the product
// it annihilates would need a tighter stop, that is another sweep), as
// sign(g) 2d / (|g| + sqrt(g^2 + 4 d^2)) with g = ny - nx: the reciprocal of 2d
// would cost four instructions more, and a step's time is its instructions (as
// would a branch for small operands: columns are scaled so that squares of
// their products stay in range).  FP32 takes the root of a z bounded against
// overflow: it is |z| itself long before the bound.
__device__ __forceinline__ float jac_tan(float d, float nx, float ny) {
  const float z = (ny - nx) * __builtin_amdgcn_rcpf(d + d);
  const float az = fabsf(z);
  const float q = fminf(az, 1e18f);
  const float w = fmaf(q, q, 1.0f);
  return copysignf(__builtin_amdgcn_rcpf(az + fmaxf(w * __builtin_amdgcn_rsqf(w), az)), z);
}
__device__ __forceinline__ double jac_tan(double d, double nx, double ny) {
  const double g = ny - nx, e = d + d;
  const double w = fma(g, g, e * e);
  const double v = __builtin_amdgcn_rsq(w);
  const double h0 = w * v, f = fma(-h0, v, 1.0);
  const double h = fma(h0 * f, fma(0.375, f, 0.5), h0);  // sqrt(w)
  const double D = fabs(g) + h;
  const double y = __builtin_amdgcn_rcp(D);
  const double t0 = e * y, r = fma(-D, y, 1.0);
  const double t = fma(t0, fma(r, r, r), t0);
  return g < 0.0 ? -t : t;
}
// Exponent that the squared norms of columns with a trace of at most 1 are
// scaled by (even): with it, squares of dot products of columns down to 1e-150
// of the largest are normal numbers, and none overflows.
template <typename T>
constexpr int kJacExp = sizeof(T) == 8 ? 508 : 0;

}  // namespace tk
