// FP64 helpers of the Green's function and plane-wave kernels (device inline).
#pragma once
#include <hip/hip_runtime.h>

namespace r3m {

// 1 / sqrt(x) for x > 0: the hardware estimate and one cubic step
__device__ __forceinline__ double rsqrt64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// cos and sin of x by reduction to |r| <= pi / 4 (one fused product with
// pi / 2 to 53 bits and its remainder) and the Taylor series to r^16 and r^15
// (truncation below 5e-18 and 5e-17); without the large-argument path of the
// library function, which its callers' accuracy does not need (x is a phase
// k r below some thousand radians, rounded to |x| 2^-53 itself)
__device__ __forceinline__ void cos_sin(double x, double& c, double& s) {
  const double n = rint(x * 0.63661977236758134);
  double r = fma(-n, 1.5707963267948966, x);
  r = fma(-n, 6.123233995736766e-17, r);
  const double z = r * r;
  double ps = -1.0 / 1307674368000.0;  // -1 / 15!
  ps = fma(ps, z, 1.0 / 6227020800.0);
  ps = fma(ps, z, -1.0 / 39916800.0);
  ps = fma(ps, z, 1.0 / 362880.0);
  ps = fma(ps, z, -1.0 / 5040.0);
  ps = fma(ps, z, 1.0 / 120.0);
  ps = fma(ps, z, -1.0 / 6.0);
  const double sr = fma(r * z, ps, r);
  double pc = 1.0 / 20922789888000.0;  // 1 / 16!
  pc = fma(pc, z, -1.0 / 87178291200.0);
  pc = fma(pc, z, 1.0 / 479001600.0);
  pc = fma(pc, z, -1.0 / 3628800.0);
  pc = fma(pc, z, 1.0 / 40320.0);
  pc = fma(pc, z, -1.0 / 720.0);
  pc = fma(pc, z, 1.0 / 24.0);
  const double cr = fma(z * z, pc, fma(z, -0.5, 1.0));
  const int q = (int)fma(-4.0, rint(0.25 * n), n);  // quadrant, -2 .. 2
  const bool swap = q & 1;
  const double a = swap ? sr : cr, b = swap ? cr : sr;
  c = (q + 1) & 2 ? -a : a;
  s = q & 2 ? -b : b;
}

}  // namespace r3m
