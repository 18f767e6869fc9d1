// Scalar helpers of the triangle and vertex bodies.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace rd {

// Periodic difference: d shifted by one period into [-period/2, period/2]
// on a periodic axis. The half period is given: 0.5 period (exact) on a
// periodic axis, +inf on another (no difference exceeds it), so the
// comparisons read it where it is, with nothing to keep per thread.
__host__ __device__ inline double unwrap(double d, double period, double half) {
  if (d > half) d -= period;
  else if (d < -half) d += period;
  return d;
}

// The same value, selected rather than branched to (the forward triangle
// bodies: no basic-block boundaries between their loads and arithmetic).
__host__ __device__ inline double unwrap_select(double d, double period, double half) {
  const double hi = d - period, lo = d + period;
  return d > half ? hi : (d < -half ? lo : d);
}

// max / min of non-NaN values (one v_max / v_min instruction; the sign of a
// zero result is unspecified, which no result depends on).
template <typename R> __host__ __device__ inline R rmax(R a, R b) { return fmax(a, b); }
template <typename R> __host__ __device__ inline R rmin(R a, R b) { return fmin(a, b); }

// One third-order step from the hardware approximation r0 of 1 / x, whose
// relative error e (about 2^-24) it takes to e^3: r0 (1 + e + e^2), e = 1 - x r0.
__host__ __device__ inline double rcp_step(double x, double r0) {
  const double e = fma(-x, r0, 1.0);
  return fma(r0, fma(e, e, e), r0);
}

// The same for 1 / sqrt(x): y0 (1 + e / 2 + 3 e^2 / 8), e = 1 - x y0^2.
__host__ __device__ inline double rsq_step(double x, double y0) {
  const double e = fma(-(x * y0), y0, 1.0);
  return fma(y0 * e, fma(0.375, e, 0.5), y0);
}

// Reciprocal within about an ulp of 1 / x; where the step is not finite (x
// zero or infinite, or so small that 1 / x overflows) the hardware value.
__host__ __device__ inline double rcp(double x) {
#ifdef __HIP_DEVICE_COMPILE__
  const double r0 = __builtin_amdgcn_rcp(x), r = rcp_step(x, r0);
  return r == r ? r : r0;
#else
  return 1.0 / x;
#endif
}

// Reciprocal of a positive normal x whose reciprocal is normal too: as rcp
// without its fallback.
__host__ __device__ inline double rcp_normal(double x) {
#ifdef __HIP_DEVICE_COMPILE__
  return rcp_step(x, __builtin_amdgcn_rcp(x));
#else
  return 1.0 / x;
#endif
}

// Length L = sqrt(e2) > 0 and its reciprocal (e2 is a squared edge length or
// the squared sound speed of a Roe state, positive and finite), each within
// about an ulp or two: iL from the hardware reciprocal square root, L = e2 iL.
__host__ __device__ inline void len_rcp(double e2, double& L, double& iL) {
#ifdef __HIP_DEVICE_COMPILE__
  iL = rsq_step(e2, __builtin_amdgcn_rsq(e2));
  L = e2 * iL;
#else
  L = sqrt(e2);
  iL = 1.0 / L;
#endif
}

}  // namespace rd
