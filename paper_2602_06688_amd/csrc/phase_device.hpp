// phase_device.hpp -- sine and cosine of an optical phase.
#pragma once

#include <hip/hip_runtime.h>

namespace pwfs {

// sin and cos of t quarter turns (t = 4 OPD / lambda in float64): the quarter
// turn nearest to t leaves at most pi / 4, whose Taylor series to x^9 and x^10
// end below 3e-9.  Worst error 9.7e-8, rms 2.0e-8 (reduction to [-pi, pi] and
// the library's float32 functions: 1.3e-7 and 3.6e-8), no branch, and the
// instructions of several calls interleave.  Not finite: NaN.
__device__ __forceinline__ void sincos_quarters(double t, float& sn, float& cs) {
  const double k = rint(t), k4 = 0.25 * k;
  const int q = (int)(4.0 * (k4 - rint(k4)));   // k mod 4, in -2 .. 2
  const float x = (float)(t - k) * 1.57079632679489662f, z = x * x;
  float s = fmaf(z, 2.75573192e-6f, -1.98412698e-4f);
  s = fmaf(z, s, 8.33333333e-3f);
  s = fmaf(z, s, -1.66666667e-1f);
  s = fmaf(x * z, s, x);
  float c = fmaf(z, -2.75573192e-7f, 2.48015873e-5f);
  c = fmaf(z, c, -1.38888889e-3f);
  c = fmaf(z, c, 4.16666667e-2f);
  c = fmaf(z, c, -0.5f);
  c = fmaf(z, c, 1.f);
  const float a = (q & 1) ? c : s, b = (q & 1) ? s : c;
  sn = (q & 2) ? -a : a;
  cs = ((q + 1) & 2) ? -b : b;
}

}  // namespace pwfs
