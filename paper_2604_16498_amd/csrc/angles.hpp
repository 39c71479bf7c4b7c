// cos and sin of the rotary embedding's angles.  Internal to the library; plain arithmetic, so that a host build of it
// can be checked over the whole range.
#pragma once
#include <math.h>

namespace forge {

// cos and sin of an angle 0 <= a < 2^31 in fp64: quadrant by two-part reduction (both products are
// exact in the fused multiply-add; what pi / 2 still lacks is below 1e-32 per turn), Taylor series up to
// x^15 / x^16 on [-pi/4, pi/4] (truncated below 1e-16).  Rounded to fp32 once, like the library call it stands
// for, which takes three times the registers and twice the instructions (for arguments that no position
// reaches).
__host__ __device__ inline void cos_sin(double a, float& cosine, float& sine) {
  const double n = rint(a * 0.63661977236758134308);                     // 2 / pi
  double x = __builtin_fma(n, -1.5707963267948966192, a);               // pi / 2 rounded to fp64 ...
  x = __builtin_fma(n, -6.123233995736766036e-17, x);                   // ... and what that rounding dropped
  const double z = x * x;
  double s = -1.0 / 1307674368000.0, c = 1.0 / 20922789888000.0;
  s = __builtin_fma(s, z, 1.0 / 6227020800.0);
  s = __builtin_fma(s, z, -1.0 / 39916800.0);
  s = __builtin_fma(s, z, 1.0 / 362880.0);
  s = __builtin_fma(s, z, -1.0 / 5040.0);
  s = __builtin_fma(s, z, 1.0 / 120.0);
  s = __builtin_fma(s, z, -1.0 / 6.0);
  s = __builtin_fma(s * z, x, x);
  c = __builtin_fma(c, z, -1.0 / 87178291200.0);
  c = __builtin_fma(c, z, 1.0 / 479001600.0);
  c = __builtin_fma(c, z, -1.0 / 3628800.0);
  c = __builtin_fma(c, z, 1.0 / 40320.0);
  c = __builtin_fma(c, z, -1.0 / 720.0);
  c = __builtin_fma(c, z, 1.0 / 24.0);
  c = __builtin_fma(c, z, -0.5);
  c = __builtin_fma(c, z, 1.0);
  const int q = (int)n & 3;
  const double co = (q & 1) ? s : c, si = (q & 1) ? c : s;
  cosine = (float)(q == 1 || q == 2 ? -co : co);
  sine = (float)(q >= 2 ? -si : si);
}

}  // namespace forge
