// Rotary position embedding of one row, shared by the kernels that rotate: dimension i < d / 2 pairs with
// i + d / 2 and the pair is turned by pos * theta^(-2i/d).  Angles are evaluated in double
// precision, because pos * frequency reaches 1e6 rad and fp32 cannot hold its fractional turn;
// the rotation runs in fp32, with one rounding to the storage type behind it.
#pragma once

#include "star_internal.h"

namespace star {

// theta^(-2i/d), and cos and sin of pos times that
__device__ __forceinline__ double rotary_frequency(int i, int d, double log2_theta) {
  return exp2(-2.0 * (double)i / (double)d * log2_theta);
}
// Taylor sums to x^17 and x^16: for |x| <= pi / 4 what they leave out is below 1e-17, so that their own roundings
// (2^-52) are all that is lost.  (To x^13 and x^14 3e-14 was; a rotated decode call takes as long either way.)
__host__ __device__ __forceinline__ void rotary_sin_cos(double x, double* sine, double* cosine) {
  const double z = x * x;
  double s = 1.0 / 355687428096000.0, c = 1.0 / 20922789888000.0;
  s = fma(s, z, -1.0 / 1307674368000.0);
  s = fma(s, z, 1.0 / 6227020800.0);
  s = fma(s, z, -1.0 / 39916800.0);
  s = fma(s, z, 1.0 / 362880.0);
  s = fma(s, z, -1.0 / 5040.0);
  s = fma(s, z, 1.0 / 120.0);
  s = fma(s, z, -1.0 / 6.0);
  *sine = fma(s * z, x, x);
  c = fma(c, z, -1.0 / 87178291200.0);
  c = fma(c, z, 1.0 / 479001600.0);
  c = fma(c, z, -1.0 / 3628800.0);
  c = fma(c, z, 1.0 / 40320.0);
  c = fma(c, z, -1.0 / 720.0);
  c = fma(c, z, 1.0 / 24.0);
  c = fma(c, z, -0.5);
  *cosine = fma(c, z, 1.0);
}
// Quarter turns are taken off: the results are the rounded cosine and sine but for ties.
__device__ __forceinline__ void rotary_angle(int64_t pos, double inv_freq, float* cs, float* sn) {
  const double TWO_PI = 6.283185307179586476925, INV_TWO_PI = 0.1591549430918953357689;
  const double HALF_PI = 1.570796326794896619231, INV_HALF_PI = 0.6366197723675813430755;
  const double ang = (double)pos * inv_freq;
  const double r = fma(-rint(ang * INV_TWO_PI), TWO_PI, ang);     // |r| <= pi
  const double n = rint(r * INV_HALF_PI);
  double s, c;
  rotary_sin_cos(fma(-n, HALF_PI, r), &s, &c);
  const int q = (int)n;
  const float fs = (float)(q & 1 ? c : s), fc = (float)(q & 1 ? s : c);
  *sn = q & 2 ? -fs : fs;
  *cs = (q + 1) & 2 ? -fc : fc;
}

// The pair (x, y) of dimensions i and i + d / 2.  Written out as it is rounded, so that every kernel
// gives the same bits.
__device__ __forceinline__ float rotary_lo(float x, float y, float cs, float sn) { return fmaf(x, cs, -(y * sn)); }
__device__ __forceinline__ float rotary_hi(float x, float y, float cs, float sn) { return fmaf(x, sn, y * cs); }

}  // namespace star
