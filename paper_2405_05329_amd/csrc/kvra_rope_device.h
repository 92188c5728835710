// The angles of the rotary embedding, for the kernels that form them (not installed).
#ifndef KVRA_ROPE_DEVICE_H
#define KVRA_ROPE_DEVICE_H

#include "kvra_internal.h"

namespace kvra {

// cos and sin of phi, |phi| < 2^26, to about one unit in the last place of a double: phi - n pi/2 with pi/2 as a sum of two
// doubles (n has at most 26 bits, each fused multiply-add rounds once), then the Taylor series on [-pi/4, pi/4], whose
// first terms left out are below 2^-54.
__device__ __forceinline__ void sincos_reduced(double phi, double* s, double* c) {
  const double n = rint(phi * 0.63661977236758134308);
  double r = fma(-n, 1.57079632679489655800e+00, phi);
  r = fma(-n, 6.12323399573676603587e-17, r);
  const double z = r * r;
  double ps = 1.0 / 355687428096000.0, pc = -1.0 / 6402373705728000.0;   // 1/17!, -1/18!
  ps = fma(ps, z, -1.0 / 1307674368000.0);
  pc = fma(pc, z, 1.0 / 20922789888000.0);
  ps = fma(ps, z, 1.0 / 6227020800.0);
  pc = fma(pc, z, -1.0 / 87178291200.0);
  ps = fma(ps, z, -1.0 / 39916800.0);
  pc = fma(pc, z, 1.0 / 479001600.0);
  ps = fma(ps, z, 1.0 / 362880.0);
  pc = fma(pc, z, -1.0 / 3628800.0);
  ps = fma(ps, z, -1.0 / 5040.0);
  pc = fma(pc, z, 1.0 / 40320.0);
  ps = fma(ps, z, 1.0 / 120.0);
  pc = fma(pc, z, -1.0 / 720.0);
  ps = fma(ps, z, -1.0 / 6.0);
  pc = fma(pc, z, 1.0 / 24.0);
  pc = fma(pc, z, -0.5);
  ps = fma(ps * z, r, r);
  pc = fma(pc, z, 1.0);
  const int quadrant = static_cast<int>(n) & 3;
  const double s0 = quadrant & 1 ? pc : ps, c0 = quadrant & 1 ? ps : pc;
  *s = quadrant & 2 ? -s0 : s0;
  *c = quadrant == 1 || quadrant == 2 ? -c0 : c0;
}

// cos and sin of the angle position * base^(-2i/d), in fp64 (an fp32 angle would be off by ~1e-3 rad at position 32767).
__device__ __forceinline__ void rope_angle(double phi, float* cos_out, float* sin_out) {
  double s, c;
  if (phi < 67108864.0) sincos_reduced(phi, &s, &c);
  else sincos(phi, &s, &c);              // a rope base below 1
  *cos_out = static_cast<float>(c);
  *sin_out = static_cast<float>(s);
}

}  // namespace kvra

#endif
