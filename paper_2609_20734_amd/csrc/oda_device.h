// Device helpers shared by the library's kernels (HIP translation units only).
#ifndef ODA_DEVICE_H_
#define ODA_DEVICE_H_

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace oda {

// fp32 -> bf16, round to nearest, ties to even (NaN stays NaN, quietened).
__device__ __forceinline__ uint16_t bf16_rne(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// Orders a wavefront's shared-memory stores before the loads of its other lanes
// that follow, and these before the next stores, where a wavefront alone uses
// its part of LDS.  The hardware keeps one wavefront's LDS operations in order;
// this tells the compiler that the lanes communicate.  No instruction.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Rotary frequency of dims i and i + D/2 (lane i): theta^(-2i/D), from
// log2(theta) formed on the host.  Rounding the exponent, as large as
// log2(theta), makes a relative error of up to about log2(theta) 2^-53 (worst
// lane 2^-49.8 at theta = 10^6, 2^-48.8 at 10^8): at position 10^6 the angle is
// off by 2^-28 at most, far below the float that its sine and cosine become.
__device__ __forceinline__ double rope_frequency(int lane, int D, double log2_theta) {
  return exp2(-(double)(2 * lane) / (double)D * log2_theta);
}

// sin and cos of an angle up to 2^31 in double: the nearest multiple of pi/2
// is taken off in two fused steps (pi/2 as two doubles, 107 bits), then the
// Taylor series on |r| <= pi/4 up to r^15 and r^16 (truncation below 2^-54).
// Straight-line code of about 60 instructions: the library's functions, whose
// code covers every argument, cost a fused one-layer call 0.7 us more, in
// instruction fetches (Local of one request 11.3 us against 10.7).
__device__ __forceinline__ void sincos_angle(double x, double& s, double& c) {
  const double q = rint(x * 0.63661977236758134308);   // 2 / pi
  double r = fma(-q, 1.57079632679489655800, x);
  r = fma(-q, 6.12323399573676603587e-17, r);
  const double r2 = r * r;
  double ps = -1.0 / 1307674368000.0;                  // 15!
  ps = fma(ps, r2, 1.0 / 6227020800.0);
  ps = fma(ps, r2, -1.0 / 39916800.0);
  ps = fma(ps, r2, 1.0 / 362880.0);
  ps = fma(ps, r2, -1.0 / 5040.0);
  ps = fma(ps, r2, 1.0 / 120.0);
  ps = fma(ps, r2, -1.0 / 6.0);
  const double sr = fma(ps * r2, r, r);
  double pc = 1.0 / 20922789888000.0;                  // 16!
  pc = fma(pc, r2, -1.0 / 87178291200.0);
  pc = fma(pc, r2, 1.0 / 479001600.0);
  pc = fma(pc, r2, -1.0 / 3628800.0);
  pc = fma(pc, r2, 1.0 / 40320.0);
  pc = fma(pc, r2, -1.0 / 720.0);
  pc = fma(pc, r2, 1.0 / 24.0);
  pc = fma(pc, r2, -0.5);
  const double cr = fma(pc, r2, 1.0);
  const int k = (int)(int64_t)q & 3;
  s = (k & 1) ? cr : sr;
  c = (k & 1) ? sr : cr;
  if (k & 2) s = -s;
  if (k == 1 || k == 2) c = -c;
}

// Current-token preparation of one q or k head, one wavefront per head: lane
// i < D/2 holds the pair (x_i, x_{i+D/2}) that the rotation mixes
// (rotate-half convention).  In two parts, so that a caller can run the first
// while the position is still on its way: the per-head RMSNorm with `gain`
// (skipped when NULL; every lane takes part in the sum, the inactive ones
// adding zeros, so it is whole for any D/2 up to 64; called by every lane of
// the wavefront), then the rotary embedding at position `pos`: dims i and
// i + D/2 turn by pos * frequency, the angle formed in double precision since
// positions reach 10^5-10^6.
__device__ __forceinline__ void head_norm(float& x1, float& x2, bool active, int lane, int D, const float* gain,
                                          float eps) {
  if (gain == nullptr) return;
  const int half = D / 2;
  float ss = x1 * x1 + x2 * x2;
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) ss += __shfl_xor(ss, s);
  const float inv = rsqrtf(ss / (float)D + eps);
  if (active) {
    x1 = x1 * inv * gain[lane];
    x2 = x2 * inv * gain[lane + half];
  }
}
__device__ __forceinline__ void rotate_pair(float& x1, float& x2, double pos, double frequency) {
  double sd, cd;
  sincos_angle(pos * frequency, sd, cd);
  const float c = (float)cd, s = (float)sd;
  const float r1 = x1 * c - x2 * s;
  const float r2 = x2 * c + x1 * s;
  x1 = r1;
  x2 = r2;
}

}  // namespace oda

#endif  // ODA_DEVICE_H_
