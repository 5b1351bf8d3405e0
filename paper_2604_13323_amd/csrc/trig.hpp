// FP64 sine and cosine from a table in LDS, and where the leaf-to-root walks take them from.
#pragma once

#include "common.hpp"

namespace mc {

// Sine and cosine of k pi / 32, k = 0 .. 63 (correctly rounded).
constexpr double kSinTab[64][2] = {
    {0.0, 1.0}, {0.0980171403295606, 0.9951847266721969},
    {0.19509032201612828, 0.9807852804032304}, {0.2902846772544624, 0.9569403357322088},
    {0.3826834323650898, 0.9238795325112867}, {0.47139673682599764, 0.881921264348355},
    {0.5555702330196022, 0.8314696123025452}, {0.6343932841636455, 0.773010453362737},
    {0.7071067811865476, 0.7071067811865476}, {0.773010453362737, 0.6343932841636455},
    {0.8314696123025452, 0.5555702330196022}, {0.881921264348355, 0.47139673682599764},
    {0.9238795325112867, 0.3826834323650898}, {0.9569403357322088, 0.2902846772544624},
    {0.9807852804032304, 0.19509032201612828}, {0.9951847266721969, 0.0980171403295606},
    {1.0, 0.0}, {0.9951847266721969, -0.0980171403295606},
    {0.9807852804032304, -0.19509032201612828}, {0.9569403357322088, -0.2902846772544624},
    {0.9238795325112867, -0.3826834323650898}, {0.881921264348355, -0.47139673682599764},
    {0.8314696123025452, -0.5555702330196022}, {0.773010453362737, -0.6343932841636455},
    {0.7071067811865476, -0.7071067811865476}, {0.6343932841636455, -0.773010453362737},
    {0.5555702330196022, -0.8314696123025452}, {0.47139673682599764, -0.881921264348355},
    {0.3826834323650898, -0.9238795325112867}, {0.2902846772544624, -0.9569403357322088},
    {0.19509032201612828, -0.9807852804032304}, {0.0980171403295606, -0.9951847266721969},
    {0.0, -1.0}, {-0.0980171403295606, -0.9951847266721969},
    {-0.19509032201612828, -0.9807852804032304}, {-0.2902846772544624, -0.9569403357322088},
    {-0.3826834323650898, -0.9238795325112867}, {-0.47139673682599764, -0.881921264348355},
    {-0.5555702330196022, -0.8314696123025452}, {-0.6343932841636455, -0.773010453362737},
    {-0.7071067811865476, -0.7071067811865476}, {-0.773010453362737, -0.6343932841636455},
    {-0.8314696123025452, -0.5555702330196022}, {-0.881921264348355, -0.47139673682599764},
    {-0.9238795325112867, -0.3826834323650898}, {-0.9569403357322088, -0.2902846772544624},
    {-0.9807852804032304, -0.19509032201612828}, {-0.9951847266721969, -0.0980171403295606},
    {-1.0, 0.0}, {-0.9951847266721969, 0.0980171403295606},
    {-0.9807852804032304, 0.19509032201612828}, {-0.9569403357322088, 0.2902846772544624},
    {-0.9238795325112867, 0.3826834323650898}, {-0.881921264348355, 0.47139673682599764},
    {-0.8314696123025452, 0.5555702330196022}, {-0.773010453362737, 0.6343932841636455},
    {-0.7071067811865476, 0.7071067811865476}, {-0.6343932841636455, 0.773010453362737},
    {-0.5555702330196022, 0.8314696123025452}, {-0.47139673682599764, 0.881921264348355},
    {-0.3826834323650898, 0.9238795325112867}, {-0.2902846772544624, 0.9569403357322088},
    {-0.19509032201612828, 0.9807852804032304}, {-0.0980171403295606, 0.9951847266721969},};
constexpr int kSinTabDoubles = 128;

// The table staged in LDS by the whole block (the caller synchronises).
__device__ __forceinline__ void stage_sin_tab(double* lds) {
  for (int i = threadIdx.x; i < 64; i += blockDim.x) {
    lds[2 * i] = kSinTab[i][0];
    lds[2 * i + 1] = kSinTab[i][1];
  }
}

using SinTabP = const __attribute__((address_space(3))) double*;

// FP64 sine and cosine by the table: x = k pi/32 + r with pi/32 split into two doubles, |r| <= pi/64,
// the Taylor series of sin r (to r^7) and cos r - 1 (to r^8), whose truncation errors are below 5e-18,
// and the angle sum. 21 operations and one 16-byte LDS read, against 35 for the reduction to pi/4 with
// its series to r^15 and r^16.
// In two parts, so that other work can stand between the read and its use: the entry (and k), then the rest.
using SinTabV = double __attribute__((ext_vector_type(2)));
// x 32/pi is rounded to the whole number k by adding 1.5 2^52, whose low bits are then k's (|k| < 2^51; a conversion to 32
// bits ended at |x| = 2.1e8).
__host__ __device__ __forceinline__ int sin_tab_index(double x, double& k) {
  const double t = __builtin_fma(x, 10.185916357881302, 6755399441055744.0);
  k = t - 6755399441055744.0;
  return int(__builtin_bit_cast(uint64_t, t)) & 63;
}
__device__ __forceinline__ SinTabV sin_tab_entry(double x, SinTabP tab, double& k) {
  return *(const __attribute__((address_space(3))) SinTabV*)(tab + 2 * sin_tab_index(x, k));
}
__host__ __device__ __forceinline__ void sincos_finish(double x, double k, SinTabV t, double& s, double& c) {
  double r = __builtin_fma(-k, 0.09817477042468103, x);
  r = __builtin_fma(-k, 3.827021247335479e-18, r);
  const double r2 = r * r;
  double ps = __builtin_fma(r2, -1.0 / 5040.0, 1.0 / 120.0);
  double pc = __builtin_fma(r2, 1.0 / 40320.0, -1.0 / 720.0);
  ps = __builtin_fma(r2, ps, -1.0 / 6.0);
  pc = __builtin_fma(r2, pc, 1.0 / 24.0);
  const double sr = __builtin_fma(r * r2, ps, r);
  pc = __builtin_fma(r2, pc, -0.5);
  const double cm = r2 * pc;
  s = __builtin_fma(t.y, sr, __builtin_fma(t.x, cm, t.x));
  c = __builtin_fma(-t.x, sr, __builtin_fma(t.y, cm, t.y));
}
__device__ __forceinline__ void sincos_tab(double x, SinTabP tab, double& s, double& c) {
  double k;
  const SinTabV t = sin_tab_entry(x, tab, k);
  sincos_finish(x, k, t, s, c);
}

// Where the walks take sines and cosines from. TrigLive: computed from the iterate in every pass.
// TrigTile: the residual pass stores them, rounded to FP32, in a per-lane column of a [D][64] LDS tile
// (a prismatic joint's slot holds its coordinate) and the FP32 step passes read them there.
// fresh(): the same source for another pass, whose reads the compiler cannot merge with an earlier pass's (it would
// keep every value in registers in between).
struct TrigLive {
  static constexpr bool tile = false;
  SinTabP tab;
  __device__ __forceinline__ TrigLive fresh() const { return *this; }
};
struct TrigTile {
  static constexpr bool tile = true;
  using V2 = float __attribute__((ext_vector_type(2)));
  using LP = __attribute__((address_space(3))) V2*;
  SinTabP tab;
  LP base;
  __device__ __forceinline__ void set(int j, float a, float b) const {
    V2 v;
    v.x = a;
    v.y = b;
    base[j * 64] = v;
  }
  __device__ __forceinline__ V2 get(int j) const { return base[j * 64]; }
  __device__ __forceinline__ TrigTile fresh() const {
    TrigTile t = *this;
    asm volatile("" : "+v"(t.base));
    return t;
  }
};

}  // namespace mc
