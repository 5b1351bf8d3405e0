// FP64 sine and cosine from a table in LDS, and where the leaf-to-root walks take them from.
#pragma once

#include "common.hpp"

namespace mc {

// Sine and cosine of k pi / 32, k = 0 .. 63, rounded to double, and what the rounding left of each.
constexpr double kSinTab[64][4] = {
    {0.0, 1.0, 0.0, 0.0},
    {0.0980171403295606, 0.9951847266721969, -1.634582362244256e-18, -4.248691367830441e-17},
    {0.19509032201612828, 0.9807852804032304, -7.991079068461731e-18, 1.8546939997825006e-17},
    {0.2902846772544624, 0.9569403357322088, -1.892797870777425e-17, 4.05538698618757e-17},
    {0.3826834323650898, 0.9238795325112867, -1.0050772696461588e-17, 1.7645047084336677e-17},
    {0.47139673682599764, 0.881921264348355, 6.516678136069013e-18, -1.9843248405890562e-17},
    {0.5555702330196022, 0.8314696123025452, 4.709410940561677e-17, 1.4073856984728024e-18},
    {0.6343932841636455, 0.773010453362737, 1.0420901929280035e-17, -3.256590703364977e-17},
    {0.7071067811865476, 0.7071067811865476, -4.833646656726457e-17, -4.833646656726457e-17},
    {0.773010453362737, 0.6343932841636455, -3.256590703364977e-17, 1.0420901929280035e-17},
    {0.8314696123025452, 0.5555702330196022, 1.4073856984728024e-18, 4.709410940561677e-17},
    {0.881921264348355, 0.47139673682599764, -1.9843248405890562e-17, 6.516678136069013e-18},
    {0.9238795325112867, 0.3826834323650898, 1.7645047084336677e-17, -1.0050772696461588e-17},
    {0.9569403357322088, 0.2902846772544624, 4.05538698618757e-17, -1.892797870777425e-17},
    {0.9807852804032304, 0.19509032201612828, 1.8546939997825006e-17, -7.991079068461731e-18},
    {0.9951847266721969, 0.0980171403295606, -4.248691367830441e-17, -1.634582362244256e-18},
    {1.0, 0.0, 0.0, 0.0},
    {0.9951847266721969, -0.0980171403295606, -4.248691367830441e-17, 1.634582362244256e-18},
    {0.9807852804032304, -0.19509032201612828, 1.8546939997825006e-17, 7.991079068461731e-18},
    {0.9569403357322088, -0.2902846772544624, 4.05538698618757e-17, 1.892797870777425e-17},
    {0.9238795325112867, -0.3826834323650898, 1.7645047084336677e-17, 1.0050772696461588e-17},
    {0.881921264348355, -0.47139673682599764, -1.9843248405890562e-17, -6.516678136069013e-18},
    {0.8314696123025452, -0.5555702330196022, 1.4073856984728024e-18, -4.709410940561677e-17},
    {0.773010453362737, -0.6343932841636455, -3.256590703364977e-17, -1.0420901929280035e-17},
    {0.7071067811865476, -0.7071067811865476, -4.833646656726457e-17, 4.833646656726457e-17},
    {0.6343932841636455, -0.773010453362737, 1.0420901929280035e-17, 3.256590703364977e-17},
    {0.5555702330196022, -0.8314696123025452, 4.709410940561677e-17, -1.4073856984728024e-18},
    {0.47139673682599764, -0.881921264348355, 6.516678136069013e-18, 1.9843248405890562e-17},
    {0.3826834323650898, -0.9238795325112867, -1.0050772696461588e-17, -1.7645047084336677e-17},
    {0.2902846772544624, -0.9569403357322088, -1.892797870777425e-17, -4.05538698618757e-17},
    {0.19509032201612828, -0.9807852804032304, -7.991079068461731e-18, -1.8546939997825006e-17},
    {0.0980171403295606, -0.9951847266721969, -1.634582362244256e-18, 4.248691367830441e-17},
    {0.0, -1.0, 0.0, 0.0},
    {-0.0980171403295606, -0.9951847266721969, 1.634582362244256e-18, 4.248691367830441e-17},
    {-0.19509032201612828, -0.9807852804032304, 7.991079068461731e-18, -1.8546939997825006e-17},
    {-0.2902846772544624, -0.9569403357322088, 1.892797870777425e-17, -4.05538698618757e-17},
    {-0.3826834323650898, -0.9238795325112867, 1.0050772696461588e-17, -1.7645047084336677e-17},
    {-0.47139673682599764, -0.881921264348355, -6.516678136069013e-18, 1.9843248405890562e-17},
    {-0.5555702330196022, -0.8314696123025452, -4.709410940561677e-17, -1.4073856984728024e-18},
    {-0.6343932841636455, -0.773010453362737, -1.0420901929280035e-17, 3.256590703364977e-17},
    {-0.7071067811865476, -0.7071067811865476, 4.833646656726457e-17, 4.833646656726457e-17},
    {-0.773010453362737, -0.6343932841636455, 3.256590703364977e-17, -1.0420901929280035e-17},
    {-0.8314696123025452, -0.5555702330196022, -1.4073856984728024e-18, -4.709410940561677e-17},
    {-0.881921264348355, -0.47139673682599764, 1.9843248405890562e-17, -6.516678136069013e-18},
    {-0.9238795325112867, -0.3826834323650898, -1.7645047084336677e-17, 1.0050772696461588e-17},
    {-0.9569403357322088, -0.2902846772544624, -4.05538698618757e-17, 1.892797870777425e-17},
    {-0.9807852804032304, -0.19509032201612828, -1.8546939997825006e-17, 7.991079068461731e-18},
    {-0.9951847266721969, -0.0980171403295606, 4.248691367830441e-17, 1.634582362244256e-18},
    {-1.0, 0.0, 0.0, 0.0},
    {-0.9951847266721969, 0.0980171403295606, 4.248691367830441e-17, -1.634582362244256e-18},
    {-0.9807852804032304, 0.19509032201612828, -1.8546939997825006e-17, -7.991079068461731e-18},
    {-0.9569403357322088, 0.2902846772544624, -4.05538698618757e-17, -1.892797870777425e-17},
    {-0.9238795325112867, 0.3826834323650898, -1.7645047084336677e-17, -1.0050772696461588e-17},
    {-0.881921264348355, 0.47139673682599764, 1.9843248405890562e-17, 6.516678136069013e-18},
    {-0.8314696123025452, 0.5555702330196022, -1.4073856984728024e-18, 4.709410940561677e-17},
    {-0.773010453362737, 0.6343932841636455, 3.256590703364977e-17, 1.0420901929280035e-17},
    {-0.7071067811865476, 0.7071067811865476, 4.833646656726457e-17, -4.833646656726457e-17},
    {-0.6343932841636455, 0.773010453362737, -1.0420901929280035e-17, -3.256590703364977e-17},
    {-0.5555702330196022, 0.8314696123025452, -4.709410940561677e-17, 1.4073856984728024e-18},
    {-0.47139673682599764, 0.881921264348355, -6.516678136069013e-18, -1.9843248405890562e-17},
    {-0.3826834323650898, 0.9238795325112867, 1.0050772696461588e-17, 1.7645047084336677e-17},
    {-0.2902846772544624, 0.9569403357322088, 1.892797870777425e-17, 4.05538698618757e-17},
    {-0.19509032201612828, 0.9807852804032304, 7.991079068461731e-18, 1.8546939997825006e-17},
    {-0.0980171403295606, 0.9951847266721969, 1.634582362244256e-18, -4.248691367830441e-17}};
constexpr int kSinTabDoubles = 256;

// The table staged in LDS by the whole block (the caller synchronises).
__device__ __forceinline__ void stage_sin_tab(double* lds) {
  for (int i = threadIdx.x; i < 64; i += blockDim.x)
    for (int k = 0; k < 4; ++k) lds[4 * i + k] = kSinTab[i][k];
}

using SinTabP = const __attribute__((address_space(3))) double*;

// FP64 sine and cosine by the table: x = k pi/32 + r, |r| <= pi/64, with pi/32 split into two doubles: r0 = x - k hi is exact
// (its bits are multiples of hi's last one) and r = r0 + el. Polynomials: sin r to r^7, its coefficients from interpolating
// (sin r / r - 1) / r^2 at the three Chebyshev points of r^2 (off by less than 2e-19), cos r - 1 to r^8 by Taylor (1e-19).
// Then the angle sum. What the roundings of r and of the table's entry left (el, lo) is added to the corrections, so the last
// addition is the one rounding of the result's own size. 22 operations and two 16-byte LDS reads, against 35 for
// the reduction to pi/4 with its series to r^15 and r^16. Root mean square error over +-20 rad 2.7e-17, largest relative
// error 1.9e-16 (that of the series 3.2e-17 and 2.1e-16; without el and lo, 18 operations, 4.6e-17 and 3.5e-16).
// In two parts, so that other work can stand between the reads and their use: the entry (and k), then the rest.
// EXACT = false, for values that are rounded to FP32 at once: without el and lo, and one read.
using SinTabV = double __attribute__((ext_vector_type(2)));
struct SinTabE {
  SinTabV v, lo;
};
// x 32/pi is rounded to the whole number k by adding 1.5 2^52, whose low bits are then k's (|k| < 2^51; a conversion to 32
// bits ended at |x| = 2.1e8).
__host__ __device__ __forceinline__ int sin_tab_index(double x, double& k) {
  const double t = __builtin_fma(x, 10.185916357881302, 6755399441055744.0);
  k = t - 6755399441055744.0;
  return int(__builtin_bit_cast(uint64_t, t)) & 63;
}
__device__ __forceinline__ SinTabE sin_tab_entry(double x, SinTabP tab, double& k) {
  using P = const __attribute__((address_space(3))) SinTabV*;
  const SinTabP p = tab + 4 * sin_tab_index(x, k);
  return SinTabE{*(P)p, *(P)(p + 2)};
}
template <bool EXACT = true>
__host__ __device__ __forceinline__ void sincos_finish(double x, double k, const SinTabE& t, double& s, double& c) {
  const double r0 = __builtin_fma(-k, 0.09817477042468103, x);
  const double el = -k * 3.827021247335479e-18;
  const double r = EXACT ? r0 + el : __builtin_fma(-k, 3.827021247335479e-18, r0);
  const double r2 = r * r;
  double ps = __builtin_fma(r2, -0.00019840273844900185, 0.008333333324333671);
  double pc = __builtin_fma(r2, 1.0 / 40320.0, -1.0 / 720.0);
  ps = __builtin_fma(r2, ps, -0.16666666666666546);
  pc = __builtin_fma(r2, pc, 1.0 / 24.0);
  const double sr = __builtin_fma(r * r2, ps, EXACT ? el : r);  // sin r - r0, or sin r
  pc = __builtin_fma(r2, pc, -0.5);
  const double cm = r2 * pc;
  if constexpr (!EXACT) {
    s = __builtin_fma(t.v.y, sr, __builtin_fma(t.v.x, cm, t.v.x));
    c = __builtin_fma(-t.v.x, sr, __builtin_fma(t.v.y, cm, t.v.y));
    return;
  }
  s = t.v.x + __builtin_fma(t.v.y, r0, __builtin_fma(t.v.y, sr, __builtin_fma(t.v.x, cm, t.lo.x)));
  c = t.v.y + __builtin_fma(-t.v.x, r0, __builtin_fma(-t.v.x, sr, __builtin_fma(t.v.y, cm, t.lo.y)));
}
template <bool EXACT = true>
__device__ __forceinline__ void sincos_tab(double x, SinTabP tab, double& s, double& c) {
  double k;
  const SinTabE t = sin_tab_entry(x, tab, k);
  sincos_finish<EXACT>(x, k, t, s, c);
}

// Where the walks take sines and cosines from. TrigLive: computed from the iterate in every pass (EXACT: the FP64 passes').
// TrigTile: the residual pass stores them, rounded to FP32, in a per-lane column of a [D][64] LDS tile
// (a prismatic joint's slot holds its coordinate) and the FP32 step passes read them there.
// fresh(): the same source for another pass, whose reads the compiler cannot merge with an earlier pass's (it would
// keep every value in registers in between).
template <bool EXACT>
struct TrigLiveOf {
  static constexpr bool tile = false, exact = EXACT;
  SinTabP tab;
  __device__ __forceinline__ TrigLiveOf fresh() const { return *this; }
};
using TrigLive = TrigLiveOf<true>;
struct TrigTile {
  static constexpr bool tile = true, exact = true;
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
