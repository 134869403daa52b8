// Device math for the per-point path: sine/cosine of any angle of the
// model, rotation by small angles, and fast reciprocals.
//
// sincos_rr: y = x - 2*pi*k with k = rint(x / 2*pi) (a two-part 2*pi, the
// product exact inside the fused multiply-add), then, in float, the Taylor
// series of sin and cos (1/n! coefficients) at h = y / 2 in [-pi/2, pi/2]
// (through h^13 / h^12, truncation below 7e-9) and the double-angle
// identities sin 2h = 2 sin h cos h, cos 2h = 1 - 2 sin^2 h (no quadrant
// selection, so nothing depends on k fitting an integer); in double, a table
// of sin and cos at multiples of pi / 64, indexed straight from the rounded
// quotient, and the short series of the remainder (see the function).
//
// rotate_small: (sin x, cos x) -> (sin(x+d), cos(x+d)) by angle addition with
// the series of sin d and cos d; used for |d| <= kRotMax, exact to rounding
// there (double: d^9/9! < 6e-18 at |d| = 0.05; float: see small_sc).
#pragma once

#include <hip/hip_runtime.h>

namespace sgp4mi {

constexpr double kRotMax = 0.05;

// Double-precision constants live in constant memory: gfx9 VALU instructions
// take no 64-bit literals, and scalar-register operands (one per instruction)
// avoid holding every coefficient in a vector register pair.  Arrays of their own:
// from one array the compiler loads all of them at once, and the scalar registers
// that takes spill (100,000 x 1008 FP64 1,246 -> 1,261 us).
__constant__ double kTurn64 = 0.15915494309189533577;  // 1 / (2 pi)
// sin d = d + d^3 (-1/3! + d^2 (1/5! - d^2 / 7!)), highest order first
__constant__ double kSinSmall64[3] = {-1.98412698412698412698e-4, 8.33333333333333333333e-3,
                                      -1.66666666666666666667e-1};
// cos d = 1 + d^2 (-1/2 + d^2 (1/4! + d^2 (-1/6! + d^2 / 8!)))
__constant__ double kCosSmall64[3] = {2.48015873015873015873e-5, -1.38888888888888888889e-3,
                                      4.16666666666666666667e-2};

__device__ __forceinline__ void half_angle(float h, float* s, float* c) {
  const float h2 = h * h;
  float p = fmaf(h2, 1.60590438368e-10f, -2.50521083854e-8f);
  p = fmaf(p, h2, 2.75573192240e-6f);
  p = fmaf(p, h2, -1.98412698413e-4f);
  p = fmaf(p, h2, 8.33333333333e-3f);
  p = fmaf(p, h2, -1.66666666667e-1f);
  const float sh = fmaf(p * h2, h, h);
  float q = fmaf(h2, 2.08767569879e-9f, -2.75573192240e-7f);
  q = fmaf(q, h2, 2.48015873016e-5f);
  q = fmaf(q, h2, -1.38888888889e-3f);
  q = fmaf(q, h2, 4.16666666667e-2f);
  q = fmaf(q, h2, -0.5f);
  const float ch = fmaf(q, h2, 1.0f);
  *s = 2.0f * sh * ch;
  *c = fmaf(-2.0f * sh, sh, 1.0f);
}

// sin and cos of j pi / 64 for j = -64 .. 64, interleaved (sin, cos), each the
// double nearest the exact value.
__constant__ double kSinCos64[258] = {
    0.0, -1.0, -0.049067674327418015, -0.9987954562051724,
    -0.0980171403295606, -0.9951847266721969, -0.14673047445536175, -0.989176509964781,
    -0.19509032201612828, -0.9807852804032304, -0.2429801799032639, -0.970031253194544,
    -0.2902846772544624, -0.9569403357322088, -0.33688985339222005, -0.9415440651830208,
    -0.3826834323650898, -0.9238795325112867, -0.4275550934302821, -0.9039892931234433,
    -0.47139673682599764, -0.881921264348355, -0.5141027441932218, -0.8577286100002721,
    -0.5555702330196022, -0.8314696123025452, -0.5956993044924334, -0.8032075314806449,
    -0.6343932841636455, -0.773010453362737, -0.6715589548470184, -0.7409511253549591,
    -0.7071067811865476, -0.7071067811865476, -0.7409511253549591, -0.6715589548470184,
    -0.773010453362737, -0.6343932841636455, -0.8032075314806449, -0.5956993044924334,
    -0.8314696123025452, -0.5555702330196022, -0.8577286100002721, -0.5141027441932218,
    -0.881921264348355, -0.47139673682599764, -0.9039892931234433, -0.4275550934302821,
    -0.9238795325112867, -0.3826834323650898, -0.9415440651830208, -0.33688985339222005,
    -0.9569403357322088, -0.2902846772544624, -0.970031253194544, -0.2429801799032639,
    -0.9807852804032304, -0.19509032201612828, -0.989176509964781, -0.14673047445536175,
    -0.9951847266721969, -0.0980171403295606, -0.9987954562051724, -0.049067674327418015,
    -1.0, 0.0, -0.9987954562051724, 0.049067674327418015,
    -0.9951847266721969, 0.0980171403295606, -0.989176509964781, 0.14673047445536175,
    -0.9807852804032304, 0.19509032201612828, -0.970031253194544, 0.2429801799032639,
    -0.9569403357322088, 0.2902846772544624, -0.9415440651830208, 0.33688985339222005,
    -0.9238795325112867, 0.3826834323650898, -0.9039892931234433, 0.4275550934302821,
    -0.881921264348355, 0.47139673682599764, -0.8577286100002721, 0.5141027441932218,
    -0.8314696123025452, 0.5555702330196022, -0.8032075314806449, 0.5956993044924334,
    -0.773010453362737, 0.6343932841636455, -0.7409511253549591, 0.6715589548470184,
    -0.7071067811865476, 0.7071067811865476, -0.6715589548470184, 0.7409511253549591,
    -0.6343932841636455, 0.773010453362737, -0.5956993044924334, 0.8032075314806449,
    -0.5555702330196022, 0.8314696123025452, -0.5141027441932218, 0.8577286100002721,
    -0.47139673682599764, 0.881921264348355, -0.4275550934302821, 0.9039892931234433,
    -0.3826834323650898, 0.9238795325112867, -0.33688985339222005, 0.9415440651830208,
    -0.2902846772544624, 0.9569403357322088, -0.2429801799032639, 0.970031253194544,
    -0.19509032201612828, 0.9807852804032304, -0.14673047445536175, 0.989176509964781,
    -0.0980171403295606, 0.9951847266721969, -0.049067674327418015, 0.9987954562051724,
    0.0, 1.0, 0.049067674327418015, 0.9987954562051724,
    0.0980171403295606, 0.9951847266721969, 0.14673047445536175, 0.989176509964781,
    0.19509032201612828, 0.9807852804032304, 0.2429801799032639, 0.970031253194544,
    0.2902846772544624, 0.9569403357322088, 0.33688985339222005, 0.9415440651830208,
    0.3826834323650898, 0.9238795325112867, 0.4275550934302821, 0.9039892931234433,
    0.47139673682599764, 0.881921264348355, 0.5141027441932218, 0.8577286100002721,
    0.5555702330196022, 0.8314696123025452, 0.5956993044924334, 0.8032075314806449,
    0.6343932841636455, 0.773010453362737, 0.6715589548470184, 0.7409511253549591,
    0.7071067811865476, 0.7071067811865476, 0.7409511253549591, 0.6715589548470184,
    0.773010453362737, 0.6343932841636455, 0.8032075314806449, 0.5956993044924334,
    0.8314696123025452, 0.5555702330196022, 0.8577286100002721, 0.5141027441932218,
    0.881921264348355, 0.47139673682599764, 0.9039892931234433, 0.4275550934302821,
    0.9238795325112867, 0.3826834323650898, 0.9415440651830208, 0.33688985339222005,
    0.9569403357322088, 0.2902846772544624, 0.970031253194544, 0.2429801799032639,
    0.9807852804032304, 0.19509032201612828, 0.989176509964781, 0.14673047445536175,
    0.9951847266721969, 0.0980171403295606, 0.9987954562051724, 0.049067674327418015,
    1.0, 0.0, 0.9987954562051724, -0.049067674327418015,
    0.9951847266721969, -0.0980171403295606, 0.989176509964781, -0.14673047445536175,
    0.9807852804032304, -0.19509032201612828, 0.970031253194544, -0.2429801799032639,
    0.9569403357322088, -0.2902846772544624, 0.9415440651830208, -0.33688985339222005,
    0.9238795325112867, -0.3826834323650898, 0.9039892931234433, -0.4275550934302821,
    0.881921264348355, -0.47139673682599764, 0.8577286100002721, -0.5141027441932218,
    0.8314696123025452, -0.5555702330196022, 0.8032075314806449, -0.5956993044924334,
    0.773010453362737, -0.6343932841636455, 0.7409511253549591, -0.6715589548470184,
    0.7071067811865476, -0.7071067811865476, 0.6715589548470184, -0.7409511253549591,
    0.6343932841636455, -0.773010453362737, 0.5956993044924334, -0.8032075314806449,
    0.5555702330196022, -0.8314696123025452, 0.5141027441932218, -0.8577286100002721,
    0.47139673682599764, -0.881921264348355, 0.4275550934302821, -0.9039892931234433,
    0.3826834323650898, -0.9238795325112867, 0.33688985339222005, -0.9415440651830208,
    0.2902846772544624, -0.9569403357322088, 0.2429801799032639, -0.970031253194544,
    0.19509032201612828, -0.9807852804032304, 0.14673047445536175, -0.989176509964781,
    0.0980171403295606, -0.9951847266721969, 0.049067674327418015, -0.9987954562051724,
    0.0, -1.0,
};

// A constant held in a scalar register.  gfx9 three-operand
// instructions take no literal, so a fused multiply-add with a literal factor
// and a second constant costs an extra vector move; with the factor in a
// scalar register (set by a scalar move) it is one instruction.
__device__ __forceinline__ float sgpr_const(float x) {
  asm("" : "+s"(x));
  return x;
}
__device__ __forceinline__ double sgpr_const(double x) {
  asm("" : "+s"(x));
  return x;
}

// Double: b = x - n pi / 64 with n the nearest whole number (a two-part pi / 64,
// the product exact inside the fused multiply-add, |b| <= pi / 128), the table's
// sin and cos of (n mod 128) pi / 64 and the series of sin b through b^7 and
// cos b through b^6 (the next terms are below 4e-19 and 3.3e-18 relative),
// combined by angle addition.  n is rounded by adding 1.5 * 2^52 + 64: the low
// bits of the sum are n + 64, so the table index takes no conversion, and the
// mask keeps it inside the table for every input (NaN, infinity, huge).  The sum
// holds n to a whole number up to |x| = 1.1e14; larger angles (elements of that
// size, or the drag polynomials long after a decay) must first be reduced by
// whole turns (reduced: in two parts, which leaves them below that up to 1e29).
// The propagation checks its angles together (a check in each sine cost 6 % at
// 100,000 x 1008 FP64); sincos_any checks its own.
constexpr double kTableMax = 0x1p46;
__device__ __forceinline__ double reduced(double x) {
  if (fabs(x) > kTableMax) {
    const double turns = rint(x * 0.15915494309189533577);
    x = fma(-turns, 6.2831853071795864769, x);  // 2 pi, nearest double
    x = fma(-turns, 2.4492935982947063e-16, x);  // 2 pi minus that
  }
  return x;
}
__device__ __forceinline__ void sincos_rr(double x, double* s, double* c) {
  const double round64 = 6755399441055808.0;       // 1.5 * 2^52 + 64
  const double m = fma(x, sgpr_const(20.371832715762604), round64);  // 64 / pi
  const double n = m - round64;
  double b = fma(-n, sgpr_const(0.04908738521234052), x);  // pi / 64, nearest double
  b = fma(-n, sgpr_const(1.9135106236677394e-18), b);      // pi / 64 minus that
  // Read the pair at a 32-bit byte offset from the table's base, seen in the
  // global address space (the load then takes the base from scalar registers
  // and needs no 64-bit address).
  uint32_t off = (uint32_t(__double2loint(m)) & 127u) * 16u;
  asm("" : "+v"(off));
  typedef const __attribute__((address_space(1))) char* GBytes;
  typedef const __attribute__((address_space(1))) double* GDouble;
  const GDouble e = (GDouble)((GBytes)(const char*)kSinCos64 + off);
  const double sa = e[0], ca = e[1];
  const double b2 = b * b;
  // Coefficients in scalar registers (an instruction reads at most one); the
  // first step of each polynomial holds two of them, so it is a product and a
  // sum instead of a fused multiply-add that would need one moved into vector
  // registers first.
  double p, q;
  {
#pragma clang fp contract(off)
    p = b2 * sgpr_const(-1.98412698412698412698e-4) + sgpr_const(8.33333333333333333333e-3);
    q = b2 * sgpr_const(-1.38888888888888888889e-3) + sgpr_const(4.16666666666666666667e-2);
  }
  p = fma(p, b2, sgpr_const(-1.66666666666666666667e-1));
  const double sb = fma(p * b2, b, b);
  q = fma(q, b2, -0.5) * b2;  // cos b - 1
  *s = fma(ca, sb, fma(sa, q, sa));
  *c = fma(-sa, sb, fma(ca, q, ca));
}

__device__ __forceinline__ void sincos_any(double x, double* s, double* c) { sincos_rr(reduced(x), s, c); }

__device__ __forceinline__ void sincos_rr(float x, float* s, float* c) {
  const float n = rintf(x * 0.15915494309189533577f);
  float y = fmaf(-n, 6.28318548202514648438f, x);   // float nearest 2*pi
  y = fmaf(-n, -1.7484556e-7f, y);                   // 2*pi minus that
  half_angle(0.5f * y, s, c);
}

// Hardware sine and cosine (v_sin_f32 / v_cos_f32 take the argument in
// revolutions): the angle is reduced to a fraction of a turn in its own type,
// then rounded to float.  sincos_hw keeps 1 / (2 pi) in scalar registers (read
// from memory, as sincos_hw_mem does, the wavefront waits for it amid the secular
// terms: 700,000 ragged tiles 366 -> 378 us).  The mixed derivatives, whose
// results are double, use sincos_hw_mem: the compiler fuses their sums differently
// with the other, which moves single results by a float rounding.
__device__ __forceinline__ void sincos_hw(double x, float* s, float* c) {
  const float r = float(__builtin_amdgcn_fract(x * sgpr_const(0.15915494309189533577)));
  *s = __builtin_amdgcn_sinf(r);
  *c = __builtin_amdgcn_cosf(r);
}
__device__ __forceinline__ void sincos_hw_mem(double x, float* s, float* c) {
  const float r = float(__builtin_amdgcn_fract(x * kTurn64));
  *s = __builtin_amdgcn_sinf(r);
  *c = __builtin_amdgcn_cosf(r);
}
__device__ __forceinline__ void sincos_hw(float x, float* s, float* c) {
  const float r = __builtin_amdgcn_fractf(x * 0.15915494309189533577f);
  *s = __builtin_amdgcn_sinf(r);
  *c = __builtin_amdgcn_cosf(r);
}

__device__ __forceinline__ void small_sc(double d, double* sd, double* cd) {
  const double d2 = d * d;
  double ps = fma(d2, kSinSmall64[0], kSinSmall64[1]);
  ps = fma(ps, d2, kSinSmall64[2]);
  *sd = fma(ps * d2, d, d);
  double pc = fma(d2, kCosSmall64[0], kCosSmall64[1]);
  pc = fma(pc, d2, kCosSmall64[2]);
  pc = fma(pc, d2, -0.5);
  *cd = fma(pc, d2, 1.0);
}

// Float: through d^3 (sine) and d^4 (cosine); the next terms are below
// 2.6e-9 and 2.2e-11 at |d| = 0.05, under the float rounding of the result.
__device__ __forceinline__ void small_sc(float d, float* sd, float* cd) {
  const float d2 = d * d;
  *sd = fmaf(d2 * d, -1.6666666667e-1f, d);
  float pc = fmaf(d2, sgpr_const(4.1666666667e-2f), -0.5f);
  *cd = fmaf(pc, d2, 1.0f);
}

template <class T>
__device__ __forceinline__ void rotate_small(T* s, T* c, T d) {
  T sd, cd;
  small_sc(d, &sd, &cd);
  const T s0 = *s, c0 = *c;
  *s = s0 * cd + c0 * sd;
  *c = c0 * cd - s0 * sd;
}

// Rotations by still smaller angles (double), with fewer terms: |d| <= kRotMid
// (the sine through d^5, the cosine through d^4; the next terms are below 2e-22
// and 2e-18) and |d| <= kRotTiny (the sine through d^3; the next is below 3e-17).
constexpr double kRotMid = 3.2e-3, kRotTiny = 1.25e-3;
__device__ __forceinline__ void rotate_by(double* s, double* c, double sd, double cd1) {  // sin d, cos d - 1
  const double s0 = *s, c0 = *c;
  *s = fma(c0, sd, fma(s0, cd1, s0));
  *c = fma(-s0, sd, fma(c0, cd1, c0));
}
__device__ __forceinline__ void rotate_mid(double* s, double* c, double d) {
  const double d2 = d * d;
  double p;
  {
#pragma clang fp contract(off)
    p = d2 * sgpr_const(8.33333333333333333333e-3) + sgpr_const(-1.66666666666666666667e-1);
  }
  rotate_by(s, c, fma(p * d2, d, d), d2 * fma(d2, sgpr_const(4.16666666666666666667e-2), -0.5));
}
__device__ __forceinline__ void rotate_tiny(double* s, double* c, double d) {
  const double d2 = d * d;
  rotate_by(s, c, fma(d2 * sgpr_const(-1.66666666666666666667e-1), d, d),
            d2 * fma(d2, sgpr_const(4.16666666666666666667e-2), -0.5));
}

// Float: the sine through d, the cosine through d^2; the next terms are below
// 4e-10 and 2e-13.
__device__ __forceinline__ void rotate_tiny(float* s, float* c, float d) {
  const float h = -0.5f * d * d, s0 = *s, c0 = *c;
  *s = fmaf(c0, d, fmaf(s0, h, s0));
  *c = fmaf(-s0, d, fmaf(c0, h, c0));
}

// Reciprocal and reciprocal square root: in double the hardware estimate y
// (relative error e of 1e-7 or less) and one third-order step, 1 + e + e^2 and
// 1 + e / 2 + 3 e^2 / 8 (an ulp or so; the root for positive arguments); in
// float the hardware estimate alone (about 1 ulp).  rcp_from refines an estimate
// that the caller has (relative error below 1e-5).  x^(-2/3), the semi-major axis
// of a mean motion: a float estimate of x^(-1/3) (relative error below 2^-19 from
// 1e-30 to 1e30: half an ulp of the exponent, up to 33, in the power) and one
// third-order step; arguments beyond float's comfortable range take the
// library's cube root.
__device__ __forceinline__ double rcp_from(double x, double y) {
  const double e = fma(-x, y, 1.0);
  return fma(y, fma(e, e, e), y);
}
__device__ __forceinline__ double rcp(double x) { return rcp_from(x, __builtin_amdgcn_rcp(x)); }
__device__ __forceinline__ double rsq(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, sgpr_const(0.375), 0.5), y);
}
__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double pow_m23(double x) {
  if (!(x > 1.0e-30 && x < 1.0e30)) {
    const double c = ::cbrt(1.0 / x);
    return c * c;
  }
  const double y = double(__builtin_amdgcn_exp2f(-0.33333333333f * __builtin_amdgcn_logf(float(x))));
  const double e = fma(-x * y, y * y, 1.0);
  const double z = y * fma(e, fma(e, 2.0 / 9.0, 1.0 / 3.0), 1.0);
  return z * z;
}
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }

}  // namespace sgp4mi
