// Device helpers shared by the tiled kernels and the all-pairs kernels.
//
// Every float operation that decides a result is an explicit round-to-nearest
// intrinsic (no contraction), so results match a plain IEEE binary32
// evaluation of the same expressions.
#pragma once

#include "clue_internal.h"

namespace clue {

__device__ __forceinline__ float dist2(float xi, float yi, float xj, float yj) {
  float dx = __fsub_rn(xi, xj);
  float dy = __fsub_rn(yi, yj);
  return __fadd_rn(__fmul_rn(dx, dx), __fmul_rn(dy, dy));
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

__device__ __forceinline__ int wave_incl_scan(int v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  return v;
}
__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Order-preserving map of a float to uint32 (-0 folds onto +0), so that
// (rho, index) compares as one 64-bit unsigned key.
__device__ __forceinline__ unsigned ord_f32(float v) {
  const unsigned u = __float_as_uint(__fadd_rn(v, 0.0f));
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
// Inverse of ord_f32 (gives +0 for a folded -0, which compares the same).
__device__ __forceinline__ float ord_inv(unsigned o) {
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

// ---------------------------------------------------------------------------
// Terms of Eq. 3.
// ---------------------------------------------------------------------------
// exp(x) for x <= 0 as one fixed binary32 evaluation, after Cody and Waite's
// range reduction: x = k ln2 + r with k = floor(x / ln2 + 1/2) and ln2 split
// into a high part with trailing zero bits (k * hi exact) and the remainder;
// exp(r) by its degree-7 Taylor polynomial in Horner form; then the scale by
// 2^k. Every step is an explicit binary32 rounding, so any IEEE evaluation of
// the same steps gives the same bits. 0 when k < -125.
__device__ __forceinline__ float exp32(float x) {
  constexpr float inv_ln2 = (float)(1.0 / 0.69314718055994530942);
  constexpr float ln2_hi = 0.693145751953125f;
  constexpr float ln2_lo = (float)(0.69314718055994530942 - 0.693145751953125);
  const float kf = floorf(__fadd_rn(__fmul_rn(x, inv_ln2), 0.5f));
  if (!(kf >= -125.0f)) return 0.0f;
  const float r = __fsub_rn(__fsub_rn(x, __fmul_rn(kf, ln2_hi)), __fmul_rn(kf, ln2_lo));
  float p = (float)(1.0 / 5040.0);
  p = __fadd_rn(__fmul_rn(p, r), (float)(1.0 / 720.0));
  p = __fadd_rn(__fmul_rn(p, r), (float)(1.0 / 120.0));
  p = __fadd_rn(__fmul_rn(p, r), (float)(1.0 / 24.0));
  p = __fadd_rn(__fmul_rn(p, r), (float)(1.0 / 6.0));
  p = __fadd_rn(__fmul_rn(p, r), 0.5f);
  p = __fadd_rn(__fmul_rn(p, r), 1.0f);
  p = __fadd_rn(__fmul_rn(p, r), 1.0f);
  return __fmul_rn(p, __uint_as_float((unsigned)((int)kf + 127) << 23));
}

// Correctly rounded binary32 square root of x >= 0: the hardware estimate
// (within an ulp) is corrected by comparing x with the squares of the
// midpoints to its neighbours, which are exact in binary64. Subnormal x is
// scaled by 2^64 first (exact, and exactly undone by 2^-32).
__device__ __forceinline__ float sqrt_rn(float x) {
  if (!(x > 0.0f) || x == __int_as_float(0x7f800000)) return x;
  const bool tiny = x < 1.17549435e-38f;
  const float xs = tiny ? __fmul_rn(x, 18446744073709551616.0f) : x;
  float s = __builtin_sqrtf(xs);
  const double xd = (double)xs;
  const float up = __uint_as_float(__float_as_uint(s) + 1u);
  const double mh = 0.5 * ((double)s + (double)up);
  if (mh * mh < xd) {
    s = up;
  } else {
    const float dn = __uint_as_float(__float_as_uint(s) - 1u);
    const double ml = 0.5 * ((double)dn + (double)s);
    if (ml * ml > xd) s = dn;
  }
  return tiny ? __fmul_rn(s, 2.3283064365386963e-10f) : s;
}

// One term of Eq. 3 for a neighbour at squared distance d2 with energy e:
// e (flat kernel), fl(exp(-fl(d2 a)) e) (Gaussian, a = 1 / (2 s^2)) or
// fl(exp(-fl(sqrt(d2) a)) e) (exponential, a = 1 / s).
template <int K>
__device__ __forceinline__ float kernel_term(float d2, float ka, float e) {
  if constexpr (K == 0) {
    return e;
  } else if constexpr (K == 1) {
    return __fmul_rn(exp32(-__fmul_rn(d2, ka)), e);
  } else {
    return __fmul_rn(exp32(-__fmul_rn(sqrt_rn(d2), ka)), e);
  }
}

}  // namespace clue
