// sie64.h -- the singular isothermal ellipsoid in float64, for the general models
// and for the re-tracing next to a cuspy source centre.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lensed {

constexpr double LN2 = 0.693147180559945309417;
// 1 - q^2 below which a lens is nearly round: u and v stay within 1/q, so the
// arguments (1 - q^2) u^2 of the series stay below 0.053.
constexpr double SIE_SERIES_S = 0.05;

// G of F(z) = 1 + z G(z) = sum z^k / (2k + 1) (fit_atan64.py), so that
// atan(w) = w + w (-w^2) G(-w^2) and atanh(w) = w + w w^2 G(w^2).
// ATAN64: z in [-tan(pi/8)^2, 0], error of F 7e-18; ATANH64: z in [-0.053, 1/9], 9e-18.
constexpr double ATAN64[11] = {0.3333333333333333,   0.19999999999995652,  0.1428571428469138,  0.11111111017100327,
                               0.0909090464769568,   0.07692184699371778,  0.06664531369805009, 0.05858311810501153,
                               0.05086254885823143,  0.03925369632061856,  0.019202529268412274};
constexpr double ATANH64[11] = {0.33333333333333337, 0.19999999999999435, 0.14285714285666257, 0.1111111111324447,
                                0.0909090915748564,  0.076923052325015,   0.06666645019219468, 0.05883461534086029,
                                0.05260033375561835, 0.04602098948800171, 0.05970391161562347};
__device__ __forceinline__ double poly10(const double (&c)[11], double z) {
  double p = c[10];
#pragma unroll
  for (int i = 9; i >= 0; --i) p = fma(p, z, c[i]);
  return p;
}

// 1/sqrt(a) and 1/a from the hardware's 25-bit estimates by one step of third
// order (relative error of the estimate cubed: below the float64 rounding).
__device__ __forceinline__ double rsqrt64(double a) {
  const double r = __builtin_amdgcn_rsq(a);
  const double e = fma(-(a * r), r, 1.0);
  return fma(r, e * fma(e, 0.375, 0.5), r);
}
__device__ __forceinline__ double rcp64(double a) {
  const double r = __builtin_amdgcn_rcp(a);
  const double e = fma(-a, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// The SIE in its own frame: (a, b) with alpha' = f (a, b), at the offset (xp, yp)
// from its centre; f = k in closed form, theta_E sqrt(q) in the series. x'^2 carries
// SIE_TINY64, so that at the centre itself the arguments are 0 and so is the
// deflection; anywhere else (|x'| > 1e-32) it is below float64 resolution. The smallest
// product there is 2 q^3 SIE_TINY64^(3/2) under the closed form's reciprocal: a normal
// number for every float32 q > 0 (down to 1.4e-45), since a subnormal's reciprocal is
// infinite and the deflection would be 0 x inf.
//   closed   a = atan(q' x'/psi) as the angle of (psi, q'|x'|), reduced by 0, pi/4 or
//            pi/2 to an argument within tan(pi/8); b = atanh(q' y'/psi) =
//            1/2 ln(P/M), P = psi + q'|y'|, M = psi - q'|y'|, with P M = q^2 r^2, so
//            P/M = P^2 / (q^2 r^2) without cancellation for any q; its power of
//            two k comes off by the exponents, and the rest is
//            atanh((P^2 - 2^k q^2 r^2) / (P^2 + 2^k q^2 r^2)), argument within 1/3.
//            The two quotients share one reciprocal. P^2 is taken as psi^2 + q'|y'| (2 psi +
//            q'|y'|), which at y' = 0 is q^2 r^2 bit for bit, so that b is exactly 0 there: a
//            residue of 1e-16 of the deflection at the lens centre would move the light of
//            a cuspy source that lies right behind it by 1e-3 (its light goes with R^(1/n)).
//   series   a = u F(-(1 - q^2) u^2), b = v F((1 - q^2) v^2), u = x'/psi, v = y'/psi, the
//            same functions divided by q', through q = 1.
// Errors: a few 1e-16 in a and b.
constexpr double SIE_TINY64 = 1e-80;
struct SieAB {
  double a, b, psi2, r2, rs;   // rs = 1/psi
};
template <bool CLOSED>
__device__ __forceinline__ SieAB sie_ab(double q2, double qp, double s2, double xp, double yp) {
  SieAB o;
  const double xx = fma(xp, xp, SIE_TINY64), yy = yp * yp;
  o.psi2 = fma(q2, xx, yy);
  o.r2 = xx + yy;
  o.rs = rsqrt64(o.psi2);
  if (CLOSED) {
    const double psi = o.psi2 * o.rs, X = qp * fabs(xp), Y = qp * fabs(yp);
    const bool mid = X > 0.4142135623730950488 * psi, high = X > 2.414213562373095049 * psi;
    const double num = high ? -psi : (mid ? X - psi : X), den = high ? X : (mid ? X + psi : psi);
    const double base = high ? 1.570796326794896619 : (mid ? 0.785398163397448310 : 0.0);
    const double P2 = fma(Y, fma(2.0, psi, Y), o.psi2), Q2 = q2 * o.r2;
    const int k = (int)((__builtin_bit_cast(uint64_t, P2) >> 52) & 0x7ff) -
                  (int)((__builtin_bit_cast(uint64_t, Q2) >> 52) & 0x7ff);
    const double Qk = ldexp(Q2, k);
    const double n2 = P2 - Qk, d2 = P2 + Qk, rr = rcp64(den * d2);
    const double w1 = num * (d2 * rr), w2 = n2 * (den * rr);
    const double z1 = -w1 * w1, z2 = w2 * w2;
    const double a = base + fma(w1 * z1, poly10(ATAN64, z1), w1);
    const double b = fma((double)k, 0.5 * LN2, fma(w2 * z2, poly10(ATANH64, z2), w2));
    o.a = copysign(a, xp);
    o.b = copysign(b, yp);
  } else {
    const double u = xp * o.rs, v = yp * o.rs, z1 = -s2 * u * u, z2 = s2 * v * v;
    o.a = fma(u * z1, poly10(ATANH64, z1), u);
    o.b = fma(v * z2, poly10(ATANH64, z2), v);
  }
  return o;
}

}  // namespace lensed
