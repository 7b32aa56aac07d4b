// model.hip -- general models: several SIEs with free centres, an external
// shear, several Sersic components in the image or the source plane, a flat
// sky (the models of the paper's fits of real lenses, Sec. 5), and lenses on
// several planes (the multi-plane extension named in Sec. 6).
//
// Coordinates, deflections and radii are float64 (the float32 folding of the
// 17-parameter render does not carry over to an arbitrary number of
// components), and so are the SIE's atan and atanh, whose errors would move
// rays near a cuspy source centre. The Sersic profiles take their powers of
// two as an exact integer part and a float32 fraction (exp2_split,
// log2_split): errors of a few 1e-7 of each subsample's light that vary with
// the argument, at a fraction of the float64 library functions' cost. Each
// pixel is rounded once; the PSF and chi^2 stages are the common ones.
//
// What bounds it: the float64 issue rate. With the library's atan, atanh, sqrt
// and divisions a subsample of the 41-parameter model took about 770 issue
// slots, 500 of them in its two SIEs. The SIE now takes one reciprocal square
// root and one reciprocal (both refined to float64), and 13 multiply-adds each
// for the atan and the atanh, with constants folded per point in the prologue
// and two subsamples interleaved: about 340 slots. 256 points of the 41-parameter model
// (200 x 200 pixels, N = 4) on one card: render 3.65 -> 1.65 ms; gradients of 64
// points 2.62 -> 0.65 ms (closed-form moments in two kinds of passes instead of dual
// numbers in one pass per component).
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "sb_device.h"
#include "sie64.h"

namespace lensed {
namespace {

// 2^a for float64 a (0 below a = -1100): the integer part exact (ldexp), the fraction in [0, 1)
// by the float32 hardware exp2 (relative error about 1e-7).
__device__ inline double exp2_split(double a) {
  a = fmax(a, -1100.0);
  const double k = floor(a);
  return ldexp((double)__builtin_amdgcn_exp2f((float)(a - k)), (int)k);
}

// log2 u for finite u >= 0: the binary exponent exact, the mantissa in [1/2, 1)
// by the float32 hardware log2 (absolute error about 1e-7).
__device__ inline double log2_split(double u) {
  int k;
  const double f = frexp(u, &k);
  return (double)k + (double)__builtin_amdgcn_logf((float)f);
}

template <bool CLOSED>
__device__ __forceinline__ SieAB sie_ab(const SieConst& c, double xp, double yp) {
  return lensed::sie_ab<CLOSED>(c.q2, c.qp, c.s2, xp, yp);
}

// The deflection of SIE c at S points (x, y), taken off (bx, by) (Eq. 1).
template <bool CLOSED, int S>
__device__ __forceinline__ void sub_sie_as(const SieConst& c, const double (&x)[S], const double (&y)[S], double (&bx)[S],
                                        double (&by)[S]) {
#pragma unroll
  for (int i = 0; i < S; ++i) {
    const double dx = x[i] - c.x, dy = y[i] - c.y;
    const double xp = fma(c.c, dx, c.s * dy), yp = fma(c.c, dy, -(c.s * dx));
    const SieAB o = sie_ab<CLOSED>(c, xp, yp);
    const double f = CLOSED ? c.k : c.tesq;
    const double a1 = f * o.a, a2 = f * o.b;
    bx[i] -= fma(c.c, a1, -(c.s * a2));
    by[i] -= fma(c.s, a1, c.c * a2);
  }
}
template <int S>
__device__ __forceinline__ void sub_sie(const SieConst& c, const double (&x)[S], const double (&y)[S], double (&bx)[S],
                                        double (&by)[S]) {
  if (c.closed)   // uniform
    sub_sie_as<true, S>(c, x, y, bx, by);
  else
    sub_sie_as<false, S>(c, x, y, bx, by);
}

// Sersic component c (Eq. 22) at (px, py): the offset, rotation and radius in
// float64; the profile exp(-b ((R/R_e)^{1/n} - 1)) as powers of two, whose
// exponents are float64 and whose fractional parts go through the hardware
// float32 exp2 / log2 (per-subsample relative errors of a few 1e-7 that
// vary with the argument, against the float64 library functions' many
// instructions each).
__device__ __forceinline__ double sersic_at(const SersicConst& c, double px, double py) {
  const double dx = px - c.x, dy = py - c.y;
  const double X = fma(c.s11, dx, c.s12 * dy), Y = fma(c.s21, dx, c.s22 * dy);
  const double R2 = fma(X, X, Y * Y);
  // (R/R_e)^{1/n} = 2^(log2(R^2 / R_e^2) / (2n)); at R = 0 the logarithm is -inf, and
  // exp2_split's clamp makes the power 0
  const double t = exp2_split(c.e * log2_split(R2));
  return c.I * exp2_split(c.B * (1.0 - t));
}

// Surface brightness of a general model with one lens plane at S points (Eqs.
// 1-2 with several deflectors in one plane, Eq. 22 for every Sersic, plus the
// sky).
template <int S>
__device__ __forceinline__ void model_sb(const ModelConst& m, const double (&x)[S], const double (&y)[S],
                                         double (&I)[S]) {
  double bx[S], by[S];
#pragma unroll
  for (int i = 0; i < S; ++i) {
    bx[i] = x[i] - (m.g1 * x[i] + m.g2 * y[i]);
    by[i] = y[i] - (m.g2 * x[i] - m.g1 * y[i]);
    I[i] = m.sky;
  }
  for (int k = 0; k < m.n_sie; ++k) sub_sie<S>(m.sie[k], x, y, bx, by);
  for (int j = 0; j < m.n_sersic; ++j) {
    const SersicConst& c = m.ser[j];
    if (m.plane[j] != 0) {   // uniform
#pragma unroll
      for (int i = 0; i < S; ++i) I[i] += sersic_at(c, bx[i], by[i]);
    } else {
#pragma unroll
      for (int i = 0; i < S; ++i) I[i] += sersic_at(c, x[i], y[i]);
    }
  }
}

// The same with P = spec.n_planes lens planes: the ray's position on plane j
// is x_j = x - sum_{i<j} beta_ij alpha_i(x_i) (beta_iP = 1 for the source
// plane P), taken plane by plane in order of distance; alpha_i sums the SIEs
// of plane i (and the shear on plane 0); each Sersic is evaluated at the
// position on its own plane.
__device__ double model_sb_planes(const ModelConst& m, const ModelSpec& spec, double x, double y) {
  const int P = spec.n_planes;
  double ax[MAX_PLANES], ay[MAX_PLANES];
  double I = m.sky;
  for (int j = 0; j <= P; ++j) {
    double px[1] = {x}, py[1] = {y};
    for (int i = 0; i < j; ++i) {
      const double b = j == P ? 1.0 : spec.beta[i][j];
      px[0] -= b * ax[i];
      py[0] -= b * ay[i];
    }
    for (int k = 0; k < m.n_sersic; ++k)
      if (m.plane[k] == j) I += sersic_at(m.ser[k], px[0], py[0]);
    if (j < P) {
      double dx[1] = {0.0}, dy[1] = {0.0};   // minus the deflection
      for (int k = 0; k < m.n_sie; ++k)
        if (spec.sie_plane[k] == j) sub_sie<1>(m.sie[k], px, py, dx, dy);
      if (j == 0) {
        dx[0] -= m.g1 * px[0] + m.g2 * py[0];
        dy[0] -= m.g2 * px[0] - m.g1 * py[0];
      }
      ax[j] = -dx[0];
      ay[j] = -dy[0];
    }
  }
  return I;
}

// One thread per pixel, one block per (point, render tile): the pixel's
// quadrature (N x N midpoint or Gauss-Kronrod), times the pixel weight.
// A rule's abscissae (in pixels from the centre) and weights in LDS, so that no
// subsample repeats the division.
struct RuleTable {
  double off[16], w[16];
};
__device__ __forceinline__ void fill_rule(RuleTable& t, const SysDesc& sd) {
  const int k = (int)threadIdx.x;
  if (k < sd.N) {
    const GkRule* R = sd.rule > 0 ? &kGkRules[sd.rule - 1] : nullptr;
    t.off[k] = R ? R->xd[k] : ((double)k + 0.5) / sd.N - 0.5;
    t.w[k] = R ? (double)R->w[k] : 1.0;
  }
  __syncthreads();
}

// A row of the rule goes two subsamples at a time (their chains interleave, and the
// scalar loads of a component's constants serve both); the sum keeps the rule's
// order. PLANES: several lens planes.
template <bool PLANES>
__global__ __launch_bounds__(RENDER_BLOCK, PLANES ? 1 : 3) void model_render_kernel(WorkArgs w, ModelSpec spec,
                                                                                    const ModelConst* __restrict__ mcs,
                                                                                    float* __restrict__ L) {
  int point, tile;
  if (w.items) {
    const int2 it = w.items[blockIdx.x];
    point = it.x;
    tile = it.y;
  } else {
    point = w.point0;
    tile = blockIdx.x;
  }
  const SysDesc sd = w.sys_table ? w.sys_table[w.point_sys ? w.point_sys[point] : 0] : w.single;
  const int64_t loff = w.point_loff ? w.point_loff[point] : 0;
  __shared__ RuleTable rule;
  fill_rule(rule, sd);
  // render units are single pixels: the whole image, or in a gradient plan the
  // support of g (the only pixels the PSF outputs with w > 0 read)
  const int unit = tile * RENDER_BLOCK + (int)threadIdx.x;
  if (unit >= unit_count(sd, 1)) return;
  const int pix = unit_pixel(sd, unit, 1);
  const ModelConst& m = mcs[point];
  const int r = row_of(sd, pix), c = pix - r * sd.W;
  const double ux = (double)c - 0.5 * (double)(sd.W - 1), uy = (double)r - 0.5 * (double)(sd.H - 1);
  const double d = sd.d, cx = sd.cx, cy = sd.cy;
  const int N = sd.N;
  double acc = 0.0;
  for (int ky = 0; ky < N; ++ky) {
    const double y = cy + (uy + rule.off[ky]) * d;
    const double wy = rule.w[ky];
    if constexpr (PLANES) {
      for (int kx = 0; kx < N; ++kx) acc += rule.w[kx] * wy * model_sb_planes(m, spec, cx + (ux + rule.off[kx]) * d, y);
    } else {
      int kx = 0;
      for (; kx + 2 <= N; kx += 2) {
        const double xs[2] = {cx + (ux + rule.off[kx]) * d, cx + (ux + rule.off[kx + 1]) * d}, ys[2] = {y, y};
        double I[2];
        model_sb<2>(m, xs, ys, I);
        acc += rule.w[kx] * wy * I[0];
        acc += rule.w[kx + 1] * wy * I[1];
      }
      if (kx < N) {
        const double xs[1] = {cx + (ux + rule.off[kx]) * d}, ys[1] = {y};
        double I[1];
        model_sb<1>(m, xs, ys, I);
        acc += rule.w[kx] * wy * I[0];
      }
    }
  }
  L[loff + pix] = (float)(acc * sd.wgt);
}

// ---------------------------------------------------------------------------
// Adjoint of general models: d log L / d theta =
// sum_j g_j wgt sum_k w_k dI(x_jk)/d theta, g = A^T rho (the common adjoint PSF
// stage), the derivative of Eq. 17 through Eqs. 15, 14, 2, 1 and 22, in float64.
//
// One lens plane (model_grad_kernel): the partials in closed form.
//   SIE k        dI/dtheta_k = -G . d alpha_k/d theta_k  (x_c, y_c, theta_E, q, phi)
//   Sersic j     dS_j/d(x, y, I_e, R_e, n, q, phi) at x (foreground) or beta
//   shear, sky   G . d beta/d(gamma, phi_gamma), 1
// with G = sum over the lensed Sersics of grad S_j(beta). Every partial is a
// per-point linear combination of a few sums over the subsamples (moments), so the
// kernel accumulates those. A pass (blockIdx.y) covers two SIEs, the first of
// them also the shear and the sky, or two Sersics, so that a thread keeps at most 14
// sums; the ray (every SIE) and G are evaluated once per pass.
//
// Several lens planes (model_grad_planes_kernel): forward-mode dual numbers, one
// component per pass.
// ---------------------------------------------------------------------------

// Value and M partial derivatives.
template <int M>
struct Dl {
  double v;
  double d[M];
};

template <int M>
__device__ inline Dl<M> dconst(double v) {
  Dl<M> r;
  r.v = v;
#pragma unroll
  for (int i = 0; i < M; ++i) r.d[i] = 0.0;
  return r;
}
// f(a) with f'(a) = fp
template <int M>
__device__ inline Dl<M> dchain(const Dl<M>& a, double f, double fp) {
  Dl<M> r;
  r.v = f;
#pragma unroll
  for (int i = 0; i < M; ++i) r.d[i] = fp * a.d[i];
  return r;
}
template <int M>
__device__ inline Dl<M> operator+(const Dl<M>& a, const Dl<M>& b) {
  Dl<M> r;
  r.v = a.v + b.v;
#pragma unroll
  for (int i = 0; i < M; ++i) r.d[i] = a.d[i] + b.d[i];
  return r;
}
template <int M>
__device__ inline Dl<M> operator-(const Dl<M>& a, const Dl<M>& b) {
  Dl<M> r;
  r.v = a.v - b.v;
#pragma unroll
  for (int i = 0; i < M; ++i) r.d[i] = a.d[i] - b.d[i];
  return r;
}
template <int M>
__device__ inline Dl<M> operator-(const Dl<M>& a) {
  return dchain(a, -a.v, -1.0);
}
template <int M>
__device__ inline Dl<M> operator*(const Dl<M>& a, const Dl<M>& b) {
  Dl<M> r;
  r.v = a.v * b.v;
#pragma unroll
  for (int i = 0; i < M; ++i) r.d[i] = a.d[i] * b.v + a.v * b.d[i];
  return r;
}
template <int M>
__device__ inline Dl<M> operator*(const Dl<M>& a, double b) {
  return dchain(a, a.v * b, b);
}
template <int M>
__device__ inline Dl<M> operator+(const Dl<M>& a, double b) {
  return dchain(a, a.v + b, 1.0);
}
template <int M>
__device__ inline Dl<M> operator/(const Dl<M>& a, const Dl<M>& b) {
  Dl<M> r;
  r.v = a.v / b.v;
  const double ib = 1.0 / b.v;
#pragma unroll
  for (int i = 0; i < M; ++i) r.d[i] = (a.d[i] - r.v * b.d[i]) * ib;
  return r;
}
template <int M>
__device__ inline Dl<M> dsqrt(const Dl<M>& a) {
  const double s = sqrt(a.v);
  return dchain(a, s, 0.5 / s);
}
// exp and log of a Sersic argument, as in sersic_at (relative errors of a few
// 1e-7 in the value and the derivatives).
template <int M>
__device__ inline Dl<M> dexp(const Dl<M>& a) {
  const double e = exp2_split(a.v * LOG2E);
  return dchain(a, e, e);
}
template <int M>
__device__ inline Dl<M> dlog(const Dl<M>& a) {
  return dchain(a, log2_split(a.v) * LN2, 1.0 / a.v);
}
template <int M>
__device__ inline Dl<M> datan(const Dl<M>& a) {
  return dchain(a, atan(a.v), 1.0 / (1.0 + a.v * a.v));
}
template <int M>
__device__ inline Dl<M> datanh(const Dl<M>& a) {
  return dchain(a, atanh(a.v), 1.0 / (1.0 - a.v * a.v));
}

// atan(sqrt(s) u) / sqrt(s) (HYP false) or atanh(sqrt(s) u) / sqrt(s) (HYP
// true), s = 1 - q^2 >= 0: below SIE_SERIES_S by the series
// u sum_k (-+1)^k (s u^2)^k / (2k + 1), which also gives the round limit s = 0
// and its derivative in s. The SIE keeps |u| <= 1/q for the atan and |u| <= 1
// for the atanh, so s u^2 < 0.053 there and 15 terms reach 1e-19.
template <bool HYP, int M>
__device__ inline Dl<M> atan_over_root(const Dl<M>& s, const Dl<M>& u) {
  if (s.v < SIE_SERIES_S) {
    const Dl<M> z = s * u * u;
    constexpr int K = 14;
    Dl<M> p = dconst<M>((HYP || K % 2 == 0 ? 1.0 : -1.0) / (2 * K + 1));
    for (int k = K - 1; k >= 0; --k) p = p * z + (HYP || k % 2 == 0 ? 1.0 : -1.0) / (2 * k + 1);
    return u * p;
  }
  const Dl<M> r = dsqrt(s);
  return (HYP ? datanh(r * u) : datan(r * u)) / r;
}

// ---- Several lens planes: the ray's positions in dual numbers --------------
// With lenses on several planes a deflector's parameters move the rays of every
// later plane, so the pass carries derivatives through the whole chain: the
// position on plane j is x - sum_{i<j} beta_ij alpha_i(x_i) in dual numbers
// whose variables are the pass's own parameters (those of SIE comp, of Sersic
// comp, or the shear), and every deflector and Sersic is evaluated at dual
// positions.

// SIE k at the dual position (x, y); own: its (x_c, y_c, theta_E, q, phi) are
// the variables 0..4.
__device__ inline void sie_alpha_dual(const ModelConst& m, int k, const Dl<7>& x, const Dl<7>& y, bool own,
                                      Dl<7>& ax, Dl<7>& ay) {
  const SieConst& s = m.sie[k];
  Dl<7> xc = dconst<7>(s.x), yc = dconst<7>(s.y), c = dconst<7>(s.c), sn = dconst<7>(s.s);
  Dl<7> te = dconst<7>(s.te), q = dconst<7>(s.q);
  if (own) {
    xc.d[0] = 1.0;
    yc.d[1] = 1.0;
    te.d[2] = 1.0;
    q.d[3] = 1.0;
    c.d[4] = -s.s;
    sn.d[4] = s.c;
  }
  const Dl<7> dx = x - xc, dy = y - yc;
  const Dl<7> xp = c * dx + sn * dy, yp = c * dy - sn * dx;
  const Dl<7> psi2 = q * q * xp * xp + yp * yp;
  if (!(psi2.v > 0.0)) {   // the centre itself: no deflection
    ax = ay = dconst<7>(0.0);
    return;
  }
  const Dl<7> psi = dsqrt(psi2);
  const Dl<7> ss = -(q * q) + 1.0;
  const Dl<7> f = te * dsqrt(q);
  const Dl<7> a1 = f * atan_over_root<false>(ss, xp / psi), a2 = f * atan_over_root<true>(ss, yp / psi);
  ax = c * a1 - sn * a2;
  ay = sn * a1 + c * a2;
}

// The external shear's deflection at (x, y) added to (ax, ay); own: (gamma,
// phi_gamma) are the variables 0, 1.
__device__ inline void shear_alpha_dual(const ModelConst& m, const Dl<7>& x, const Dl<7>& y, bool own, Dl<7>& ax,
                                        Dl<7>& ay) {
  Dl<7> gam = dconst<7>(m.gam), c2 = dconst<7>(m.c2g), s2 = dconst<7>(m.s2g);
  if (own) {
    gam.d[0] = 1.0;
    c2.d[1] = -2.0 * m.s2g;
    s2.d[1] = 2.0 * m.c2g;
  }
  const Dl<7> g1 = gam * c2, g2 = gam * s2;
  ax = ax + g1 * x + g2 * y;
  ay = ay + g2 * x - g1 * y;
}

// Sersic j at the dual position (px, py); own: its (x, y, I_e, R_e, n, q, phi)
// are the variables 0..6.
__device__ inline Dl<7> sersic_at_dual(const ModelConst& m, int j, const Dl<7>& px, const Dl<7>& py,
                                               bool own) {
  const SersicConst& s = m.ser[j];
  Dl<7> x0 = dconst<7>(s.x), y0 = dconst<7>(s.y), Ie = dconst<7>(s.I), Re = dconst<7>(1.0 / s.iRe);
  Dl<7> n = dconst<7>(1.0 / s.in), q = dconst<7>(s.q), c = dconst<7>(s.c), sn = dconst<7>(s.s);
  Dl<7> b = dconst<7>(s.b);
  if (own) {
    x0.d[0] = 1.0;
    y0.d[1] = 1.0;
    Ie.d[2] = 1.0;
    Re.d[3] = 1.0;
    n.d[4] = 1.0;
    b.d[4] = s.db;
    q.d[5] = 1.0;
    c.d[6] = -s.s;
    sn.d[6] = s.c;
  }
  const Dl<7> dx = px - x0, dy = py - y0;
  const Dl<7> xp = c * dx + sn * dy, yp = c * dy - sn * dx;
  const Dl<7> R2 = q * xp * xp + yp * yp / q;
  const Dl<7> t = R2.v > 0.0 ? dexp(dlog(R2 / (Re * Re)) * (dconst<7>(0.5) / n)) : dconst<7>(0.0);
  return Ie * dexp(-(b * (t + -1.0)));
}

// I at the subsample (x, y) of a model with spec.n_planes > 1 (the sky left
// out), with its derivatives in the pass's parameters (kind 0: SIE comp, 1:
// Sersic comp, 2: the shear).
__device__ Dl<7> planes_dual(const ModelConst& m, const ModelSpec& spec, double x, double y, int kind, int comp) {
  const int P = spec.n_planes;
  Dl<7> ax[MAX_PLANES], ay[MAX_PLANES];
  Dl<7> I = dconst<7>(0.0);
  for (int j = 0; j <= P; ++j) {
    Dl<7> px = dconst<7>(x), py = dconst<7>(y);
    for (int i = 0; i < j; ++i) {
      const double b = j == P ? 1.0 : spec.beta[i][j];
      px = px - ax[i] * b;
      py = py - ay[i] * b;
    }
    for (int k = 0; k < m.n_sersic; ++k)
      if (m.plane[k] == j) I = I + sersic_at_dual(m, k, px, py, kind == 1 && comp == k);
    if (j < P) {
      Dl<7> dx = dconst<7>(0.0), dy = dconst<7>(0.0);
      for (int k = 0; k < m.n_sie; ++k)
        if (spec.sie_plane[k] == j) {
          Dl<7> a, b;
          sie_alpha_dual(m, k, px, py, kind == 0 && comp == k, a, b);
          dx = dx + a;
          dy = dy + b;
        }
      if (j == 0 && spec.shear) shear_alpha_dual(m, px, py, kind == 2, dx, dy);
      ax[j] = dx;
      ay[j] = dy;
    }
  }
  return I;
}

// One component per pass (blockIdx.y): an SIE, a Sersic, or the shear and the sky.
__global__ __launch_bounds__(RENDER_BLOCK) void model_grad_planes_kernel(WorkArgs w, ModelSpec spec,
                                                                         const ModelConst* __restrict__ mcs,
                                                                         const float* __restrict__ G,
                                                                         const int* __restrict__ gpbase,
                                                                         double* __restrict__ gpart, int P) {
  __shared__ double red[RENDER_BLOCK / 64][7];
  int point, tile;
  if (w.items) {
    const int2 it = w.items[blockIdx.x];
    point = it.x;
    tile = it.y;
  } else {
    point = w.point0;
    tile = blockIdx.x;
  }
  const SysDesc sd = w.sys_table ? w.sys_table[w.point_sys ? w.point_sys[point] : 0] : w.single;
  const int64_t loff = w.point_loff ? w.point_loff[point] : 0;
  const ModelConst& m = mcs[point];
  const int pass = (int)blockIdx.y;
  const int kind = pass < spec.n_sie ? 0 : (pass < spec.n_sie + spec.n_sersic ? 1 : 2);
  const int comp = kind == 0 ? pass : pass - spec.n_sie;
  const int off = kind == 0 ? 5 * comp : (kind == 1 ? 5 * spec.n_sie + (spec.shear ? 2 : 0) + 7 * comp : 5 * spec.n_sie);
  const int npar = kind == 0 ? 5 : (kind == 1 ? 7 : (spec.shear ? 2 : 0) + (spec.sky ? 1 : 0));
  // the sky is the model's last parameter; the other slots of a pass are consecutive
  auto slot = [&](int i) { return kind == 2 && spec.sky && i == npar - 1 ? P - 1 : off + i; };
  const int n_sup = grad_support_count(sd);
  if (tile * RENDER_BLOCK >= n_sup) {   // past the support's last pixel: zero sums
    if ((int)threadIdx.x < npar) gpart[(size_t)(gpbase[point] + tile) * P + slot(threadIdx.x)] = 0.0;
    return;
  }
  double acc[7];
#pragma unroll
  for (int i = 0; i < 7; ++i) acc[i] = 0.0;
  const int unit = tile * RENDER_BLOCK + (int)threadIdx.x;
  const int pix = unit < n_sup ? grad_support_pixel(sd, unit) : 0;
  const float gp = unit < n_sup ? G[loff + pix] : 0.0f;
  if (gp != 0.0f) {   // pixels outside the reach of any weighted residual add nothing
    const int r = row_of(sd, pix), c = pix - r * sd.W;
    const double ux = (double)c - 0.5 * (double)(sd.W - 1), uy = (double)r - 0.5 * (double)(sd.H - 1);
    const double d = sd.d, cx = sd.cx, cy = sd.cy;
    const int N = sd.N;
    const GkRule* R = sd.rule > 0 ? &kGkRules[sd.rule - 1] : nullptr;
    for (int ky = 0; ky < N; ++ky) {
      const double oy = R ? R->xd[ky] : ((double)ky + 0.5) / N - 0.5;
      const double y = cy + (uy + oy) * d;
      for (int kx = 0; kx < N; ++kx) {
        const double ox = R ? R->xd[kx] : ((double)kx + 0.5) / N - 0.5;
        const double wq = R ? (double)R->w[kx] * (double)R->w[ky] : 1.0;
        const double x = cx + (ux + ox) * d;
        if (kind < 2 || spec.shear) {
          const Dl<7> I = planes_dual(m, spec, x, y, kind, comp);
          const int nd = kind == 0 ? 5 : (kind == 1 ? 7 : 2);
          for (int i = 0; i < nd; ++i) acc[i] += wq * I.d[i];
        }
        if (kind == 2 && spec.sky) acc[spec.shear ? 2 : 0] += wq;
      }
    }
    const double scale = (double)gp * sd.wgt;
#pragma unroll
    for (int i = 0; i < 7; ++i) acc[i] *= scale;
  }
  // block sums in float64, in a fixed order
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < 7; ++i) {
    double v = acc[i];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if (lane == 0) red[wid][i] = v;
  }
  __syncthreads();
  if ((int)threadIdx.x < npar) {
    const int i = threadIdx.x;
    double v = red[0][i];
    for (int k = 1; k < RENDER_BLOCK / 64; ++k) v += red[k][i];
    gpart[(size_t)(gpbase[point] + tile) * P + slot(i)] = v;
  }
}

// ---- One lens plane: moments in closed form ---------------------------------

// Sersic c at (px, py): X, Y (scaled frame), E = S/I_e, D = dS/d(X^2 + Y^2) and dn =
// dS/dn; at the centre itself D = 0 and dn = S db/dn.
struct SersicM {
  double X, Y, E, D, dn;
};
__device__ __forceinline__ SersicM sersic_moments(const SersicConst& c, double px, double py) {
  SersicM o;
  const double dx = px - c.x, dy = py - c.y;
  o.X = fma(c.s11, dx, c.s12 * dy);
  o.Y = fma(c.s21, dx, c.s22 * dy);
  const double R2 = fma(o.X, o.X, o.Y * o.Y);
  const bool pos = R2 > 0.0;
  const double R2s = pos ? R2 : 1.0, l2 = log2_split(R2s);
  const double t = pos ? exp2_split(c.e * l2) : 0.0;
  o.E = exp2_split(c.B * (1.0 - t));
  const double S = c.I * o.E, bt = c.b * t;
  o.D = -(S * bt * c.e) * rcp64(R2s);
  // dS/dn = S [b' (1 - t) + b t ln(R^2/R_e^2) / (2 n^2)], 1/(2 n^2) = e/n
  o.dn = S * fma(c.db, 1.0 - t, bt * (l2 * LN2) * (c.e * c.in));
  return o;
}
// dS/d(px, py)
__device__ __forceinline__ void sersic_gradient(const SersicConst& c, const SersicM& s, double& gx, double& gy) {
  gx = 2.0 * s.D * fma(c.s11, s.X, c.s21 * s.Y);
  gy = 2.0 * s.D * fma(c.s12, s.X, c.s22 * s.Y);
}

// The five moments of SIE c (o: its deflection at (xp, yp) in its frame) for the source
// gradient (Gx, Gy), added to M with weight wq: with G' = G in the lens frame,
// u = x'/psi, v = y'/psi, alpha' = theta_E sqrt(q) (A, B),
//   M0 = A G'x + B G'y
//   M1 = G'x (2 dA/ds + u^3 psi^2/r^2) + G'y (2 dB/ds + v u^2 psi^2/(q^2 r^2)), s = 1 - q^2
//   M2 = (v - B) G'x + (A - u) G'y
//   M3 = y' h / (psi r^2), M4 = x' h / (psi r^2), h = y' G'x - x' G'y
template <bool CLOSED>
__device__ __forceinline__ void sie_moments(const SieConst& c, const SieAB& o, double xp, double yp, double Gx,
                                            double Gy, double wq, double* __restrict__ M) {
  const double gx = wq * fma(c.c, Gx, c.s * Gy), gy = wq * fma(c.c, Gy, -(c.s * Gx));
  const double ir2 = rcp64(o.r2), pr = o.psi2 * ir2;
  const double u = xp * o.rs, v = yp * o.rs;
  double A, B, dA, dB;   // divided by q'; their derivatives in s
  if (CLOSED) {
    A = o.a * c.iqp;
    B = o.b * c.iqp;
    dA = fma(u, pr, -A) * c.hs;
    dB = fma(v * c.iq2, pr, -B) * c.hs;
  } else {
    A = o.a;
    B = o.b;
    // d/ds of u F(-s u^2) and v F(s v^2): F'(z) from the same polynomial
    auto slope = [&](double z) {   // F = 1 + z G, F' = G + z G'
      double p = ATANH64[10], dp = 0.0;
#pragma unroll
      for (int i = 9; i >= 0; --i) {
        dp = fma(dp, z, p);
        p = fma(p, z, ATANH64[i]);
      }
      return fma(z, dp, p);
    };
    dA = -u * u * u * slope(-c.s2 * u * u);
    dB = v * v * v * slope(c.s2 * v * v);
  }
  const double u2pr = u * u * pr, h = fma(yp, gx, -(xp * gy)) * (o.rs * ir2);
  M[0] += fma(A, gx, B * gy);
  M[1] += fma(gx, fma(2.0, dA, u * u2pr), gy * fma(2.0, dB, v * u2pr * c.iq2));
  M[2] += fma(v - B, gx, (A - u) * gy);
  M[3] += yp * h;
  M[4] += xp * h;
}

constexpr int GRAD_SIES = 2, GRAD_SERSICS = 2;   // components per pass
constexpr int GRAD_SUMS_LENS = 5 * GRAD_SIES + 3, GRAD_SUMS_LIGHT = 7 * GRAD_SERSICS;
// Passes over the SIEs (the first also covers the shear and the sky), and in all.
__host__ __device__ inline int grad_lens_passes(const ModelSpec& s) {
  const int n = (s.n_sie + GRAD_SIES - 1) / GRAD_SIES;
  return n == 0 && (s.shear || s.sky) ? 1 : n;
}
inline int grad_passes(const ModelSpec& s) { return grad_lens_passes(s) + (s.n_sersic + GRAD_SERSICS - 1) / GRAD_SERSICS; }

// LIGHT: the passes over the Sersics; otherwise those over the SIEs, shear and sky.
template <bool LIGHT>
__global__ __launch_bounds__(RENDER_BLOCK, LIGHT ? 4 : 3) void model_grad_kernel(WorkArgs w, ModelSpec spec,
                                                                     const ModelConst* __restrict__ mcs,
                                                                     const float* __restrict__ G,
                                                                     const int* __restrict__ gpbase,
                                                                     double* __restrict__ gpart, int P) {
  constexpr int SUMS = LIGHT ? GRAD_SUMS_LIGHT : GRAD_SUMS_LENS;
  __shared__ double red[RENDER_BLOCK / 64][SUMS];
  int point, tile;
  if (w.items) {
    const int2 it = w.items[blockIdx.x];
    point = it.x;
    tile = it.y;
  } else {
    point = w.point0;
    tile = blockIdx.x;
  }
  const SysDesc sd = w.sys_table ? w.sys_table[w.point_sys ? w.point_sys[point] : 0] : w.single;
  const int64_t loff = w.point_loff ? w.point_loff[point] : 0;
  __shared__ RuleTable rule;
  fill_rule(rule, sd);
  const ModelConst& m = mcs[point];
  const int first = (int)blockIdx.y * (LIGHT ? GRAD_SERSICS : GRAD_SIES);
  const bool extra = !LIGHT && first == 0;   // the shear and the sky
  double acc[SUMS];
#pragma unroll
  for (int i = 0; i < SUMS; ++i) acc[i] = 0.0;
  const int n_sup = grad_support_count(sd);
  const int unit = tile * RENDER_BLOCK + (int)threadIdx.x;
  const int pix = unit < n_sup ? grad_support_pixel(sd, unit) : 0;
  const float gp = unit < n_sup ? G[loff + pix] : 0.0f;
  if (gp != 0.0f) {   // pixels outside the reach of any weighted residual add nothing
    const int r = row_of(sd, pix), c = pix - r * sd.W;
    const double ux = (double)c - 0.5 * (double)(sd.W - 1), uy = (double)r - 0.5 * (double)(sd.H - 1);
    const double d = sd.d, cx = sd.cx, cy = sd.cy;
    const int N = sd.N;
    bool any_lensed = false;   // uniform
    for (int j = 0; j < (LIGHT ? GRAD_SERSICS : m.n_sersic); ++j) {
      const int jj = LIGHT ? first + j : j;
      any_lensed = any_lensed || (jj < m.n_sersic && m.plane[jj] != 0);
    }
    auto subsample = [&](int ky, int kx) {
      const double x[1] = {cx + (ux + rule.off[kx]) * d}, y[1] = {cy + (uy + rule.off[ky]) * d};
      const double wq = rule.w[kx] * rule.w[ky];
      double bx[1] = {x[0] - (m.g1 * x[0] + m.g2 * y[0])}, by[1] = {y[0] - (m.g2 * x[0] - m.g1 * y[0])};
      if constexpr (LIGHT) {
        if (any_lensed)
          for (int k = 0; k < m.n_sie; ++k) sub_sie<1>(m.sie[k], x, y, bx, by);
#pragma unroll
        for (int j = 0; j < GRAD_SERSICS; ++j) {
          if (first + j >= m.n_sersic) break;
          const bool lensed = m.plane[first + j] != 0;
          const SersicM s = sersic_moments(m.ser[first + j], lensed ? bx[0] : x[0], lensed ? by[0] : y[0]);
          double* __restrict__ a = acc + 7 * j;
          const double D = wq * s.D, DX = D * s.X, DY = D * s.Y;
          a[0] += DX;
          a[1] += DY;
          a[2] = fma(wq, s.E, a[2]);
          a[3] = fma(DX, s.X, a[3]);
          a[4] = fma(DY, s.Y, a[4]);
          a[5] = fma(DX, s.Y, a[5]);
          a[6] = fma(wq, s.dn, a[6]);
        }
      } else {
        // the ray: the pass's own SIEs keep their deflections for the moments
        SieAB own[GRAD_SIES];
        double xp[GRAD_SIES], yp[GRAD_SIES];
        if (any_lensed) {
          for (int k = 0; k < m.n_sie; ++k)
            if (k < first || k >= first + GRAD_SIES) sub_sie<1>(m.sie[k], x, y, bx, by);
#pragma unroll
          for (int k = 0; k < GRAD_SIES; ++k) {
            if (first + k >= m.n_sie) break;
            const SieConst& lc = m.sie[first + k];
            const bool closed = lc.closed;
            const double f = closed ? lc.k : lc.tesq;
            const double dx = x[0] - lc.x, dy = y[0] - lc.y;
            xp[k] = fma(lc.c, dx, lc.s * dy);
            yp[k] = fma(lc.c, dy, -(lc.s * dx));
            own[k] = closed ? sie_ab<true>(lc, xp[k], yp[k]) : sie_ab<false>(lc, xp[k], yp[k]);
            const double a1 = f * own[k].a, a2 = f * own[k].b;
            bx[0] -= fma(lc.c, a1, -(lc.s * a2));
            by[0] -= fma(lc.s, a1, lc.c * a2);
          }
        }
        double Gx = 0.0, Gy = 0.0;
        if (any_lensed) {
          for (int j = 0; j < m.n_sersic; ++j)
            if (m.plane[j] != 0) {
              double gx, gy;
              sersic_gradient(m.ser[j], sersic_moments(m.ser[j], bx[0], by[0]), gx, gy);
              Gx += gx;
              Gy += gy;
            }
#pragma unroll
          for (int k = 0; k < GRAD_SIES; ++k) {
            if (first + k >= m.n_sie) break;
            const SieConst& lc = m.sie[first + k];
            const bool closed = lc.closed;
            if (closed)
              sie_moments<true>(lc, own[k], xp[k], yp[k], Gx, Gy, wq, acc + 5 * k);
            else
              sie_moments<false>(lc, own[k], xp[k], yp[k], Gx, Gy, wq, acc + 5 * k);
          }
        }
        if (extra) {
          // beta = x - alpha_SIE - Gamma x, Gamma = gamma [[c2, s2], [s2, -c2]]
          acc[5 * GRAD_SIES] += wq * fma(Gx, x[0], -(Gy * y[0]));
          acc[5 * GRAD_SIES + 1] += wq * fma(Gx, y[0], Gy * x[0]);
          acc[5 * GRAD_SIES + 2] += wq;
        }
      }
    };
    for (int ky = 0; ky < N; ++ky)
      for (int kx = 0; kx < N; ++kx) subsample(ky, kx);
    const double scale = (double)gp * sd.wgt;
#pragma unroll
    for (int i = 0; i < SUMS; ++i) acc[i] *= scale;
  }
  // block sums of the moments in float64, in a fixed order
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < SUMS; ++i) {
    double v = acc[i];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if (lane == 0) red[wid][i] = v;
  }
  __syncthreads();
  if ((int)threadIdx.x < SUMS) {
    const int i = threadIdx.x;
    double v = red[0][i];
    for (int k = 1; k < RENDER_BLOCK / 64; ++k) v += red[k][i];
    red[0][i] = v;
  }
  __syncthreads();
  // the partials from the moments, one thread per component
  double* __restrict__ out = gpart + (size_t)(gpbase[point] + tile) * P;
  const int i = threadIdx.x;
  const double* __restrict__ M = red[0];
  if constexpr (LIGHT) {
    if (i >= GRAD_SERSICS || first + i >= m.n_sersic) return;
    const SersicConst& c = m.ser[first + i];
    const double* __restrict__ T = M + 7 * i;
    double* __restrict__ g = out + 5 * m.n_sie + (spec.shear ? 2 : 0) + 7 * (first + i);
    g[0] = -2.0 * (c.s11 * T[0] + c.s21 * T[1]);
    g[1] = -2.0 * (c.s12 * T[0] + c.s22 * T[1]);
    g[2] = T[2];
    g[3] = -2.0 * c.iRe * (T[3] + T[4]);
    g[4] = T[6];
    g[5] = (T[3] - T[4]) / c.q;
    g[6] = 2.0 * (c.q - 1.0 / c.q) * T[5];
  } else {
    if (i < GRAD_SIES && first + i < m.n_sie) {
      const SieConst& c = m.sie[first + i];
      const double* __restrict__ T = M + 5 * i;
      double* __restrict__ g = out + 5 * (first + i);
      const double sq = sqrt(c.q);
      // d I/d x_c = G . d alpha/d x, in the frame theta_E sqrt(q) (M3, -M4)
      g[0] = c.tesq * (c.c * T[3] + c.s * T[4]);
      g[1] = c.tesq * (c.s * T[3] - c.c * T[4]);
      g[2] = -sq * T[0];
      g[3] = -c.te * (0.5 / sq * T[0] - sq * c.q * T[1]);
      g[4] = -c.tesq * T[2];
    } else if (i == GRAD_SIES && extra) {
      const double* __restrict__ T = M + 5 * GRAD_SIES;
      if (spec.shear) {
        out[5 * m.n_sie] = -(m.c2g * T[0] + m.s2g * T[1]);
        out[5 * m.n_sie + 1] = -2.0 * m.gam * (m.c2g * T[1] - m.s2g * T[0]);
      }
      if (spec.sky) out[P - 1] = T[2];
    }
  }
}

// grad[p][k] = sum over the point's render tiles, float64, rounded once: a block per
// point, 64 parameters at a time, eight tile chains per parameter added in a fixed
// order.
constexpr int MFIN_CHAINS = 8;
__global__ __launch_bounds__(64 * MFIN_CHAINS) void model_finalize_grad_kernel(const double* __restrict__ gpart,
                                                                              const int* __restrict__ gpbase,
                                                                              int ntiles, int P,
                                                                              float* __restrict__ grad,
                                                                              int point_base) {
  __shared__ double part[MFIN_CHAINS][64];
  const int p = point_base + (int)blockIdx.x, lane = (int)threadIdx.x & 63, chain = (int)threadIdx.x >> 6;
  const double* __restrict__ g = gpart + (size_t)gpbase[p] * P;
  for (int k0 = 0; k0 < P; k0 += 64) {
    const int k = k0 + lane;
    double s = 0.0;
    if (k < P) {
#pragma unroll 4
      for (int i = chain; i < ntiles; i += MFIN_CHAINS) s += g[(size_t)i * P + k];
    }
    part[chain][lane] = s;
    __syncthreads();
    if (chain == 0 && k < P) {
      for (int c = 1; c < MFIN_CHAINS; ++c) s += part[c][lane];
      grad[(size_t)p * P + k] = (float)s;
    }
    __syncthreads();
  }
}

}  // namespace

hipError_t launch_model_render(const WorkArgs& w, const ModelSpec& spec, const ModelConst* mcs, float* L, int n_blocks,
                               hipStream_t stream) {
  if (n_blocks <= 0) return hipSuccess;
  return for_item_parts(w, n_blocks, [&](const WorkArgs& part, int n) {
    if (spec.n_planes > 1)
      hipLaunchKernelGGL(model_render_kernel<true>, dim3(n), dim3(RENDER_BLOCK), 0, stream, part, spec, mcs, L);
    else
      hipLaunchKernelGGL(model_render_kernel<false>, dim3(n), dim3(RENDER_BLOCK), 0, stream, part, spec, mcs, L);
    return hipGetLastError();
  });
}

hipError_t launch_model_grad(const WorkArgs& w, const ModelSpec& spec, const ModelConst* mcs, const float* G,
                            const int* gpbase, double* gpart, int P, int n_blocks, hipStream_t stream) {
  if (n_blocks <= 0) return hipSuccess;
  const int lens = grad_lens_passes(spec), light = grad_passes(spec) - lens;
  const int comps = spec.n_sie + spec.n_sersic + ((spec.shear || spec.sky) ? 1 : 0);
  return for_item_parts(w, n_blocks, [&](const WorkArgs& part, int n) {
    if (spec.n_planes > 1) {
      hipLaunchKernelGGL(model_grad_planes_kernel, dim3(n, comps), dim3(RENDER_BLOCK), 0, stream, part, spec, mcs, G,
                         gpbase, gpart, P);
      return hipGetLastError();
    }
    if (lens > 0)
      hipLaunchKernelGGL(model_grad_kernel<false>, dim3(n, lens), dim3(RENDER_BLOCK), 0, stream, part, spec, mcs, G,
                         gpbase, gpart, P);
    hipLaunchKernelGGL(model_grad_kernel<true>, dim3(n, light), dim3(RENDER_BLOCK), 0, stream, part, spec, mcs, G,
                       gpbase, gpart, P);
    return hipGetLastError();
  });
}

hipError_t launch_model_finalize_grad(const double* gpart, const int* gpbase, int ntiles, int P, int n_points,
                                      float* grad, hipStream_t stream) {
  for (int p0 = 0; p0 < n_points; p0 += 1 << 20) {
    const int np = n_points - p0 < (1 << 20) ? n_points - p0 : (1 << 20);
    hipLaunchKernelGGL(model_finalize_grad_kernel, dim3((unsigned)np), dim3(64 * MFIN_CHAINS), 0, stream, gpart, gpbase, ntiles, P,
                       grad, p0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace lensed
