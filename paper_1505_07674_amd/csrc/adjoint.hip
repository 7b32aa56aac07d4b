// adjoint.hip -- gradient of the log-likelihood with respect to the 17 parameters.
//
// log L = -1/2 sum_i w_i (d_i - L*_i)^2 (Sec. 3.2, Eq. 17), L* = A L with A the
// replicate-padded PSF convolution (Sec. 3.1, Eq. 15) and L_j the midpoint sum
// of Eq. 14. With rho = w (d - L*) (written by the PSF kernel in mode 2):
//   d log L / d theta = sum_j g_j (d^2/N^2) sum_k dI(x_jk)/d theta,  g = A^T rho.
// A^T rho is a zero-padded correlation of rho with the kernel for interior
// pixels; pixels on the first/last row or column use kernel tables folded by
// the padding (computed by the prologue). The per-subsample partial derivatives
// of I(x) = I_lens(x) + I_source(beta(x)) are written out in closed form:
// through the Sersic profiles (Eqs. 22-23, with db_n/dn), and for the lens
// parameters through beta = x - alpha(x) (Eq. 1) using the SIE Jacobian
//   d alpha'/d x' = theta_E sqrt(q)/(psi r^2) [[y'^2, -x'y'], [-x'y', x'^2]].
// Each partial is a fixed per-point linear combination of 17 moments (sums
// over subsamples of products that vary per subsample, without the per-point
// factors), so the kernels accumulate the moments and the final pass maps them
// to the 17 partials in float64 (grad_from_moments). Sums are float32 per thread,
// combined across the block and across tiles in float64.
#include <math.h>

#include <algorithm>

#include "internal.h"
#include "kernels.h"
#include "sb_device.h"
#include "stencil.h"
#include "support.h"

namespace lensed {
namespace {

__device__ __forceinline__ void resolve(const WorkArgs& w, int& point, int& tile) {
  if (w.items) {
    const int2 it = w.items[blockIdx.x];
    point = it.x;
    tile = it.y;
  } else {
    point = w.point0;
    tile = blockIdx.x;
  }
}

// ---------------------------------------------------------------------------
// g = A^T rho, interior pixels: g[u][v] = sum_{a,b} rho0[u+a][v+b] F[a][b].
// ---------------------------------------------------------------------------
// The forward stencil's tiles and threads, with zeros outside the image and the
// unflipped taps.
template <int KP>
__global__ __launch_bounds__(PSF_MAX_THREADS, KP <= 24 ? 4 : 2) void adj_psf_kernel(WorkArgs w,
                                                                                    const float* __restrict__ R,
                                                                                    float* __restrict__ G) {
  constexpr int Q = PSF_Q, C = PSF_C;
  extern __shared__ __align__(16) float S[];
  int point, tile;
  resolve(w, point, tile);
  point = uniform(point);
  tile = uniform(tile);
  const SysDesc& sd = w.sys_table ? w.sys_table[w.point_sys ? w.point_sys[point] : 0] : w.single;
  if (sd.ptile_w && !(sd.ptile_w[tile] & PTILE_G)) return;   // no pixel of the support: nothing reads this g
  const int64_t loff = uniform(w.point_loff ? w.point_loff[point] : (int64_t)0);
  const int H = uniform(sd.H), W = uniform(sd.W), TW = uniform(sd.TW), TH = uniform(sd.TH);
  const int ph = uniform(sd.ph), pw = uniform(sd.pw), tiles_x = uniform(sd.tiles_x);
  gbyte_in* taps = uniform_in(sd.psfn + 2 * ph * pw);
  gbyte_in* Rp = uniform_in(R + loff);
  gbyte_out* Gp = uniform_out(G + loff);
  const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
  const int x0 = tx * TW, y0 = ty * TH;
  const int tid = threadIdx.x;
  const int cs = psf_col_stride(TH, KP);
  float* __restrict__ T = S + (TW + pw - 1) * cs;
  const bool mine = stage_tile<false>(S, Rp, H, W, TW + pw - 1, psf_tile_rows(TH, KP) / 4, cs, y0 - ph / 2, x0 - pw / 2);
  stage_taps(T, taps, ph, pw, tap_stride(KP), 3);
  const bool finite = __syncthreads_and(mine);
  const int nc = TW / C;   // threads per row of threads
  const int jr = tid / nc;
  const bool own = jr < TH / (4 * Q);
  const int row = own ? jr * 4 * Q : 0, col = own ? (tid - jr * nc) * C : 0;
  f32x4_t acc[C][Q];
  stencil<KP, Q, C>(S + col * cs + row, T, ph, pw, cs, finite, acc);
  __syncthreads();
  if (own) outputs_to_lds<Q, C>(S, cs, row, col, acc);
  __syncthreads();
  for (int it = tid; it < TW * (TH / 4); it += blockDim.x) {
    const int g = it / TW, c = it - g * TW;
    const int gj = x0 + c, gi0 = y0 + 4 * g;
    if (gj <= 0 || gj >= W - 1) continue;   // border pixels: the folded tables
    const f32x4_t v = *(const f32x4_t*)(S + c * cs + 4 * g);
    const unsigned W4 = 4u * (unsigned)W, o = (unsigned)gi0 * W4 + 4u * (unsigned)gj;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (gi0 + r > 0 && gi0 + r < H - 1) store_at(Gp, o + (unsigned)r * W4, v[r]);
  }
}

// Border pixels of g with the folded tables. A block takes a segment of up to
// BORDER_SEG consecutive pixels on one side of the image (top row, bottom row,
// then the left and right columns without their corners; blockIdx.y is the
// point) and stages the window of rho they read in LDS, zero outside the image,
// so every table row is a full PW-tap dot product (a zero tap adds exactly
// nothing). Each pixel has BORDER_SUB lanes: lane `sub` takes the table rows
// a = a_lo + sub, a_lo + sub + BORDER_SUB, ... of the rows that fall inside the
// image, and the partial sums are added in a fixed order by shuffles. PW = 0:
// the table width is a runtime value.
constexpr int BORDER_SEG = 64;
constexpr int BORDER_SUB = 4;

__host__ __device__ inline int border_row_segments(int W) { return (W + BORDER_SEG - 1) / BORDER_SEG; }
__host__ __device__ inline int border_side_segments(int H) { return H > 2 ? (H - 2 + BORDER_SEG - 1) / BORDER_SEG : 0; }
// Segments of an H x W image: every pixel on the first or last row or column
// lies in exactly one (the bottom row is absent when H = 1, the right column
// when W = 1).
__host__ __device__ inline int border_segments(int H, int W) {
  return border_row_segments(W) * (H > 1 ? 2 : 1) + border_side_segments(H) * (W > 1 ? 2 : 1);
}
// LDS floats of the largest window for a PSF of ph x pw.
__host__ __device__ inline int border_lds_floats(int ph, int pw) {
  const int row = ph * (BORDER_SEG + pw - 1), col = (BORDER_SEG + ph - 1) * pw;
  return row > col ? row : col;
}

template <int PW>
__global__ __launch_bounds__(BORDER_SEG* BORDER_SUB) void adj_border_kernel(WorkArgs w, const float* __restrict__ R,
                                                                             float* __restrict__ G, int point_base) {
  extern __shared__ float S[];
  const int point = point_base + (int)blockIdx.y;
  const SysDesc sd = w.sys_table ? w.sys_table[w.point_sys ? w.point_sys[point] : 0] : w.single;
  const int64_t loff = w.point_loff ? w.point_loff[point] : 0;
  if (w.point_goff && w.point_goff[point] != loff) return;   // a composite model's later component: no rho of its own
  const int H = sd.H, W = sd.W, p = sd.ph / 2, q = sd.pw / 2;
  const int pw = PW > 0 ? PW : sd.pw;
  const int nrow = border_row_segments(W), nbot = H > 1 ? nrow : 0;
  const int nside = border_side_segments(H), nright = W > 1 ? nside : 0;
  int seg = (int)blockIdx.x;
  bool is_row;
  int u0, v0;
  if (seg < nrow) {
    is_row = true, u0 = 0, v0 = seg * BORDER_SEG;
  } else if ((seg -= nrow) < nbot) {
    is_row = true, u0 = H - 1, v0 = seg * BORDER_SEG;
  } else if ((seg -= nbot) < nside) {
    is_row = false, u0 = 1 + seg * BORDER_SEG, v0 = 0;
  } else if ((seg -= nside) < nright) {
    is_row = false, u0 = 1 + seg * BORDER_SEG, v0 = W - 1;
  } else {
    return;   // uniform over the block, before any barrier
  }
  const int len = is_row ? min(BORDER_SEG, W - v0) : min(BORDER_SEG, H - 1 - u0);
  if (sd.gbits) {   // a segment without a pixel of the support: nothing reads its g
    const int i = (int)threadIdx.x, u = is_row ? u0 : u0 + i, v = is_row ? v0 + i : v0;
    const bool seen = i < len && (sd.gbits[(size_t)u * support_words(sd) + v / 64] >> (v % 64) & 1);
    if (!__syncthreads_or(seen)) return;
  }
  const int u1 = is_row ? u0 : u0 + len - 1, v1 = is_row ? v0 + len - 1 : v0;
  // window of rho: rows u0 - p .. u1 + p, columns v0 - q .. v1 + q
  const int wr0 = u0 - p, wc0 = v0 - q;
  const int WC = v1 - v0 + 1 + 2 * q, n_win = (u1 - u0 + 1 + 2 * p) * WC;
  const float* __restrict__ Rp = R + loff;
  for (int i = (int)threadIdx.x; i < n_win; i += (int)blockDim.x) {
    const int r = i / WC, gi = wr0 + r, gj = wc0 + (i - r * WC);
    S[i] = (gi >= 0 && gi < H && gj >= 0 && gj < W) ? Rp[(size_t)gi * W + gj] : 0.0f;
  }
  // PW > 0: the four folded tables the segment's pixels use (one row class,
  // every column class; the side columns are all of row class 0) go to LDS too
  const int ntab = sd.ph * pw;
  float* __restrict__ SK = S + border_lds_floats(sd.ph, pw);
  const int t0 = is_row ? 4 * ((H == 1) ? 3 : (u0 == 0 ? 1 : 2)) : 0;
  if (PW > 0)
    for (int i = (int)threadIdx.x; i < 4 * ntab; i += (int)blockDim.x) SK[i] = sd.adjk[(size_t)t0 * ntab + i];
  __syncthreads();
  const int j = (int)threadIdx.x / BORDER_SUB, sub = (int)threadIdx.x % BORDER_SUB;
  float acc = 0.0f;
  const int u = is_row ? u0 : u0 + j, v = is_row ? v0 + j : v0;
  if (j < len) {
    const int cr = (H == 1) ? 3 : (u == 0 ? 1 : (u == H - 1 ? 2 : 0));
    const int cc = (W == 1) ? 3 : (v == 0 ? 1 : (v == W - 1 ? 2 : 0));
    const float* __restrict__ K =
        PW > 0 ? SK + (size_t)(cr * 4 + cc - t0) * ntab : sd.adjk + (size_t)(cr * 4 + cc) * ntab;
    const int a_lo = max(-p, -u), a_hi = min(p, H - 1 - u);
    for (int a = a_lo + sub; a <= a_hi; a += BORDER_SUB) {
      const float* __restrict__ Kr = K + (a + p) * pw;
      const float* __restrict__ Sr = S + (u + a - wr0) * WC + (v - q - wc0);
      if (PW > 0) {
#pragma unroll
        for (int b = 0; b < PW; ++b) acc = fmaf(Kr[b], Sr[b], acc);
      } else {
        for (int b = 0; b < pw; ++b) acc = fmaf(Kr[b], Sr[b], acc);
      }
    }
  }
  acc += __shfl_xor(acc, 2, BORDER_SUB);
  acc += __shfl_xor(acc, 1, BORDER_SUB);
  if (j < len && sub == 0) G[loff + (size_t)u * W + v] = acc;
}

// ---------------------------------------------------------------------------
// Per-subsample partial derivatives.
// ---------------------------------------------------------------------------

// Series of d/ds [atan(sqrt(s) u)/sqrt(s)] and d/ds [atanh(sqrt(s) v)/sqrt(s)] for small s.
__device__ __forceinline__ float datan_ds_series(float s, float u) {
  const float u2 = u * u, z = s * u2;
  // sum_{k>=1} (-1)^k k s^{k-1} u^{2k+1}/(2k+1)
  const float poly = fmaf(z, fmaf(z, fmaf(z, fmaf(z, fmaf(z, -6.0f / 13.0f, 5.0f / 11.0f), -4.0f / 9.0f), 3.0f / 7.0f),
                              -2.0f / 5.0f),
                         1.0f / 3.0f);
  return -u * u2 * poly;
}
__device__ __forceinline__ float datanh_ds_series(float s, float v) {
  const float v2 = v * v, z = s * v2;
  const float poly = fmaf(z, fmaf(z, fmaf(z, fmaf(z, fmaf(z, 6.0f / 13.0f, 5.0f / 11.0f), 4.0f / 9.0f), 3.0f / 7.0f),
                              2.0f / 5.0f),
                         1.0f / 3.0f);
  return v * v2 * poly;
}

template <int DEG>
__device__ __forceinline__ float grad_poly(const float* p, float z) {
  float v = p[DEG];
#pragma unroll
  for (int k = DEG - 1; k >= 0; --k) v = fmaf(v, z, p[k]);
  return v;
}

// Offset of subsample k of N, iN = 1/N: (k + 1/2)/N - 1/2 to a float32 rounding of the
// quotient. The gradient needs the abscissae to float32 accuracy, not bit for bit
// those of the render; but the cusp correction takes back what grad_kernel added, so
// the two share every expression from here to the moments, without contractions that
// a compiler might make in one of them only. (At an odd N that is no power of two the
// middle offset comes out as about 1e-8 of a pixel, where the render's is 0. Where a
// pixel's centre lies on the lens's, that subsample is then deflected and its steep light
// dimmed, unlike in the render: errors of the gradient of 1e-5 to 1e-3 of its norm, and of
// its own size for lens lights of n = 6 and more. (2k + 1 - N)/(2N) would be exact.)
__device__ __forceinline__ float grad_offset(int k, float iN) { return fmaf((float)k + 0.5f, iN, -0.5f); }

// What depends on the row of subsamples only.
struct GradRow {
  float sLy, cLy, rX, rY, h12y, h22y;
  __device__ __forceinline__ GradRow(const GradUniform& U, float y)
      : sLy(U.sL * y), cLy(U.cL * y), rX(fmaf(U.B1, y, U.C1)), rY(fmaf(U.B2, y, U.C2)), h12y(U.h12 * y), h22y(U.h22 * y) {}
};

// One Sersic at frame coordinates (X, Y): E = I/I_e, Et = E t and D = E t/R^2
// (dI/dR^2 = -I_e b e D; 0 at the centre, where t = 0), and its five moments. With NEAR
// D is 0 where R^2 < U.near2.
template <bool WT, bool NEAR>
__device__ __forceinline__ float sersic_moments(const GradUniform& U, float X, float Y, float e, float B, float sw,
                                                float* acc) {
  #pragma clang fp contract(off)
  const float R2 = fmaf(X, X, Y * Y);
  const float L2 = hw_log2(R2);
  const float t = hw_exp2(e * L2);
  float E = hw_exp2(fmaf(-B, t, B));
  if (WT) E *= sw;
  const float Et = E * t;
  const float D = NEAR ? (R2 < U.near2 ? 0.0f : Et * hw_rcp(R2)) : Et * hw_rcp(fmaxf(R2, GRAD_R2_MIN));
  const float DX = D * X;
  acc[0] += E;
  acc[1] += Et;
  acc[2] = fmaf(Et, fmaxf(L2, -200.0f), acc[2]);
  acc[3] = fmaf(DX, X, acc[3]);
  acc[4] = fmaf(DX, Y, acc[4]);
  return D;
}

// Adds the 17 moments of the subsample (x, row) to acc, times the quadrature
// weight sw when WT (a Gauss-Kronrod node). RM is the point's rmode, SER its
// choice of the series in s. With AT, (oX, oY) is the source frame instead of
// the float32 lens equation (the float64 re-traced value near a cuspy source);
// without LIGHT the lens light is left out.
// x'^2 carries U.tiny so that the lens centre needs no branch, as in the forward
// render. With G = D (gXx X + gYx Y, gXy X + gYy Y), which is dI/d beta
// in the SIE frame up to the per-point factor -2 I_e b e:
//   0: a Gx + b Gy   1: the q derivative beyond moment 0   2: (v0 - b) Gx + (a - u0) Gy
//   3: Gx x' - Gy y'   4: Gx y' + Gy x'   5, 6: G   7..11 lens light, 12..16 source:
//   E, E t, E t log2(R^2), D X^2, D X Y
// (D Y^2 is E t - D X^2). The q derivative is Gx (2 da + u0^3 pr) + Gy (2 db +
// v0 u0^2 pr/q^2), pr = psi^2/r^2; with da = (u0 pr - a)/(2s) and db = (v0 pr/q^2 -
// b)/(2s) that is (Gx u0 + Gy v0/q^2) pr (u0^2 + 1/s) - (moment 0)/s.
template <int RM, bool SER, bool WT, bool AT = false, bool LIGHT = true>
__device__ __forceinline__ void subsample_grad(const GradUniform& U, const GradRow& row, float x, float sw,
                                               float (&acc)[NPAR], float oX = 0.0f, float oY = 0.0f) {
#pragma clang fp contract(off)
  const float xp = fmaf(U.cL, x, row.sLy);
  const float yp = fmaf(-U.sL, x, row.cLy);
  const float yp2 = yp * yp;
  const float x2t = fmaf(xp, xp, U.tiny);
  const float r2 = x2t + yp2;
  const float psi2 = RM == 0 ? r2 : fmaf(U.q2, x2t, yp2);
  const float ip = hw_rsq(psi2);
  const float u0 = xp * ip, v0 = yp * ip;
  float a, b, pr;
  if (RM == 0) {
    a = u0;
    b = v0;
    pr = 1.0f;
  } else if (RM == 1) {
    a = u0 * grad_poly<ATAN_SMALL_POLY_DEGREE>(U.P, u0 * u0);
    b = v0 * grad_poly<ATANH_POLY_DEGREE>(U.Q, v0 * v0);
    pr = psi2 * hw_rcp(r2);
  } else {
    const float ir = hw_rsq(r2);
    const float psi = psi2 * ip;
    const float w = xp * hw_rcp(fmaf(r2, ir, psi));
    a = w * grad_poly<RM == 2 ? ATAN_SMALL_POLY_DEGREE : ATAN_UNIT_POLY_DEGREE>(U.P, w * w);
    b = copysignf(fmaf(U.kb, hw_log2(fmaf(U.qp, fabsf(yp), psi) * ir), U.kc), yp);
    const float pq = psi * ir;
    pr = pq * pq;
  }
  const float X = AT ? oX : fmaf(U.Xa, a, fmaf(U.Xb, b, fmaf(U.A1, x, row.rX)));
  const float Y = AT ? oY : fmaf(U.Ya, a, fmaf(U.Yb, b, fmaf(U.A2, x, row.rY)));
  const float D = sersic_moments<WT, !AT>(U, X, Y, U.se, U.sB, sw, acc + 12);
  const float DX = D * X, DY = D * Y;
  const float Gx = fmaf(U.gXx, DX, U.gYx * DY), Gy = fmaf(U.gXy, DX, U.gYy * DY);
  acc[0] = fmaf(b, Gy, fmaf(a, Gx, acc[0]));
  if (SER) {
    const float u2pr = u0 * u0 * pr;
    const float da = datan_ds_series(U.s, u0), db = datanh_ds_series(U.s, v0);
    acc[1] = fmaf(Gx, fmaf(2.0f, da, u0 * u2pr), acc[1]);
    acc[1] = fmaf(Gy, fmaf(2.0f, db, v0 * u2pr * U.iq2), acc[1]);
  } else {
    acc[1] = fmaf(fmaf(Gx, u0, Gy * (v0 * U.iq2)), pr * fmaf(u0, u0, U.hs2), acc[1]);
  }
  acc[2] = fmaf(a - u0, Gy, fmaf(v0 - b, Gx, acc[2]));
  acc[3] = fmaf(-Gy, yp, fmaf(Gx, xp, acc[3]));
  acc[4] = fmaf(Gy, xp, fmaf(Gx, yp, acc[4]));
  acc[5] += Gx;
  acc[6] += Gy;
  if (LIGHT)
    (void)sersic_moments<WT, false>(U, fmaf(U.h11, x, row.h12y), fmaf(U.h21, x, row.h22y), U.he, U.hB, sw, acc + 7);
}

// Calls f with the point's mode as a type: the choices are per point, taken once
// outside the subsample loops. s < GRAD_SERIES_S implies mode 0 or 1.
template <int RM_, bool SER_>
struct GradMode {
  static constexpr int RM = RM_;
  static constexpr bool SER = SER_;
};
template <class F>
__device__ __forceinline__ void with_mode(int rmode, int series, F f) {
  switch (rmode) {
    case 0: f(GradMode<0, true>()); break;
    case 1:
      if (series) f(GradMode<1, true>());
      else f(GradMode<1, false>());
      break;
    case 2: f(GradMode<2, false>()); break;
    default: f(GradMode<3, false>()); break;
  }
}

// The 17 partials from the moments, for one point, in float64. D of the moments
// stands for dI/dR^2 = -I_e b e D of the light, R^2 = X^2 + Y^2 in its frame.
__device__ void grad_from_moments(const double (&M)[NPAR], const GradConst& gc, double (&g)[NPAR]) {
  const double te = gc.theta[0], q = gc.theta[1], sq = sqrt(q), gam = gc.theta[3];
  const double cL = gc.u.cL, sL = gc.u.sL;
  const double nh = gc.theta[7], ns = gc.theta[14], qh = gc.theta[8], qs = gc.theta[15];
  const double Ih = gc.Ih, Is = gc.Is, bh = gc.bh, bs = gc.bs;
  const double kh = -Ih * bh * (0.5 / nh), ks = -Is * bs * (0.5 / ns);
  const double G = 2.0 * ks;
  const double M0 = G * M[0], M1 = G * (M[1] - (double)gc.u.hs2 * M[0]), M2 = G * M[2], M3 = G * M[3], M4 = G * M[4];
  const double Gx = G * M[5], Gy = G * M[6];
  // the shear angle relative to the SIE frame
  const double ph = 2.0 * ((double)gc.theta[4] - (double)gc.theta[2]);
  const double c2 = cos(ph), s2 = sin(ph);
  g[0] = -sq * M0;
  g[1] = -te * (0.5 / sq * M0 - sq * q * M1);
  g[2] = -te * sq * M2;
  g[3] = -(c2 * M3 + s2 * M4);
  g[4] = -2.0 * gam * (c2 * M4 - s2 * M3);
  g[10] = -(cL * Gx - sL * Gy);
  g[11] = -(sL * Gx + cL * Gy);
  // per light: dR^2/dR_e = -2 R^2/R_e, dR^2/dq = (X^2 - Y^2)/q, dR^2/dphi = 2 (q - 1/q) X Y, and
  // dI/dn = I [b'(1 - t) + b t ln(R^2)/(2 n^2)]
  const double ln2 = 0.693147180559945309417;
  const double *mh = M + 7, *ms = M + 12;
  g[5] = mh[0];
  g[6] = -2.0 / gc.theta[6] * kh * mh[1];
  g[7] = Ih * ((double)gc.dbh * (mh[0] - mh[1]) + bh * (0.5 / (nh * nh)) * ln2 * mh[2]);
  g[8] = kh * (2.0 * mh[3] - mh[1]) / qh;
  g[9] = 2.0 * kh * (qh - 1.0 / qh) * mh[4];
  g[12] = ms[0];
  g[13] = -2.0 / gc.theta[13] * ks * ms[1];
  g[14] = Is * ((double)gc.dbs * (ms[0] - ms[1]) + bs * (0.5 / (ns * ns)) * ln2 * ms[2]);
  g[15] = ks * (2.0 * ms[3] - ms[1]) / qs;
  g[16] = 2.0 * ks * (qs - 1.0 / qs) * ms[4];
}

// A pixel's subsamples: the N x N midpoints, or the Cartesian square of a
// Gauss-Kronrod rule's N nodes, each weighted by w_i w_j (the pixel weight d^2
// multiplies later).
template <bool GK>
__device__ __forceinline__ void pixel_grad(int rmode, const GradUniform& U, int rule, int N, const PixelGeom& g,
                                           float (&acc)[NPAR]) {
  with_mode(rmode, U.series, [&](auto mode) {
    using M = decltype(mode);
    if (GK) {
      const GkRule& R = kGkRules[rule - 1];
      for (int ky = 0; ky < N; ++ky) {
        const GradRow row(U, fmaf(g.uy + R.x[ky], g.d, g.cy));
        for (int kx = 0; kx < N; ++kx)
          subsample_grad<M::RM, M::SER, true>(U, row, fmaf(g.ux + R.x[kx], g.d, g.cx), R.w[kx] * R.w[ky], acc);
      }
    } else {
      const float iN = 1.0f / (float)N;
      for (int ky = 0; ky < N; ++ky) {
        const GradRow row(U, fmaf(g.uy + grad_offset(ky, iN), g.d, g.cy));
        for (int kx = 0; kx < N; ++kx)
          subsample_grad<M::RM, M::SER, false>(U, row, fmaf(g.ux + grad_offset(kx, iN), g.d, g.cx), 1.0f, acc);
      }
    }
  });
}

// Sum over the 16 lanes of a row (row rotations), in each of them.
template <int R>
__device__ __forceinline__ float add_rotated(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x120 + R, 0xf, 0xf, true));
}
template <int R>
__device__ __forceinline__ double add_rotated(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x120 + R, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x120 + R, 0xf, 0xf, true);
  return v + __hiloint2double(hi, lo);
}
template <class T>
__device__ __forceinline__ T row_sum(T v) {
  return add_rotated<1>(add_rotated<2>(add_rotated<4>(add_rotated<8>(v))));
}
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// One thread per pixel, one block per (point, render tile): sums
// g_pix * d^2/N^2 * dI/dtheta over the pixel's subsamples, then over the block.
// What bounds it: the issue rate, 117 vector instructions a subsample by the counters
// (11.5 of them transcendental; what a pixel and the block sums take is among them); 187
// before the source frame, the deflection polynomials and every per-point factor of the
// partials were folded into constants, and the q derivative and Y^2 taken from other
// moments. 1024 points
// of 200 x 200 pixels (41 % of them in the support), N = 4: 1107 -> 745 us, 30 us of it
// from the block sums by 16 lanes a moment instead of a wave. Six waves per SIMD hide
// the transcendental chains; five and seven measured the same.
__global__ __launch_bounds__(RENDER_BLOCK, 6) void grad_kernel(WorkArgs w, const PointConst* __restrict__ pcs,
                                                             const GradConst* __restrict__ gcs,
                                                             const float* __restrict__ G,
                                                             const int* __restrict__ gpbase,
                                                             float2* __restrict__ gpart) {
  static_assert(RENDER_BLOCK == 256, "the block sums take 16 entries per lane");
  __shared__ float part[NPAR][RENDER_BLOCK + 16];   // four moments' 16 entries in different banks
  int point, tile;
  resolve(w, point, tile);
  const SysDesc sd = w.sys_table ? w.sys_table[w.point_sys ? w.point_sys[point] : 0] : w.single;
  const int64_t loff = w.point_loff ? w.point_loff[point] : 0;
  const PointConst& c = pcs[point];
  const GradConst& gc = gcs[point];
  const GradUniform& U = gc.u;

  const int base = gpbase ? gpbase[point] : 0;
  const int n_sup = grad_support_count(sd);
  if (tile * RENDER_BLOCK >= n_sup) {   // past the support's last pixel: zero sums
    if ((int)threadIdx.x < NPAR) gpart[(size_t)(base + tile) * NPAR + threadIdx.x] = make_float2(0.0f, 0.0f);
    return;
  }
  float acc[NPAR];
#pragma unroll
  for (int k = 0; k < NPAR; ++k) acc[k] = 0.0f;
  const int unit = tile * RENDER_BLOCK + (int)threadIdx.x;
  const int64_t goff = w.point_goff ? w.point_goff[point] : loff;   // the composite model's g
  if (unit < n_sup) {
    const int pix = grad_support_pixel(sd, unit);
    const float gp = G[goff + pix];
    if (gp != 0.0f) {   // pixels outside the reach of any weighted residual add nothing
      const int r = row_of(sd, pix);
      const int col = pix - r * sd.W;
      PixelGeom geo;
      geo.ux = (float)col - 0.5f * (float)(sd.W - 1);
      geo.uy = (float)r - 0.5f * (float)(sd.H - 1);
      geo.d = sd.d;
      geo.cx = sd.cx;
      geo.cy = sd.cy;
      if (sd.rule == 0)
        pixel_grad<false>(c.rmode, U, 0, sd.N, geo, acc);
      else
        pixel_grad<true>(c.rmode, U, sd.rule, sd.N, geo, acc);
      const float wgt = (float)sd.wgt * gp;
#pragma unroll
      for (int k = 0; k < NPAR; ++k) acc[k] *= wgt;
    }
  }
  // block sums of the 17 moments: the threads' float32 sums go to LDS, 16 lanes
  // add a moment's in float64 (16 entries each, then row rotations; float64 holds
  // the sum of 256 float32 values exactly enough that no cancellation is lost),
  // stored as a float32 pair hi + lo
#pragma unroll
  for (int k = 0; k < NPAR; ++k) part[k][threadIdx.x] = acc[k];
  __syncthreads();
  const int j = (int)threadIdx.x & 15;
  for (int k = (int)threadIdx.x >> 4; k < NPAR; k += RENDER_BLOCK / 16) {
    double v0 = 0.0, v1 = 0.0;
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
      v0 += (double)part[k][16 * i + j];
      v1 += (double)part[k][16 * i + 16 + j];
    }
    const double v = row_sum(v0 + v1);
    if (j == 0) {
      const float hi = (float)v;
      gpart[(size_t)(base + tile) * NPAR + k] = make_float2(hi, (float)(v - (double)hi));
    }
  }
}

// Cusp correction of the gradient: the waves the forward render flagged (same
// pixels, same float32 test) get, for each subsample in the cusp zone, the
// partials at the float64 re-traced source offset minus the float32 ones,
// weighted by g d^2/N^2 (midpoint rule) or g d^2 w_i w_j (Gauss-Kronrod) and
// added to corr[point][k] in float64.
constexpr int GCUSP_WAVES = 4;
constexpr int GCUSP_BLOCKS = 1024;

// As in the forward correction, the entry's flagged pixels go to LDS, the (pixel,
// subsample) pairs inside the radius are found 64 at a time in float32 and queued,
// and the queue is re-traced 64 at a time, so that every stage runs with every lane
// busy. What bounds it: at few points the latency of one entry's chain, at many the
// registers of the moments (four waves per SIMD). 1024 points of 200 x 200 pixels,
// N = 4: 93 -> 24 us (32 us at three waves); 16 points of 87 x 101, N = 3: 16.4 -> 7.5 us.
// (Each lane testing its own pixel's subsamples one after another, with few of the 64
// pixels flagged, took 73 us with the same re-tracing.)
constexpr int GCUSP_CHUNK = 16;   // subsamples per pass

__device__ __forceinline__ PixelGeom gcusp_geom(const SysDesc& sd, int pix) {
  const int r = row_of(sd, pix);
  const int col = pix - r * sd.W;
  PixelGeom geo;
  geo.ux = (float)col - 0.5f * (float)(sd.W - 1);
  geo.uy = (float)r - 0.5f * (float)(sd.H - 1);
  geo.d = sd.d;
  geo.cx = sd.cx;
  geo.cy = sd.cy;
  return geo;
}

__global__ __launch_bounds__(64 * GCUSP_WAVES, 4) void grad_cusp_kernel(WorkArgs w, const PointConst* __restrict__ pcs,
                                                                     const PointConst64* __restrict__ p64s,
                                                                     const GradConst* __restrict__ gcs,
                                                                     const float* __restrict__ G, CuspList cl,
                                                                     double* __restrict__ corr) {
  __shared__ unsigned short queue[GCUSP_WAVES][GCUSP_CHUNK * 64];   // flagged pixel | subsample << 6
  __shared__ int fpix[GCUSP_WAVES][64];                             // the entry's flagged pixels
  const int n = *cl.count;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  // a scalar, so that an entry's point and its constants are read with uniform addresses
  const int wave = uniform((int)blockIdx.x * GCUSP_WAVES + wv);
  unsigned short* __restrict__ qu = queue[wv];
  int* __restrict__ fp = fpix[wv];
  for (int i = wave; i < n; i += gridDim.x * GCUSP_WAVES) {
    const CuspEntry e = cl.entries[i];
    const bool mine = (e.mask >> lane) & 1ull;
    const int F = __popcll(e.mask);
    const int point = uniform(e.point);
    const SysDesc& sd = w.sys_table ? w.sys_table[w.point_sys ? w.point_sys[point] : 0] : w.single;
    const int64_t loff = w.point_loff ? w.point_loff[point] : 0;
    const int64_t goff = w.point_goff ? w.point_goff[point] : loff;   // the composite model's g
    const PointConst& c = pcs[point];
    const GradConst& gc = gcs[point];
    const GradUniform& U = gc.u;
    if (mine) fp[__popcll(e.mask & ((1ull << lane) - 1ull))] = unit_pixel(sd, e.unit0 + lane, e.ppt) + e.half;
    wave_lds_sync();
    const int N = sd.N, NN = N * N;
    const GkRule* Rg = sd.rule > 0 ? &kGkRules[sd.rule - 1] : nullptr;
    float acc[NPAR];
#pragma unroll
    for (int k = 0; k < NPAR; ++k) acc[k] = 0.0f;
    for (int s0 = 0; s0 < NN; s0 += GCUSP_CHUNK) {
      const int ns = min(GCUSP_CHUNK, NN - s0);
      int qn = 0;
      for (int b = 0; b < F * ns; b += 64) {
        const int item = b + lane;
        bool within = false;
        int f = 0, j = 0;
        if (item < F * ns) {
          f = item / ns;
          j = item - f * ns;
          const int ky = (s0 + j) / N, kx = s0 + j - ky * N;
          const PixelGeom geo = gcusp_geom(sd, fp[f]);
          const int prow = row_of(sd, fp[f]);
          const float y = fmaf(geo.uy + (Rg ? Rg->x[ky] : sub_offset_rt(ky, N)), geo.d, geo.cy);
          const float x = fmaf(geo.ux + (Rg ? Rg->x[kx] : sub_offset_rt(kx, N)), geo.d, geo.cx);
          // with the render constants the forward render used for the pixel
          within = render_source_R2(c, c.rv[render_variant(prow, fp[f] - prow * sd.W)], x, y) < c.cusp_r2;
        }
        const unsigned long long bal = __ballot(within);
        if (within) qu[qn + __popcll(bal & ((1ull << lane) - 1ull))] = (unsigned short)(f | (j << 6));
        qn += __popcll(bal);
      }
      wave_lds_sync();
      for (int q0 = 0; q0 < qn; q0 += 64) {
        if (q0 + lane < qn) {
          const int item = qu[q0 + lane];
          const int j = item >> 6;
          const int ky = (s0 + j) / N, kx = s0 + j - ky * N;
          const int qpix = fp[item & 63];
          const PixelGeom gq = gcusp_geom(sd, qpix);
          const float iN = 1.0f / (float)N;
          const float y = fmaf(gq.uy + (Rg ? Rg->x[ky] : grad_offset(ky, iN)), gq.d, gq.cy);
          const float x = fmaf(gq.ux + (Rg ? Rg->x[kx] : grad_offset(kx, iN)), gq.d, gq.cx);
          // the middle subsample of an odd N in a pixel centred on the lens (y and x may miss it
          // by 1e-8 of a pixel): no deflection there, while 1e-8 of a pixel off it is
          // theta_E and would multiply the steep source's gradient
          const bool centre = 2 * ky + 1 == N && 2 * kx + 1 == N && fmaf(gq.uy, gq.d, gq.cy) == 0.0f &&
                              fmaf(gq.ux, gq.d, gq.cx) == 0.0f;
          const double oy = Rg ? Rg->xd[ky] : ((double)ky + 0.5) / N - 0.5;
          const double ox = Rg ? Rg->xd[kx] : ((double)kx + 0.5) / N - 0.5;
          const float sw = Rg ? Rg->w[kx] * Rg->w[ky] : 1.0f;
          float dx, dy;
          source_offset_f64(p64s[point], gq, ox, oy, dx, dy);
          float diff[NPAR];   // moments at the float32 offset minus those at the float64 one
#pragma unroll
          for (int k = 0; k < NPAR; ++k) diff[k] = 0.0f;
          const float X = fmaf(U.s11, dx, U.s12 * dy), Y = fmaf(U.s21, dx, U.s22 * dy);
          with_mode(c.rmode, U.series, [&](auto mode) {
            using M = decltype(mode);
            const GradRow row(U, y);
            subsample_grad<M::RM, M::SER, true, true, false>(U, row, x, sw, diff, X, Y);
#pragma unroll
            for (int k = 0; k < NPAR; ++k) diff[k] = centre && k < 5 ? 0.0f : -diff[k];   // 0..4: the deflection's
            subsample_grad<M::RM, M::SER, true, false, false>(U, row, x, sw, diff);
          });
          const float wg = -(float)sd.wgt * G[goff + qpix];
#pragma unroll
          for (int k = 0; k < NPAR; ++k) acc[k] = fmaf(diff[k], wg, acc[k]);
        }
      }
      wave_lds_sync();
    }
    // every lane of an entry belongs to the same point; a lane per moment adds its sum
    float mine_sum = 0.0f;
#pragma unroll
    for (int k = 0; k < NPAR; ++k) {
      const float v = row_sum(acc[k]);
      const float sum = (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
      mine_sum = lane == k ? sum : mine_sum;
    }
    if (lane < NPAR && mine_sum != 0.0f) atomicAdd(&corr[(size_t)point * NPAR + lane], (double)mine_sum);
    wave_lds_sync();   // the queue and the pixel list are written anew
  }
}

// One block per point: wave w sums the moments k = w, w + 4, ... over the
// point's render tiles (hi + lo, float64, lanes striding over the tiles, then
// a fixed shuffle tree) and adds the cusp correction.
constexpr int FGRAD_THREADS = 256;

// With magnitudes, slots 5 and 12 of the sums hold d log L / d I_e and slots
// 6, 7 and 13, 14 the derivatives at fixed I_e; the chain rule through
// I_e(m, R_e, n) gives d/dm = g_I I_e dlnI/dm and adds g_I I_e dlnI/dR_e and
// g_I I_e dlnI/dn to the radius and index entries. With an image-plane source
// position, slots 10 and 11 hold d log L / d beta; the chain rule through
// beta(x_I, y_I, theta_E, q_L, phi_L, gamma, phi_gamma) gives d/dx_I, d/dy_I and
// adds g_beta . d beta / d theta_k to the five lens entries.
__global__ __launch_bounds__(FGRAD_THREADS) void finalize_grad_kernel(
    const float2* __restrict__ gpart, const int* __restrict__ gpbase, int ntiles, const double* __restrict__ corr,
    const GradConst* __restrict__ gcs, float* __restrict__ grad, int point_base) {
  __shared__ double M[NPAR];
  const int p = point_base + (int)blockIdx.x;
  const int base = gpbase ? gpbase[p] : 0;
  const int lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
  for (int k = wv; k < NPAR; k += FGRAD_THREADS / 64) {
    double s = 0.0;
    for (int i = lane; i < ntiles; i += 64) {
      const float2 v = gpart[(size_t)(base + i) * NPAR + k];
      s += (double)v.x + (double)v.y;
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if (lane == 0) M[k] = s + (corr ? corr[(size_t)p * NPAR + k] : 0.0);
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  double g[NPAR];
  const GradConst& gc = gcs[p];
  grad_from_moments(M, gc, g);
  if (gc.srcpos) {
    const float* J = gc.src_jac;
    const double gx = g[10], gy = g[11];
    for (int k = 0; k <= 4; ++k) g[k] += gx * (double)J[k + 2] + gy * (double)J[7 + k + 2];
    g[10] = gx * (double)J[0] + gy * (double)J[7];
    g[11] = gx * (double)J[1] + gy * (double)J[8];
  }
  if (gc.amp) {
    const double gIh = g[5], gIs = g[12];
    g[5] = gIh * (double)gc.amp_chain[0];
    g[6] += gIh * (double)gc.amp_chain[1];
    g[7] += gIh * (double)gc.amp_chain[2];
    g[12] = gIs * (double)gc.amp_chain[3];
    g[13] += gIs * (double)gc.amp_chain[4];
    g[14] += gIs * (double)gc.amp_chain[5];
  }
  for (int k = 0; k < NPAR; ++k) grad[(size_t)p * NPAR + k] = (float)g[k];
}

}  // namespace

hipError_t launch_adjoint_psf(const WorkArgs& w, const float* R, float* G, int n_blocks, int TW, int TH, int ph,
                              int pw, int n_points, int H, int W, hipStream_t st) {
  if (n_blocks <= 0) return hipSuccess;
  const int threads = psf_threads(TW, TH);
  const size_t lds = psf_lds_bytes(TW, TH, ph, pw);
  if (threads > PSF_MAX_THREADS || lds > PSF_MAX_LDS || TH % (4 * PSF_Q) != 0 || TW % PSF_C != 0)
    return hipErrorInvalidValue;
  const hipError_t e = with_psf_steps(ph, [&](auto steps) {
    constexpr int KP = decltype(steps)::value;
    return for_item_parts(w, n_blocks, [&](const WorkArgs& part, int n) {
      hipLaunchKernelGGL((adj_psf_kernel<KP>), dim3(n), dim3(threads), lds, st, part, R, G);
      return hipGetLastError();
    });
  });
  if (e != hipSuccess) return e;
  const int nseg = border_segments(H, W);
  // the window, and with 21-wide tables also the four tables of a segment
  const size_t blds = (size_t)(border_lds_floats(ph, pw) + (pw == 21 ? 4 * ph * pw : 0)) * sizeof(float);
  // one grid row per point, at most 65535 rows per launch
  for (int p0 = 0; p0 < n_points; p0 += 65535) {
    const int np = n_points - p0 < 65535 ? n_points - p0 : 65535;
    if (pw == 21)
      hipLaunchKernelGGL(adj_border_kernel<21>, dim3((unsigned)nseg, np), dim3(BORDER_SEG * BORDER_SUB), blds, st, w,
                         R, G, p0);
    else
      hipLaunchKernelGGL(adj_border_kernel<0>, dim3((unsigned)nseg, np), dim3(BORDER_SEG * BORDER_SUB), blds, st, w,
                         R, G, p0);
    const hipError_t le = hipGetLastError();
    if (le != hipSuccess) return le;
  }
  return hipSuccess;
}

// The lists of the adjoint's support from its bits (support.h), and zeros in the
// unconvolved image of every point outside its system's support: a gradient plan
// renders only the support, and the PSF stage, which multiplies w = 0 by its
// outputs there, must read finite values, not what an earlier launch left (a NaN
// point's image, or g). Both need only the bits, so one launch does both: the
// first list_blocks blocks of each system write COMPACT_SEGMENTS row segments'
// pixels and units each (their first slots are the counts of the segments before,
// summed by each block), the others clear CLEAR_WORDS words of a point each.
// Only the windows of the PSF tiles with w > 0 are read, so only those are cleared.
// What bounds it: the launch, and at many points the zeros. The row, column,
// list and clear passes it replaces took 31.4 us at 16 points of 87 x 101 pixels and
// 106 us at 1024 of 200 x 200; now 7.9 and 25.8 us, and the prologue as long as before
// at 16 points, 4 us longer at 1024 (4 blocks of 8 rows fit a compute unit).
constexpr int COMPACT_SEGMENTS = 16;
constexpr int CLEAR_WORDS = 256;   // 64 a wave
static_assert(COMPACT_SEGMENTS % (SUPPORT_THREADS / 64) == 0 && CLEAR_WORDS == SUPPORT_THREADS, "per wave");

__device__ unsigned long long word_of_lane(unsigned long long v, int lane) {
  return (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, lane) |
         (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(v >> 32), lane) << 32;
}

__device__ void support_lists(SysDesc& sd, int block, int2 (&wsum)[SUPPORT_THREADS / 64]) {
  // every field before the first store, which may alias the descriptor
  int* gsup = sd.gsup;
  int* uact = sd.uact;
  const unsigned long long* gbits = sd.gbits;
  const int2* gcount = sd.gcount;
  const int W = sd.W, uppt = sd.uppt;
  const int nseg = support_segments(sd), nw = support_words(sd), total = sd.H * nseg;
  if (!gsup) return;
  const int e0 = block * COMPACT_SEGMENTS;
  if (e0 >= total) return;   // uniform over the block, before its barrier
  const int t = (int)threadIdx.x, wv = t >> 6, lane = t & 63;
  int2 before = make_int2(0, 0);
  for (int i = t; i < e0; i += SUPPORT_THREADS) {
    const int2 c = gcount[i];
    before.x += c.x;
    before.y += c.y;
  }
  for (int o = 32; o > 0; o >>= 1) {
    before.x += __shfl_xor(before.x, o, 64);
    before.y += __shfl_xor(before.y, o, 64);
  }
  if (lane == 0) wsum[wv] = before;
  int2 own = make_int2(0, 0);
  if (lane < COMPACT_SEGMENTS && e0 + lane < total) own = gcount[e0 + lane];
  __syncthreads();
  before = wsum[0];
  for (int k = 1; k < SUPPORT_THREADS / 64; ++k) {
    before.x += wsum[k].x;
    before.y += wsum[k].y;
  }
  constexpr int PER_WAVE = COMPACT_SEGMENTS / (SUPPORT_THREADS / 64);
  const unsigned long long below = (1ull << lane) - 1ull;
  for (int k = 0; k < COMPACT_SEGMENTS; ++k) {
    if (k / PER_WAVE == wv && e0 + k < total) {
      const int row = (e0 + k) / nseg, w0 = (e0 + k - row * nseg) * SUPPORT_SEG_WORDS;
      unsigned long long words = 0;
      if (lane < SUPPORT_SEG_WORDS && w0 + lane < nw) words = gbits[(size_t)row * nw + w0 + lane];
      int px = before.x, un = before.y;
      for (int j = 0; j < SUPPORT_SEG_WORDS; ++j) {
        const unsigned long long bits = word_of_lane(words, j);
        const unsigned long long units = uppt == 2 ? (bits | bits >> 1) & 0x5555555555555555ull : bits;
        const int pix = row * W + 64 * (w0 + j) + lane;
        if (bits >> lane & 1) gsup[px + __popcll(bits & below)] = pix;
        if (uact && (units >> lane & 1)) uact[un + __popcll(units & below)] = pix;
        px += __popcll(bits);
        un += __popcll(units);
      }
    }
    before.x += __builtin_amdgcn_readlane(own.x, k);
    before.y += __builtin_amdgcn_readlane(own.y, k);
  }
  if (e0 + COMPACT_SEGMENTS >= total && t == 0) {
    *sd.gsup_n = before.x;
    if (uact) sd.n_active = before.y;
  }
}

__global__ __launch_bounds__(SUPPORT_THREADS) void grad_support_kernel(WorkArgs w, SysDesc* sys,
                                                                       float* __restrict__ L, int list_blocks,
                                                                       int n_lists, int clear_blocks, int point_base) {
  if ((int)blockIdx.x < n_lists) {
    __shared__ int2 wsum[SUPPORT_THREADS / 64];
    support_lists(sys[blockIdx.x / list_blocks], blockIdx.x % list_blocks, wsum);
    return;
  }
  const int b = (int)blockIdx.x - n_lists, pt = b / clear_blocks;
  const int point = point_base + pt;
  const SysDesc& sd = w.sys_table[w.point_sys ? w.point_sys[point] : 0];
  if (!sd.uact) return;
  const int lane = (int)threadIdx.x & 63, W = sd.W, nw = support_words(sd), total = sd.H * nw;
  const int first = (b - pt * clear_blocks) * CLEAR_WORDS + ((int)threadIdx.x & ~63);
  if (first >= total) return;
  float* img = L + w.point_loff[point];
  // lane i: the pixels of word first + i to clear: those outside the support, where
  // the windows of the PSF tiles with w > 0, the only ones that are read, reach
  unsigned long long clear = 0;
  int at = 0;
  if (first + lane < total) {
    const int r = (first + lane) / nw, c = 64 * (first + lane - r * nw), p = sd.ph / 2, q = sd.pw / 2;
    const int above = r + p - psf_tile_rows(sd.TH, psf_steps(sd.ph));   // the last row before a window ending at r
    const int ty0 = above < 0 ? 0 : above / sd.TH + 1, ty1 = min(r + p, sd.H - 1) / sd.TH;
    const int tx1 = min(c + 63 + q, W - 1) / sd.TW;
    bool read = false;
    for (int ty = ty0; ty <= ty1; ++ty)
      for (int tx = max(c - q, 0) / sd.TW; tx <= tx1; ++tx) read = read || (sd.ptile_w[ty * sd.tiles_x + tx] & PTILE_W);
    at = r * W + c;
    if (read) clear = ~sd.gbits[first + lane] & (~0ull >> max(c + 64 - W, 0));
  }
  for (unsigned long long todo = __ballot(clear != 0); todo; todo &= todo - 1) {
    const int i = __builtin_ctzll(todo);
    if (word_of_lane(clear, i) >> lane & 1) img[__builtin_amdgcn_readlane(at, i) + lane] = 0.0f;
  }
}

hipError_t launch_grad_support(const WorkArgs& w, SysDesc* sys, int n_sys, const SupportSizes& n, float* L,
                               int n_points, hipStream_t st) {
  if (n_sys <= 0 || n.segments <= 0) return hipSuccess;
  const int list_blocks = (n.segments + COMPACT_SEGMENTS - 1) / COMPACT_SEGMENTS;
  const int clear_blocks = (n.words + CLEAR_WORDS - 1) / CLEAR_WORDS;
  const int per_launch = std::max(1, (1 << 23) / clear_blocks);   // points per launch, at most 2^23 blocks
  for (int p0 = 0; p0 == 0 || p0 < n_points; p0 += per_launch) {
    const int np = std::min(per_launch, n_points - p0), n_lists = p0 == 0 ? n_sys * list_blocks : 0;
    hipLaunchKernelGGL(grad_support_kernel, dim3((unsigned)(n_lists + np * clear_blocks)), dim3(SUPPORT_THREADS), 0, st,
                       w, sys, L, list_blocks, n_lists, clear_blocks, p0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

__global__ __launch_bounds__(256) void grad_sky_kernel(const float* __restrict__ R, const int64_t* __restrict__ loff,
                                                        const int* __restrict__ point_sys,
                                                        const SysDesc* __restrict__ sys, int K,
                                                        float* __restrict__ grad_sky, int model_base) {
  __shared__ double part[256];
  const int m = model_base + (int)blockIdx.x;
  const int64_t p0 = (int64_t)m * K;
  const SysDesc& sd = sys[point_sys ? point_sys[p0] : 0];
  const int npix = sd.H * sd.W;
  const float* rho = R + loff[p0];
  double acc = 0.0;
  for (int i = (int)threadIdx.x; i < npix; i += 256) acc += (double)rho[i];
  part[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) grad_sky[m] = (float)(part[0] * (double)sd.d * (double)sd.d);
}

hipError_t launch_grad_sky(const float* R, const int64_t* loff, const int* point_sys, const SysDesc* sys, int K,
                           int n_models, float* grad_sky, hipStream_t st) {
  for (int m0 = 0; m0 < n_models; m0 += 1 << 20) {   // at most 2^20 blocks per launch
    const int nm = n_models - m0 < (1 << 20) ? n_models - m0 : (1 << 20);
    hipLaunchKernelGGL(grad_sky_kernel, dim3((unsigned)nm), dim3(256), 0, st, R, loff, point_sys, sys, K, grad_sky,
                       m0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_grad(const WorkArgs& w, const PointConst* pcs, const PointConst64* p64s, const GradConst* gcs,
                       const float* G, const int* gpbase, float2* gpart, int n_blocks, const CuspList& cl,
                       double* corr, hipStream_t st, hipEvent_t between) {
  if (n_blocks <= 0) return between ? hipEventRecord(between, st) : hipSuccess;
  hipError_t e = for_item_parts(w, n_blocks, [&](const WorkArgs& part, int n) {
    hipLaunchKernelGGL(grad_kernel, dim3(n), dim3(RENDER_BLOCK), 0, st, part, pcs, gcs, G, gpbase, gpart);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  if (between && (e = hipEventRecord(between, st)) != hipSuccess) return e;
  const int waves = n_blocks * (RENDER_BLOCK / 64);
  int grid = (waves + GCUSP_WAVES - 1) / GCUSP_WAVES;
  if (grid > GCUSP_BLOCKS) grid = GCUSP_BLOCKS;
  hipLaunchKernelGGL(grad_cusp_kernel, dim3(grid), dim3(64 * GCUSP_WAVES), 0, st, w, pcs, p64s, gcs, G, cl, corr);
  return hipGetLastError();
}

hipError_t launch_finalize_grad(const float2* gpart, const int* gpbase, int ntiles, int n_points, const double* corr,
                                const GradConst* gcs, float* grad, hipStream_t st) {
  if (n_points <= 0) return hipSuccess;
  // at most 2^20 blocks per launch (the grid stays far below 2^32 work-items)
  for (int p0 = 0; p0 < n_points; p0 += 1 << 20) {
    const int np = n_points - p0 < (1 << 20) ? n_points - p0 : (1 << 20);
    hipLaunchKernelGGL(finalize_grad_kernel, dim3((unsigned)np), dim3(FGRAD_THREADS), 0, st, gpart, gpbase, ntiles,
                       corr, gcs, grad, p0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace lensed
