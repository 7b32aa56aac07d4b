// prologue.hip -- per-point derived constants and PSF normalisation.
//
// Half a wave per parameter point turns its 17 float32 parameters into the
// wave-uniform constants the render kernels consume (trigonometry, the shear
// matrix, reciprocal radii and the Sersic b_n, where R_e is the half-light
// radius, Sec. 4.1 Eq. 22). Extra blocks normalise each system's PSF to unit sum
// (Sec. 3.1).
//
// What bounds it: latency. The launch holds a few waves per SIMD even at 4096
// points, and every call waits for it, so what counts is the longest chain of
// dependent float64 operations, not the rate. So the lanes take one sine and
// cosine, one light component's roots and reciprocals, and one folded
// constant's roundings each, and b_n is a polynomial from a table.
// (The gradient's instance keeps the PSF's summed-area table in the LDS that the points'
// blocks share, 33 KB, and spills 64 bytes a thread; at 1024 points its 179 blocks have a
// compute unit each all the same.)
// One point with a 21 x 21 PSF 17.6 -> 5.2 us, 4096 points 32.5 -> 8.5 us; 16 points
// with the adjoint's tables 31.3 -> 7.1 us (two launches before); a general model's
// 256 points 33.3 -> 5.9 us (three launches before).
#include <math.h>

#include "bn_poly.h"
#include "internal.h"
#include "kernels.h"
#include "sie64.h"
#include "sie_poly.h"
#include "support.h"

namespace lensed {
namespace {

// b_n, the root of P(2n, b) = 1/2, and db_n/dn for 0.2 <= n <= 10: the polynomial
// of n's quarter octave (fit_bn.py; both within 4e-16 relative). An iteration on
// the incomplete gamma function's series to the same accuracy runs hundreds of
// dependent operations.
struct SersicBn {
  double b, db;
};
__device__ SersicBn sersic_bn(double n) {
  const int hi = __double2hiint(n), e = (hi >> 20) - 1023;
  const double* c = BN_POLY[(hi >> 18) - ((1023 + BN_E_MIN) << 2)];
  const double mid = __hiloint2double((hi & ~0x3ffff) | 0x20000, 0), scale = __hiloint2double((1026 - e) << 20, 0);
  const double t = (n - mid) * scale;
  double v = c[BN_DEGREE], d = 0.0;
#pragma unroll
  for (int k = BN_DEGREE - 1; k >= 0; --k) {
    d = __builtin_fma(d, t, v);
    v = __builtin_fma(v, t, c[k]);
  }
  return {v, d * scale};
}

// Digamma psi(z), z > 0: psi(z) = psi(z + 1) - 1/z up to z >= 8, then the
// asymptotic expansion psi(z) ~ ln z - 1/(2z) - sum_k B_2k / (2k z^2k)
// (Abramowitz & Stegun 6.3.18) to z^-12, below 1e-15 relative there.
__device__ double digamma_d(double z) {
  double shift = 0.0;
  while (z < 8.0) {
    shift += 1.0 / z;
    z += 1.0;
  }
  const double w = 1.0 / (z * z);
  const double tail =
      w * (1.0 / 12.0 + w * (-1.0 / 120.0 + w * (1.0 / 252.0 + w * (-1.0 / 240.0 + w * (1.0 / 132.0 + w * (-691.0 / 32760.0))))));
  return log(z) - 0.5 / z - tail - shift;
}

// Sersic amplitude from a total magnitude (Sec. 4.1: the amplitude is set by
// the total magnitude). The elliptical profile with the geometric-mean radius
// has the circular profile's flux F = 2 pi n R_e^2 I_e e^{b} Gamma(2n) / b^{2n},
// and F = 10^{-0.4 (m - zp)}, so
//   ln I_e = -0.4 ln 10 (m - zp) + 2n ln b - ln(2 pi n R_e^2) - b - ln Gamma(2n),
// and with b = b_n(n):
//   d ln I_e/dm = -0.4 ln 10,  d ln I_e/dR_e = -2/R_e,
//   d ln I_e/dn = 2 ln b + (2n/b - 1) db/dn - 1/n - 2 psi(2n).
struct AmpFromMag {
  double I;          // I_e
  double dm, dR, dn; // I_e times the three logarithmic derivatives
};
__device__ AmpFromMag amplitude_from_magnitude(double m, double Re, double n, double b, double db_dn, double zp) {
  const double ln10 = 2.302585092994045684;
  const double two_pi = 6.283185307179586477;
  const double lnI = -0.4 * ln10 * (m - zp) + 2.0 * n * log(b) - log(two_pi * n * Re * Re) - b - lgamma(2.0 * n);
  AmpFromMag a;
  a.I = exp(lnI);
  a.dm = a.I * (-0.4 * ln10);
  a.dR = a.I * (-2.0 / Re);
  a.dn = a.I * (2.0 * log(b) + (2.0 * n / b - 1.0) * db_dn - 1.0 / n - 2.0 * digamma_d(2.0 * n));
  return a;
}

// Lens equation in float64 (Eq. 1): beta = x - alpha_SIE(x) - alpha_shear(x),
// SIE in the area-preserving convention about the origin (alpha = 0 at its
// centre), external shear about the same centre.
__device__ void lens_map_f64(const double (&v)[7], double& bx, double& by) {
  const double x = v[0], y = v[1], te = v[2], q = v[3], ph = v[4], g = v[5], phg = v[6];
  const double c = cos(ph), s = sin(ph);
  const double xp = c * x + s * y, yp = c * y - s * x;
  const double psi = sqrt(q * q * xp * xp + yp * yp);
  double axp = 0.0, ayp = 0.0;
  if (psi > 0.0) {
    const double s2 = (1.0 - q) * (1.0 + q);
    if (s2 > 0.0) {
      const double qp = sqrt(s2), k = te * sqrt(q) / qp;
      axp = k * atan(qp * xp / psi);
      ayp = k * atanh(qp * yp / psi);
    } else {
      axp = te * xp / psi;
      ayp = te * yp / psi;
    }
  }
  const double g1 = g * cos(2.0 * phg), g2 = g * sin(2.0 * phg);
  bx = x - (c * axp - s * ayp) - (g1 * x + g2 * y);
  by = y - (s * axp + c * ayp) - (g2 * x - g1 * y);
}

// The source centre beta(v) of an image-plane source position and d beta / d v
// by central differences in float64 (step 1e-6 of the scale: error ~1e-10
// relative); q_L steps backwards with a second-order stencil where a forward
// step would leave q <= 1. Lane 2c + s of the point (s: side) maps its shifted
// v, lane 14 v itself (to maps[lane]); lens_map_slope then combines column c.
__device__ double lens_map_step(const double (&v)[7], int c) {
  double vc = v[0];
#pragma unroll
  for (int i = 1; i < 7; ++i) vc = i == c ? v[i] : vc;
  return 1e-6 * fmax(fabs(vc), 1.0) * (c == 3 ? 0.25 : 1.0);
}
__device__ void lens_map_lane(const double (&v)[7], int lane, double2* maps) {
  const int c = lane >> 1;
  const double h = lens_map_step(v, c);
  const bool back = c == 3 && v[3] + h > 1.0;
  const double shift = back ? ((lane & 1) ? -2.0 * h : -h) : ((lane & 1) ? -h : h);
  double a[7];
#pragma unroll
  for (int i = 0; i < 7; ++i) a[i] = i == c && lane < 14 ? v[i] + shift : v[i];
  lens_map_f64(a, maps[lane].x, maps[lane].y);
}
__device__ void lens_map_slope(const double (&v)[7], int c, const double2* maps, float* jac) {
  const double h = lens_map_step(v, c);
  const double2 a = maps[2 * c], b = maps[2 * c + 1], o = maps[14];
  const bool back = c == 3 && v[3] + h > 1.0;
  const double dx = back ? 3.0 * o.x - 4.0 * a.x + b.x : a.x - b.x;
  const double dy = back ? 3.0 * o.y - 4.0 * a.y + b.y : a.y - b.y;
  jac[c] = (float)(dx / (2.0 * h));
  jac[7 + c] = (float)(dy / (2.0 * h));
}

__device__ bool ok_q(float q) { return q > 0.0f && q <= 1.0f; }
__device__ bool ok_n(float n) { return n >= 0.2f && n <= 10.0f; }

// Float32 roundings of c for the render variants: below() and above() are the
// float32 neighbours of c, and variant v takes the one above for a share of the
// RENDER_VARIANTS variants equal to c's position between the two (so the mean
// over the variants is c to within 1/32 of their gap). Exactly representable
// and non-finite values stay as they are.
struct Dither {
  float lo, hi;
  double frac;
  __device__ explicit Dither(double c) {
    const float f = (float)c;
    lo = hi = f;
    frac = 0.0;
    if (!isfinite(f) || (double)f == c) return;
    if ((double)f < c)
      hi = nextafterf(f, __builtin_inff());
    else
      lo = nextafterf(f, -__builtin_inff());
    // hi - lo is a power of two, so the quotient is an exact scaling
    frac = ldexp(c - (double)lo, -ilogb((double)hi - (double)lo));
  }
  __device__ float variant(int v) const { return frac + ((v + 0.5) / RENDER_VARIANTS - 0.5) >= 0.5 ? hi : lo; }
};

// PSF blocks: one per system, or with the adjoint one per system and border
// class, of PROLOGUE_THREADS threads. The PSF is normalised to unit sum in
// float64 and stored three ways (row-major; column-major flipped, the
// convolution's taps; column-major, the transpose's taps), and for the adjoint
// the 16 folded tables of the transposed convolution. For border class
// cls = 4 cr + cc (0 interior, 1 first, 2 last, 3 both, per axis) the entry at
// offset (a, b) sums the kernel over the offsets the replicate padding maps
// there: first -> offsets a..p, last -> -p..a, both -> all (only a = 0). Each
// such sum is a rectangle of a float64 summed-area table of the PSF, which each
// of the 16 blocks makes for itself: 16 short blocks end long before one that
// fills 16 tables.
constexpr int PROLOGUE_THREADS = 256;
constexpr int PSF_CLASSES = 16;
template <bool ADJ>
struct PsfScratch {
  double part[PROLOGUE_THREADS / 64];
  double sat[ADJ ? (MAX_PSF + 1) * (MAX_PSF + 1) : 1];
};

// Sum of the block's acc, in every thread.
__device__ double block_sum(double acc, double* part) {
  for (int w = 32; w > 0; w >>= 1) acc += __shfl_down(acc, w, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x / 64] = acc;
  __syncthreads();
  double sum = part[0];
  for (int k = 1; k < PROLOGUE_THREADS / 64; ++k) sum += part[k];
  return sum;
}

// 1 / (sum of the PSF); store: also its three normalised copies.
__device__ double psf_normalise(const SysDesc& sd, double* part, bool store) {
  const int n = sd.ph * sd.pw, t = (int)threadIdx.x;
  double acc = 0.0;
  for (int i = t; i < n; i += PROLOGUE_THREADS) acc += (double)sd.psf[i];
  const double inv = 1.0 / block_sum(acc, part);
  if (store)
    for (int i = t; i < n; i += PROLOGUE_THREADS) {
      const int l = i / sd.ph, k = i - l * sd.ph;
      sd.psfn[i] = (float)((double)sd.psf[i] * inv);
      sd.psfn[n + i] = (float)((double)sd.psf[(sd.ph - 1 - k) * sd.pw + (sd.pw - 1 - l)] * inv);
      sd.psfn[2 * n + i] = (float)((double)sd.psf[k * sd.pw + l] * inv);
    }
  return inv;
}

// Running sums of `count` entries of v, `stride` apart, in place; eight at a
// time, so that the LDS reads of a chunk are in flight together.
__device__ void running_sum(double* v, int count, int stride) {
  double r = 0.0;
  for (int j0 = 0; j0 < count; j0 += 8) {
    double x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = j0 + u < count ? v[(j0 + u) * stride] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      r += x[u];
      if (j0 + u < count) v[(j0 + u) * stride] = r;
    }
  }
}

__device__ void psf_adjoint_class(const SysDesc& sd, int cls, PsfScratch<true>& s) {
  const int n = sd.ph * sd.pw, t = (int)threadIdx.x;
  const int SW = sd.pw + 1, SH = sd.ph + 1;
  // S[i][j] = sum of psf[a][b] over a < i, b < j: row sums, then column sums
  for (int i = t; i < SW * SH; i += PROLOGUE_THREADS) {
    const int r = i / SW, c = i - r * SW;
    s.sat[i] = r > 0 && c > 0 ? (double)sd.psf[(r - 1) * sd.pw + c - 1] : 0.0;
  }
  const double inv = psf_normalise(sd, s.part, cls == 0);   // its barrier ends the staging
  if (!sd.adjk) return;   // uniform over the block
  const int cr = cls >> 2, cc = cls & 3;
  if (cls) {
    if (t < SH) running_sum(s.sat + t * SW, SW, 1);
    __syncthreads();
    if (t < SW) running_sum(s.sat + t, SH, SW);
    __syncthreads();
  }
  const int p = sd.ph / 2, q = sd.pw / 2;
  for (int e = t; e < n; e += PROLOGUE_THREADS) {
    const int row = e / sd.pw, a = row - p, b = e - row * sd.pw - q;
    int a0, a1, b0, b1;
    switch (cr) {
      case 0: a0 = a; a1 = a; break;
      case 1: a0 = a; a1 = a >= 0 ? p : a - 1; break;
      case 2: a0 = -p; a1 = a <= 0 ? a : -p - 1; break;
      default: a0 = -p; a1 = a == 0 ? p : -p - 1; break;
    }
    switch (cc) {
      case 0: b0 = b; b1 = b; break;
      case 1: b0 = b; b1 = b >= 0 ? q : b - 1; break;
      case 2: b0 = -q; b1 = b <= 0 ? b : -q - 1; break;
      default: b0 = -q; b1 = b == 0 ? q : -q - 1; break;
    }
    double sum = 0.0;
    if (a1 >= a0 && b1 >= b0) {
      if (a0 == a1 && b0 == b1) {
        sum = (double)sd.psf[(a0 + p) * sd.pw + (b0 + q)];   // a single tap, exactly
      } else {
        const int r0 = a0 + p, r1 = a1 + p + 1, c0 = b0 + q, c1 = b1 + q + 1;
        sum = (s.sat[r1 * SW + c1] - s.sat[r0 * SW + c1]) - (s.sat[r1 * SW + c0] - s.sat[r0 * SW + c0]);
      }
    }
    sd.adjk[cls * n + e] = (float)(sum * inv);
  }
}

// The blocks after the points': the PSFs', then (gradient plans) the supports',
// `support` of them for each system.
static_assert(PROLOGUE_THREADS == SUPPORT_THREADS, "one launch");
template <bool ADJ>
union SystemScratch {
  PsfScratch<ADJ> psf;
  SupportScratch support;
};
template <bool ADJ>
__device__ void system_block(const SysDesc* table, const SysDesc& single, int n_sys, int block, int support,
                             SystemScratch<ADJ>& s) {
  if constexpr (ADJ) {
    const int psf_blocks = n_sys * PSF_CLASSES;
    if (block >= psf_blocks) {
      const int k = block - psf_blocks;
      const SysDesc sd = table ? table[k / support] : single;
      support_block(sd, k % support, s.support);
      return;
    }
    const SysDesc sd = table ? table[block / PSF_CLASSES] : single;
    psf_adjoint_class(sd, block % PSF_CLASSES, s.psf);
  } else {
    psf_normalise(table ? table[block] : single, s.psf.part, true);
  }
}
inline int system_blocks(bool adj, int n_sys, int support) { return n_sys * (adj ? PSF_CLASSES + support : 1); }

// Lanes of a point, and what they pass to each other.
constexpr int PROLOGUE_LANES = 32;
constexpr int PROLOGUE_POINTS = PROLOGUE_THREADS / PROLOGUE_LANES;
enum Trig { T_L, T_SHEAR, T_H, T_S, N_TRIG };   // phi_L, 2 phi_gamma, phi of the lights
enum Comp { C_H, C_S, C_SIE, N_COMP };
struct PointScratch {
  double2 cs[N_TRIG];          // (cos, sin)
  SersicBn bn[2];
  // lights: sqrt(q)/R_e, 1/(sqrt(q) R_e), q/R_e^2, 1/(q R_e^2), 1/(2n);
  // SIE: theta_E sqrt(q)/q', 1/q, 1/q^2, 1/q', 1/(2 (1 - q^2)); then sqrt(q)
  double comp[N_COMP][6];
  AmpFromMag amp[2];
  double2 maps[15];
  float jac[14];
  double folded[32];
};
template <bool ADJ>
union PrologueScratch {
  PointScratch point[PROLOGUE_POINTS];
  SystemScratch<ADJ> system;
};

template <bool ADJ>
__global__ __launch_bounds__(PROLOGUE_THREADS) void prologue_kernel(
    const float* __restrict__ theta, int n_points, PointConst* __restrict__ pcs, PointConst64* __restrict__ p64s,
    GradConst* __restrict__ gcs, const SysDesc* __restrict__ table, const int* __restrict__ point_sys,
    int* __restrict__ cusp_count, double* __restrict__ grad_corr, SysDesc single, int point_blocks,
    int n_sys, int support) {
  if (cusp_count && blockIdx.x == 0 && threadIdx.x < 2) cusp_count[threadIdx.x] = 0;
  __shared__ PrologueScratch<ADJ> lds;
  if ((int)blockIdx.x >= point_blocks) {
    system_block<ADJ>(table, single, n_sys, blockIdx.x - point_blocks, support, lds.system);
    return;
  }
  const int pl = threadIdx.x / PROLOGUE_LANES, j = threadIdx.x % PROLOGUE_LANES;
  const int p = blockIdx.x * PROLOGUE_POINTS + pl;
  if (p >= n_points) return;   // no barrier below waits for these lanes' points
  PointScratch& s = lds.point[pl];
  const SysDesc* own = table ? &table[point_sys ? point_sys[p] : 0] : &single;
  const int amp = own->amp, srcpos = own->srcpos;
  const float zp = own->zp;
  float t[NPAR];
  bool valid = true;
  for (int k = 0; k < NPAR; ++k) {
    t[k] = theta[(size_t)p * NPAR + k];
    valid = valid && isfinite(t[k]);
  }
  valid = valid && ok_q(t[1]) && ok_q(t[8]) && ok_q(t[15]) && t[6] > 0.0f && t[13] > 0.0f && ok_n(t[7]) &&
          ok_n(t[14]);
  const double te = t[0], q = t[1], phL = t[2], g = t[3];
  const double s2 = (1.0 - q) * (1.0 + q);
  const double qp = sqrt(s2);

  // lane j: angle j; light j (0 lens, 1 source) and SIE (2)
  {
    const double arg = j == T_L ? phL : j == T_SHEAR ? 2.0 * (double)t[4] : j == T_H ? (double)t[9]
                     : j == T_S ? (double)t[16] : 0.0;
    double sn, cn;
    sincos(arg, &sn, &cn);
    if (j < N_TRIG) s.cs[j] = make_double2(cn, sn);
  }
  if (j < N_COMP) {
    const bool sie = j == C_SIE;
    const double Re = j == C_H ? t[6] : t[13], n = j == C_H ? t[7] : t[14];
    const double qc = sie ? t[1] : j == C_H ? t[8] : t[15], rq = sqrt(qc);
    s.comp[j][0] = (sie ? te * rq : rq) / (sie ? qp : Re);
    s.comp[j][1] = 1.0 / (sie ? qc : rq * Re);
    s.comp[j][2] = (sie ? 1.0 : qc) / (sie ? qc * qc : Re * Re);
    s.comp[j][3] = 1.0 / (sie ? qp : qc * Re * Re);
    s.comp[j][4] = 0.5 / (sie ? s2 : n);
    s.comp[j][5] = rq;
    if (!sie) {
      const SersicBn bn = sersic_bn(valid ? n : 1.0);
      s.bn[j] = valid ? bn : SersicBn{0.0, 0.0};
      s.amp[j] = AmpFromMag{0.0, 0.0, 0.0, 0.0};
      if (valid && amp)   // amplitudes from total magnitudes (the point's system decides)
        s.amp[j] = amplitude_from_magnitude(j == C_H ? t[5] : t[12], Re, n, bn.b, bn.db, zp);
    }
  }
  const double v[7] = {t[10], t[11], t[0], t[1], t[2], t[3], t[4]};
  if (valid && srcpos && (j == 14 || (ADJ && j < 14))) lens_map_lane(v, j, s.maps);
  wave_lds_sync();
  if (ADJ) {
    if (j < 7) {
      if (valid && srcpos)
        lens_map_slope(v, j, s.maps, s.jac);
      else
        s.jac[j] = s.jac[7 + j] = 0.0f;
    }
    if (grad_corr && j < NPAR) grad_corr[(size_t)p * NPAR + j] = 0.0;
    wave_lds_sync();
  }

  if (j == 0) {   // the point's head, its float64 folded constants (to LDS) and the adjoint's constants
    PointHead c;
    const double cL = s.cs[T_L].x, sL = s.cs[T_L].y;
    const double k = s2 == 0.0 ? te : s.comp[C_SIE][0];
    const double g1 = g * s.cs[T_SHEAR].x, g2 = g * s.cs[T_SHEAR].y;
    const double bh = s.bn[C_H].b, bs = s.bn[C_S].b;
    // amplitudes: I_e given, or from total magnitudes
    const double Ih = valid && amp ? s.amp[C_H].I : (double)t[5], Is = valid && amp ? s.amp[C_S].I : (double)t[12];
    // source centre: given, or the image of an image-plane point (Sec. 5)
    const double xs = valid && srcpos ? s.maps[14].x : (double)t[10], ys = valid && srcpos ? s.maps[14].y : (double)t[11];
    c.hI = (float)Ih;
    c.sI = (float)Is;
    c.hIlo = (float)(Ih - (double)c.hI);
    c.sIlo = (float)(Is - (double)c.sI);
    // re-trace in float64 near a cuspy (n > 1) source centre (source-plane radius)
    {
      const double Re = t[13], rc = (srcpos ? CUSP_RADIUS_IMAGE_PLANE_ARCSEC : CUSP_RADIUS_ARCSEC) / Re;
      c.cusp_r2 = t[14] > 1.0f ? (float)(rc * rc) : 0.0f;
    }
    // folded constants of the forward render (float64); their dithered float32
    // roundings, one set per variant, follow below
    double tac = te, tas = 0.0, thc = 0.0, ths = 0.0;
    c.rmode = 0;
    for (int i = 0; i < 11; ++i) c.poly[i] = 0.0f;
    if (s2 != 0.0) {
      const double fh = qp <= 0.5 ? 1.0 : 0.693147180559945309417, fa = qp <= 0.5 ? 1.0 : 2.0;
      c.rmode = qp <= 0.5 ? 1 : (q >= 0.5 ? 2 : 3);
      tac = fa * k * cL;
      tas = fa * k * sL;
      thc = fh * k * cL;
      ths = fh * k * sL;
      // deflection polynomials with q' folded in: coefficient i is c_i q'^(2i+1)
      const double qp2 = qp * qp;
      double pw = qp * qp2;
      if (c.rmode == 3) {
        for (int i = 1; i <= ATAN_UNIT_POLY_DEGREE; ++i, pw *= qp2) c.poly[i] = (float)(ATAN_UNIT_POLY_D[i] * pw);
      } else {
        for (int i = 1; i <= ATAN_SMALL_POLY_DEGREE; ++i, pw *= qp2) c.poly[i] = (float)(ATAN_SMALL_POLY_D[i] * pw);
      }
      if (c.rmode == 1) {
        pw = qp * qp2;
        for (int i = 1; i <= ATANH_POLY_DEGREE; ++i, pw *= qp2)
          c.poly[ATAN_SMALL_POLY_DEGREE + i] = (float)(ATANH_POLY_D[i] * pw);
      }
    }
    double f[32];
    for (int i = 0; i < 32; ++i) f[i] = 0.0;
    f[0] = cL;
    f[1] = sL;
    f[2] = q * q;
    f[3] = s.comp[C_SIE][1];
    f[4] = qp;
    const double m11 = 1.0 - g1, m12 = -g2, m22 = 1.0 + g1;
    const double s11 = s.comp[C_S][0] * s.cs[T_S].x, s12 = s.comp[C_S][0] * s.cs[T_S].y;
    const double s21 = -s.comp[C_S][1] * s.cs[T_S].y, s22 = s.comp[C_S][1] * s.cs[T_S].x;
    const double h11 = s.comp[C_H][0] * s.cs[T_H].x, h12 = s.comp[C_H][0] * s.cs[T_H].y;
    const double h21 = -s.comp[C_H][1] * s.cs[T_H].y, h22 = s.comp[C_H][1] * s.cs[T_H].x;
    {
      // the source frame of the lens equation in one step (float64 products, one rounding each)
      f[5] = s11 * m11 + s12 * m12;            // A1
      f[6] = s21 * m11 + s22 * m12;            // A2
      f[7] = s11 * m12 + s12 * m22;            // B1
      f[8] = s21 * m12 + s22 * m22;            // B2
      f[9] = -(s11 * xs + s12 * ys);           // C1
      f[10] = -(s21 * xs + s22 * ys);          // C2
      f[11] = -(s11 * tac + s12 * tas);        // cXt
      f[12] = s11 * ths - s12 * thc;           // cXh
      f[13] = -(s21 * tac + s22 * tas);        // cYt
      f[14] = s21 * ths - s22 * thc;           // cYh
      f[23] = s11;
      f[24] = s12;
      f[25] = s21;
      f[26] = s22;
    }
    // lens light about the origin: R^2/R_e^2 = X^2 + Y^2 = (ha x + hb y) x + hc y^2
    f[15] = h11 * h11 + h21 * h21;             // ha
    f[16] = 2.0 * (h11 * h12 + h21 * h22);     // hb
    f[17] = h12 * h12 + h22 * h22;             // hc
    f[18] = s.comp[C_H][4];                    // he
    f[19] = bh * LOG2E;                        // hB
    f[20] = s.comp[C_S][4];                    // se
    f[21] = bs * LOG2E;                        // sB
    f[22] = tac;
    if (!valid) f[5] = f[6] = __builtin_nan("");
    for (int i = 0; i < 32; ++i) s.folded[i] = f[i];
    for (float& v : c.pad) v = 0.0f;
    if (!valid) c.hI = c.sI = __builtin_nanf("");
    static_cast<PointHead&>(pcs[p]) = c;
    if (p64s) {
      PointConst64 e;
      e.cL = cL;
      e.sL = sL;
      e.q2 = q * q;
      e.qp = qp;
      e.s2 = s2;
      e.closed = s2 >= SIE_SERIES_S;
      e.f = e.closed ? k : te * s.comp[C_SIE][5];
      e.pad0 = 0;
      e.m11 = m11;
      e.m12 = m12;
      e.m22 = m22;
      e.sx0 = xs;
      e.sy0 = ys;
      e.snap = srcpos ? 1e-14 * (1.0 + fabs(te) + fabs(v[0]) + fabs(v[1])) : 0.0;
      for (int i = 0; i < 3; ++i) e.pad[i] = 0.0;
      if (!valid) e.m11 = e.m12 = e.m22 = __builtin_nan("");
      p64s[p] = e;
    }

    if (ADJ && gcs) {
      GradConst gc;
      for (int i = 0; i < NPAR; ++i) gc.theta[i] = t[i];
      gc.bh = (float)bh;
      gc.bs = (float)bs;
      gc.dbh = (float)s.bn[C_H].db;
      gc.dbs = (float)s.bn[C_S].db;
      gc.Ih = c.hI;
      gc.Is = c.sI;
      gc.amp_chain[0] = (float)s.amp[C_H].dm;
      gc.amp_chain[1] = (float)s.amp[C_H].dR;
      gc.amp_chain[2] = (float)s.amp[C_H].dn;
      gc.amp_chain[3] = (float)s.amp[C_S].dm;
      gc.amp_chain[4] = (float)s.amp[C_S].dR;
      gc.amp_chain[5] = (float)s.amp[C_S].dn;
      gc.amp = amp;
      for (int i = 0; i < 14; ++i) gc.src_jac[i] = s.jac[i];
      gc.srcpos = srcpos;
      GradUniform& u = gc.u;
      const double tesq = te * s.comp[C_SIE][5], qp2 = qp * qp;
      u.cL = (float)cL;
      u.sL = (float)sL;
      // the render's SIE_TINY; more below q = 3.5e-4 (1.2e-25 at 1e-6), and q^2 itself is held up
      // where the most is too little (q < 3.5e-12)
      const double tiny = fmin(fmax((double)SIE_TINY, GRAD_PSI2_MIN / (q * q)), 1e-14);
      u.tiny = (float)tiny;
      u.q2 = (float)fmax(q * q, GRAD_PSI2_MIN / tiny);
      u.qp = (float)qp;
      u.A1 = (float)f[5];
      u.A2 = (float)f[6];
      u.B1 = (float)f[7];
      u.B2 = (float)f[8];
      u.C1 = (float)f[9];
      u.C2 = (float)f[10];
      // S R(phi_L): the SIE frame into the source frame
      u.gXx = (float)(s11 * cL + s12 * sL);
      u.gXy = (float)(s12 * cL - s11 * sL);
      u.gYx = (float)(s21 * cL + s22 * sL);
      u.gYy = (float)(s22 * cL - s21 * sL);
      u.Xa = (float)(-tesq * (s11 * cL + s12 * sL));
      u.Xb = (float)(-tesq * (s12 * cL - s11 * sL));
      u.Ya = (float)(-tesq * (s21 * cL + s22 * sL));
      u.Yb = (float)(-tesq * (s22 * cL - s21 * sL));
      u.h11 = valid ? (float)h11 : __builtin_nanf("");
      u.h12 = (float)h12;
      u.h21 = (float)h21;
      u.h22 = (float)h22;
      u.he = (float)s.comp[C_H][4];
      u.hB = (float)(bh * LOG2E);
      u.se = (float)s.comp[C_S][4];
      u.sB = (float)(bs * LOG2E);
      const float near = GRAD_ROUNDING * (float)(fabs(te) + fabs(xs) + fabs(ys)) / t[13];
      u.near2 = fmaxf(near * near, GRAD_R2_MIN);
      if (c.cusp_r2 > 0.0f) u.near2 = fminf(u.near2, 0.25f * c.cusp_r2);   // well inside the re-traced radius
      u.s11 = (float)s11;
      u.s12 = (float)s12;
      u.s21 = (float)s21;
      u.s22 = (float)s22;
      u.series = s2 < GRAD_SERIES_S;
      u.s = (float)s2;
      u.hs2 = u.series ? 0.0f : (float)(2.0 * s.comp[C_SIE][4]);
      u.iq2 = (float)s.comp[C_SIE][2];
      const bool log_form = c.rmode >= 2;
      u.kb = log_form ? (float)(0.693147180559945309417 * s.comp[C_SIE][3]) : 0.0f;
      u.kc = log_form ? (float)(-log(q) * s.comp[C_SIE][3]) : 0.0f;
      double pw = log_form ? 2.0 : 1.0;
      for (int i = 0; i <= 8; ++i, pw *= qp2)
        u.P[i] = c.rmode == 3                       ? (float)(ATAN_UNIT_POLY_D[i] * pw)
                 : i <= ATAN_SMALL_POLY_DEGREE ? (float)(ATAN_SMALL_POLY_D[i <= ATAN_SMALL_POLY_DEGREE ? i : 0] * pw)
                                               : 0.0f;
      pw = 1.0;
      for (int i = 0; i <= ATANH_POLY_DEGREE; ++i, pw *= qp2) u.Q[i] = (float)(ATANH_POLY_D[i] * pw);
      for (float& v : gc.pad) v = 0.0f;
      gcs[p] = gc;
    }
  }
  // the dithered float32 roundings of the folded constants, one set per render
  // variant: lane j of the point rounds constant j
  wave_lds_sync();
  const Dither d(s.folded[j]);
  float* rv = reinterpret_cast<float*>(pcs[p].rv) + j;
#pragma unroll
  for (int k = 0; k < RENDER_VARIANTS; ++k) rv[32 * k] = d.variant(k);
}

// General models: the PROLOGUE_LANES lanes of a point turn its parameters (layout
// of lensed_model: per SIE x_c, y_c, theta_E, q, phi; shear gamma, phi_gamma; per
// Sersic x, y, I_e, R_e, n, q, phi; sky) into ModelConst, one component per lane:
// lane k < MAX_SIE SIE k, lane MAX_SIE + k Sersic k, and one lane the shear and
// the sky. An invalid point gets sky = NaN, which makes its image NaN.
constexpr int SHEAR_LANE = MAX_SIE + MAX_SERSIC;
static_assert(SHEAR_LANE < PROLOGUE_LANES, "a lane per component");
template <bool ADJ>
__global__ __launch_bounds__(PROLOGUE_THREADS) void model_prologue_kernel(const float* __restrict__ theta, int n_points,
                                                                          int n_params, ModelSpec spec,
                                                                          ModelConst* __restrict__ out,
                                                                          const SysDesc* __restrict__ table,
                                                                          SysDesc single, int point_blocks, int n_sys,
                                                                          int support) {
  if ((int)blockIdx.x >= point_blocks) {
    __shared__ SystemScratch<ADJ> lds;
    system_block<ADJ>(table, single, n_sys, blockIdx.x - point_blocks, support, lds);
    return;
  }
  const int pl = threadIdx.x / PROLOGUE_LANES, j = threadIdx.x % PROLOGUE_LANES;
  const int p = blockIdx.x * PROLOGUE_POINTS + pl;
  if (p >= n_points) return;   // no barrier below waits for these lanes' points
  const float* t = theta + (size_t)p * n_params;
  bool valid = true;
  for (int i = j; i < n_params; i += PROLOGUE_LANES) valid = valid && isfinite(t[i]);
  ModelConst& m = out[p];
  const int o_shear = 5 * spec.n_sie, o_ser = o_shear + (spec.shear ? 2 : 0);
  const bool sie = j < spec.n_sie, sersic = j >= MAX_SIE && j < MAX_SIE + spec.n_sersic;
  const int comp = sie ? j : j - MAX_SIE;
  const float* tc = t + (sie ? 5 * comp : sersic ? o_ser + 7 * comp : o_shear);
  const bool shear = j == SHEAR_LANE && spec.shear;
  double cn, sn;
  sincos(sie ? (double)tc[4] : sersic ? (double)tc[6] : shear ? 2.0 * (double)tc[1] : 0.0, &sn, &cn);
  if (sie) {
    const double te = tc[2], q = tc[3];
    valid = valid && q > 0.0 && q <= 1.0;
    const double s2 = (1.0 - q) * (1.0 + q), qp = sqrt(fmax(s2, 0.0));
    SieConst c;
    c.x = tc[0];
    c.y = tc[1];
    c.c = cn;
    c.s = sn;
    c.q2 = q * q;
    c.qp = qp;
    c.tesq = te * sqrt(q);
    c.k = s2 == 0.0 ? te : te * sqrt(q) / qp;
    c.s2 = s2;
    c.te = te;
    c.q = q;
    c.iq2 = 1.0 / (q * q);
    c.closed = s2 >= SIE_SERIES_S;
    c.iqp = c.closed ? 1.0 / qp : 0.0;
    c.hs = c.closed ? 0.5 / s2 : 0.0;
    for (int k = 0; k < 3; ++k) c.pad[k] = 0;
    m.sie[comp] = c;
  } else if (sersic) {
    const double Re = tc[3], n = tc[4], q = tc[5];
    const bool ok = Re > 0.0 && n >= 0.2 && n <= 10.0 && q > 0.0 && q <= 1.0;
    valid = valid && ok;
    m.plane[comp] = spec.plane[comp];
    SersicConst c;
    c.x = tc[0];
    c.y = tc[1];
    c.c = cn;
    c.s = sn;
    const double ax = sqrt(q) / Re, ay = 1.0 / (sqrt(q) * Re);
    c.s11 = ax * cn;
    c.s12 = ax * sn;
    c.s21 = -ay * sn;
    c.s22 = ay * cn;
    c.e = 0.5 / n;
    c.I = tc[2];
    c.q = q;
    c.iRe = 1.0 / Re;
    c.in = 1.0 / n;
    const SersicBn bn = sersic_bn(ok ? n : 1.0);
    c.b = bn.b;
    c.B = bn.b * LOG2E;
    c.db = bn.db;
    m.ser[comp] = c;
  }
  const unsigned bad = (unsigned)(__ballot(!valid) >> (threadIdx.x & 32));
  if (j == SHEAR_LANE) {
    m.gam = shear ? (double)tc[0] : 0.0;
    m.c2g = shear ? cn : 0.0;
    m.s2g = shear ? sn : 0.0;
    m.g1 = m.gam * m.c2g;
    m.g2 = m.gam * m.s2g;
    m.sky = bad ? __builtin_nan("") : spec.sky ? (double)t[o_ser + 7 * spec.n_sersic] : 0.0;
    m.n_sie = spec.n_sie;
    m.n_sersic = spec.n_sersic;
  }
}

template <bool ADJ>
hipError_t model_prologue(const float* theta, int n_points, int n_params, const ModelSpec& spec, ModelConst* out,
                          const SysDesc& single, const SysDesc* table, int n_sys, int support, hipStream_t stream) {
  const int point_blocks = (n_points + PROLOGUE_POINTS - 1) / PROLOGUE_POINTS;
  const int blocks = point_blocks + system_blocks(ADJ, n_sys, support);
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(model_prologue_kernel<ADJ>, dim3(blocks), dim3(PROLOGUE_THREADS), 0, stream, theta, n_points,
                     n_params, spec, out, table, single, point_blocks, n_sys, support);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_model_prologue(const float* theta, int n_points, int n_params, const ModelSpec& spec,
                                 ModelConst* out, const SysDesc& single, const SysDesc* table, int n_sys,
                                 hipStream_t stream, bool adjoint_tables, int support) {
  return adjoint_tables
             ? model_prologue<true>(theta, n_points, n_params, spec, out, single, table, n_sys, support, stream)
             : model_prologue<false>(theta, n_points, n_params, spec, out, single, table, n_sys, support, stream);
}

hipError_t launch_prologue(const float* theta, int n_points, PointConst* pcs, PointConst64* p64s, GradConst* gcs,
                           const SysDesc& single, SysDesc* table, int n_sys, int* cusp_count, hipStream_t stream,
                           double* grad_corr, const int* point_sys, bool adjoint_tables, int support) {
  const int point_blocks = (n_points + PROLOGUE_POINTS - 1) / PROLOGUE_POINTS;
  const int blocks = point_blocks + system_blocks(adjoint_tables, n_sys, support);
  if (blocks == 0) return hipSuccess;
  if (adjoint_tables)
    hipLaunchKernelGGL(prologue_kernel<true>, dim3(blocks), dim3(PROLOGUE_THREADS), 0, stream, theta, n_points, pcs,
                       p64s, gcs, table, point_sys, cusp_count, grad_corr, single, point_blocks, n_sys, support);
  else
    hipLaunchKernelGGL(prologue_kernel<false>, dim3(blocks), dim3(PROLOGUE_THREADS), 0, stream, theta, n_points, pcs,
                       p64s, gcs, table, point_sys, cusp_count, grad_corr, single, point_blocks, n_sys, support);
  return hipGetLastError();
}

}  // namespace lensed
