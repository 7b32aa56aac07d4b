// model.h -- shape and per-point constants of general models (several lenses
// and light components, a flat sky, free centres), evaluated in float64.
#pragma once

namespace lensed {

// General models (several lenses and light components, a flat sky, free
// centres): the model's shape (a copy of lensed_model) and per-point constants
// in float64, derived by the model prologue.
constexpr int MAX_SIE = 8, MAX_SERSIC = 8, MAX_PLANES = 8;
struct ModelSpec {
  int n_sie, shear, n_sersic, sky;
  int plane[MAX_SERSIC];          // per Sersic: its plane, 0..n_planes (n_planes: the source)
  int n_planes;                   // lens planes, 1..8
  int sie_plane[MAX_SIE];         // per SIE: its lens plane (0 with one plane)
  double beta[MAX_PLANES][MAX_PLANES];  // distance ratios beta_ij, i < j < n_planes (0 with one plane)
};
struct SieConst {
  double x, y, c, s;           // centre, cos and sin of the position angle
  double q2, qp, k;            // q^2, q' = sqrt(1 - q^2), theta_E sqrt(q)/q'
  double tesq, s2, te, q, iq2; // theta_E sqrt(q), 1 - q^2, theta_E, q, 1/q^2
  double iqp, hs;              // 1/q', 1/(2 (1 - q^2)) (0 unless closed)
  int closed;                  // 1: atan and atanh in closed form; 0: series in 1 - q^2 (nearly round lenses)
  int pad[3];
};
struct SersicConst {
  double x, y;                 // centre
  double s11, s12, s21, s22;   // (X, Y) = S (offset from the centre), (R/R_e)^2 = X^2 + Y^2
  double e, B, I;              // 1/(2n), b_n log2(e), I_e
  double b, db, q, iRe, c, s, in;   // b_n, db_n/dn (0 unless asked for), q, 1/R_e, cos, sin, 1/n
};
struct ModelConst {
  SieConst sie[MAX_SIE];
  SersicConst ser[MAX_SERSIC];
  double g1, g2;               // external shear (zero without one)
  double gam, c2g, s2g;        // gamma, cos 2 phi_gamma, sin 2 phi_gamma
  double sky;                  // flat sky surface brightness (NaN marks an invalid point)
  int n_sie, n_sersic;
  int plane[MAX_SERSIC];       // the Sersic's plane: 0 light at x, n_planes light at the source
};

}  // namespace lensed
