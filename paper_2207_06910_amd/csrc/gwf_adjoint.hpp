// gwf_adjoint.hpp -- per-point mathematics of the adjoint of the Fisher/SNR
// map with respect to the detector parameters (latitude, longitude, arm angle
// gamma and ln S0 of each site).
//
// For a figure of merit J(Gamma_e, SNR_e) the reverse-mode sensitivity
// along a detector parameter xi is
//   dJ/dxi = sum_e [ sum_ij Gbar_e,ij dGamma_e,ij/dxi + snrbar_e dSNR_e/dxi ],
// Gbar = dJ/dGamma (Gamma^-1 for J = ln det Gamma), snrbar = dJ/dSNR.  With
// Gamma_ij = sum_{k,d} w Re(D_i D_j^*) (sec. 3.2, D the noise-weighted
// derivative vectors of the phase-free form) and a symmetric Gbar, each
// grid point and interferometer contributes w (Dr^T Gbar Dr + Di^T Gbar Di)
// to sum_ij Gbar_ij Gamma_ij.  The backward pass recomputes that quadratic
// form at every point and takes its derivatives; no Jacobian is stored.
//
// Structure used (exact algebra).  An interferometer enters D only through
// its six pattern values y = (F+, Fx, dF+/dH, dFx/dH, dF+/dth, dFx/dth)
// (H the hour angle).  With Q = (c+ y0, cx y1), c+ = (1 + cos^2 i)/2,
// cx = cos i, and Z, Y as in the forward pass (gwf_model.hpp: the hour-angle
// and theta derivatives of Q with the delay's phase terms i u Q, i w Q),
//   Re D = v0 y0 + (2 c+ e6 - cx pi) y1 + gamma Re Z + e3 Re Y,
//   Im D = (c+ pi - 2 cx e6) y0 + w1 y1 + gamma Im Z + e3 Im Y,
// where e3, e6 are the unit vectors of theta and psi, v0 and w1 fixed
// per-event vectors (amplitude, distance and inclination rows), pi the PN
// phase derivatives (with 2 pi f for tc and the phase-only coefficients c_i)
// and gamma the hour-angle direction of the phase derivatives (Mc, eta
// through the sidereal angle at t(f); phi; tc).  None of these vectors knows
// the site, so the quadratic form's 14 coefficients are formed once per grid
// point from Gbar inner products <a, b> = a^T Gbar b (AdjPoint), and an
// interferometer costs 28 multiply-adds for the form's gradient h in
// (y0, y1, Z, Y).
//
// Derivatives: J_point depends on the detector parameters through y (the
// patterns: latitude and gamma move their coefficients, longitude the hour
// angle H), through the arrival-time derivatives dDelta/dH and dDelta/dth
// (latitude and longitude) and, for ln S0, through the weight (dw = -w).
// The patterns are trigonometric polynomials in H (SiteC::jk) whose five
// basis functions no direction changes: along every direction dy follows
// from that direction's coefficients and the same basis.  So the gradient is
// taken in the coefficients (4 polynomials x 5, and 2 x 5 for SNR^2), summed
// over the points a lane holds, and contracted once with each direction's
// coefficients (latitude and gamma: AdjSiteC; longitude: jk's own, turned),
// in place of evaluating each direction's polynomials at every point.
#pragma once

#include "gwf_model.hpp"

namespace gwf {

constexpr int kMaxNpi = 6;

// ----------------------------------------------------- site constants
// Pattern maps of one interferometer (as pattern_map) and their derivatives
// along its bisector angle gamma.
__host__ __device__ inline void pattern_map_g(double gamma, double zeta, double c2p, double s2p, double al[4],
                                              double be[4], double alg[4], double beg[4]) {
  pattern_map(gamma, zeta, c2p, s2p, al, be);
  const double sz = sin(zeta), s2g = sin(2.0 * gamma), c2g = cos(2.0 * gamma);
  // d/dgamma: s2g -> 2 c2g, c2g -> -2 s2g
  alg[0] = 2.0 * sz * c2g * c2p; alg[1] = 2.0 * sz * s2g * c2p; alg[2] = 2.0 * sz * c2g * s2p;
  alg[3] = 2.0 * sz * s2g * s2p;
  beg[0] = -2.0 * sz * c2g * s2p; beg[1] = -2.0 * sz * s2g * s2p; beg[2] = 2.0 * sz * c2g * c2p;
  beg[3] = 2.0 * sz * s2g * c2p;
}

// Adds k (a' b + a b') to out: the derivative of trig_mul_add(a, b, k) along
// a direction in which a and b move by a' and b'.
__host__ __device__ inline void trig_mul_add_d(const TrigLin& a, const TrigLin& ad, const TrigLin& b,
                                               const TrigLin& bd, double k, double out[5]) {
  trig_mul_add(ad, b, k, out);
  trig_mul_add(a, bd, k, out);
}

// The latitude derivatives of pattern_trig's polynomials: sin lat -> cos lat,
// cos lat -> -sin lat, which moves only NX, NY and the theta derivative of NY.
__host__ __device__ inline void pattern_trig_lat(double ct, double st, double sl, double cl, double pc[4][5],
                                                 double ptc[4][5]) {
  const TrigLin EX{0.0, 1.0, 0.0}, EY{0.0, 0.0, -ct}, NX{0.0, 0.0, -sl}, NY{-cl * st, -sl * ct, 0.0};
  const TrigLin EYt{0.0, 0.0, st}, NYt{-cl * ct, sl * st, 0.0};
  const TrigLin Z{0.0, 0.0, 0.0};
  const TrigLin NXl{0.0, 0.0, -cl}, NYl{sl * st, -cl * ct, 0.0}, NYtl{sl * ct, cl * st, 0.0};
  for (int i = 0; i < 4; ++i)
    for (int m = 0; m < 5; ++m) pc[i][m] = ptc[i][m] = 0.0;
  // P0 = (EX EX - NX NX - EY EY + NY NY)/2
  trig_mul_add_d(NX, NXl, NX, NXl, -0.5, pc[0]);
  trig_mul_add_d(NY, NYl, NY, NYl, 0.5, pc[0]);
  // P1 = EX NX - EY NY
  trig_mul_add_d(EX, Z, NX, NXl, 1.0, pc[1]);
  trig_mul_add_d(EY, Z, NY, NYl, -1.0, pc[1]);
  // P2 = EX EY - NX NY
  trig_mul_add_d(NX, NXl, NY, NYl, -1.0, pc[2]);
  // P3 = EX NY + NX EY
  trig_mul_add_d(EX, Z, NY, NYl, 1.0, pc[3]);
  trig_mul_add_d(NX, NXl, EY, Z, 1.0, pc[3]);
  // theta derivatives: Pt0 = -EY EYt + NY NYt, Pt1 = -(EYt NY + EY NYt),
  // Pt2 = EX EYt - NX NYt, Pt3 = EX NYt + NX EYt
  trig_mul_add_d(NY, NYl, NYt, NYtl, 1.0, ptc[0]);
  trig_mul_add_d(EYt, Z, NY, NYl, -1.0, ptc[1]);
  trig_mul_add_d(EY, Z, NYt, NYtl, -1.0, ptc[1]);
  trig_mul_add_d(NX, NXl, NYt, NYtl, -1.0, ptc[2]);
  trig_mul_add_d(EX, Z, NYt, NYtl, 1.0, ptc[3]);
  trig_mul_add_d(NX, NXl, EYt, Z, 1.0, ptc[3]);
}

// Per (event, site) constants of the adjoint beside SiteC: the latitude and
// gamma derivatives of the effective interferometers' pattern polynomials
// (SiteC::jk, sqrt(weff) included) and the latitude derivatives of the
// arrival-time coefficients.
struct AdjSiteC {
  double jl[2][4][5];                   // d jk / d latitude
  double jg[2][4][5];                   // d jk / d gamma
  double k1l, k1tl, k0tl;               // d(k1, k1t, k0t)/d latitude
  double pad;
};

// sc: the site's SiteC (site_setup) with the same arm_on.
__host__ __device__ inline void adj_site_setup(const double* p, const SiteDesc& sd, const SiteC& sc,
                                               AdjSiteC& as, uint32_t arm_on = 7u) {
  const double th = p[3], psi = p[6];
  const double c2p = cos(2.0 * psi), s2p = sin(2.0 * psi);
  const double ct = cos(th), st = sin(th), sl = sin(sd.lat), cl = cos(sd.lat);
  as.k1l = kREarthS * sl * st;
  as.k1tl = kREarthS * sl * ct;
  as.k0tl = kREarthS * cl * st;
  as.pad = 0.0;
  // gamma derivatives of the effective interferometers' pattern maps
  double alg[2][4] = {}, beg[2][4] = {};
  if (sd.shape == 1) {
    double ag[3][4], bg[3][4];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double al[4], be[4];
      pattern_map_g(sd.gamma + kPi / 6.0 + kTwoPi * k / 3.0, kPi / 3.0, c2p, s2p, al, be, ag[k], bg[k]);
    }
    if ((arm_on & 7u) == 7u) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        alg[0][j] = ag[0][j] + ag[1][j]; beg[0][j] = bg[0][j] + bg[1][j];
        alg[1][j] = ag[0][j] - ag[1][j]; beg[1][j] = bg[0][j] - bg[1][j];
      }
    } else {                                 // the active arms in arm order
      int m = 0;
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (arm_on >> k & 1u) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (m == 0) { alg[0][j] = ag[k][j]; beg[0][j] = bg[k][j]; }
            else { alg[1][j] = ag[k][j]; beg[1][j] = bg[k][j]; }
          }
          ++m;
        }
    }
  } else {
    double al[4], be[4];
    pattern_map_g(sd.gamma, sd.zeta, c2p, s2p, al, be, alg[0], beg[0]);
  }
  // coefficient q of effective interferometer j: sqrt(weff) (a . pm, b . pm,
  // a . ptm, b . ptm) for the maps (a, b) and polynomials (pm, ptm) given
  auto contract = [&](int j, const double (&a)[4], const double (&b)[4], const double (&pm)[4][5],
                      const double (&ptm)[4][5], double (&out)[4][5]) {
    const double w = sqrt(sc.weff[j]);
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        t[0] = fma(a[i], pm[i][m], t[0]);
        t[1] = fma(b[i], pm[i][m], t[1]);
        t[2] = fma(a[i], ptm[i][m], t[2]);
        t[3] = fma(b[i], ptm[i][m], t[3]);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) out[q][m] = w * t[q];
    }
  };
  {
    double pcl[4][5], ptcl[4][5];
    pattern_trig_lat(ct, st, sl, cl, pcl, ptcl);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      double a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { a[i] = sc.alpha[j][i]; b[i] = sc.beta[j][i]; }
      contract(j, a, b, pcl, ptcl, as.jl[j]);
    }
  }
  {
    double pc[4][5], ptc[4][5];
    pattern_trig(ct, st, sl, cl, pc, ptc);
#pragma unroll
    for (int j = 0; j < 2; ++j) contract(j, alg[j], beg[j], pc, ptc, as.jg[j]);
  }
}

// ----------------------------------------------------- event constants
// The fixed vectors (length P): e3, e6, v0 = (dlnA c+, 0, -c+/dL, 0, 0,
// dc+/di, 0, 0, 0...), w1 = (dlnA cx, 0, -cx/dL, 0, 0, dcx/di, 0, 0, 0...),
// and gamma0 = -e4 + Omega e7 (the part of gamma that does not depend on
// the point).
enum { kXe3 = 0, kXe6, kXv0, kXw1, kXg0, kNX };

__host__ __device__ constexpr int xx_index(int a, int b) {
  return a <= b ? a * kNX - (a * (a - 1)) / 2 + (b - a) : b * kNX - (b * (b - 1)) / 2 + (a - b);
}
__host__ __device__ constexpr int cc_index(int i, int j) {
  return i <= j ? i * kMaxNpi - (i * (i - 1)) / 2 + (j - i) : j * kMaxNpi - (j * (j - 1)) / 2 + (i - j);
}

// Contractions of an event's (symmetrised, masked) Gbar: rows b = Mc, eta,
// tc (the point-dependent basis rows of pi and gamma), the phase-only rows
// 8 + i and the fixed vectors.
struct AdjEventC {
  double g3[6];                              // <e_a, e_b>, (a, b) = 00, 01, 07, 11, 17, 77
  double bx[3][kNX];                         // <e_b, X>, b = Mc, eta, tc
  double cx[kNX][kMaxNpi];                   // <e_{8+i}, X>
  double cb[3][kMaxNpi];                     // <e_b, e_{8+i}>
  double cq[kMaxNpi * (kMaxNpi + 1) / 2];    // <e_{8+i}, e_{8+j}> for i = j, twice that for i < j
  double xx[kNX * (kNX + 1) / 2];            // <X, Y>
  double cpl, ccr;                           // c+, cx
  double cpp, cxx, cc4;                      // c+^2, cx^2, 4 c+ cx
  // constant parts of the point's coefficients (see AdjPoint)
  double h00c, h11c;                         // <v0,v0> + 4 cx^2 <e6,e6>, <w1,w1> + 4 c+^2 <e6,e6>
  double h01c;                               // 2 c+ <e6,v0> - 2 cx <e6,w1>
  double cp2x36, cx2x36;                     // 2 c+ <e3,e6>, 2 cx <e3,e6>
  int32_t ok, pad;
};

// gb(i, j): Gbar_ij, symmetric, zero outside the event's rows; GX: scratch
// of (8 + NPI) kNX values.  The work is shared by `lanes` callers (this one:
// `lane`), which sync() brings together; the fixed vectors have at most three
// nonzero entries each, so Gbar X takes those columns of Gbar only.
template <int NPI, class GB, class SYNC>
__host__ __device__ inline void adj_event_setup(const EventC& ec, const GB& gb, AdjEventC& ae, double* GX, int lane,
                                                int lanes, SYNC sync) {
  const double v0a = ec.dlnA_dMc * ec.cplus, v0b = -ec.cplus * ec.inv_dL, v0c = ec.dcplus;
  const double w1a = ec.dlnA_dMc * ec.ccross, w1b = -ec.ccross * ec.inv_dL, w1c = ec.dcross;
  // X_x^T v for a vector v on the binary's eight rows (Mc, eta, dL, theta,
  // phi, iota, psi, tc), its entries st apart
  auto xdot = [&](int x, const double* v, int st) -> double {
    switch (x) {
      case kXe3: return v[3 * st];
      case kXe6: return v[6 * st];
      case kXv0: return fma(v0c, v[5 * st], fma(v0b, v[2 * st], v0a * v[0]));
      case kXw1: return fma(w1c, v[5 * st], fma(w1b, v[2 * st], w1a * v[0]));
      default: return fma(kOmegaE, v[7 * st], -v[4 * st]);
    }
  };
  for (int r = lane; r < 8 + NPI; r += lanes) {      // (Gbar X)_r
    double row[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) row[c] = gb(r, c);
#pragma unroll
    for (int x = 0; x < kNX; ++x) GX[r * kNX + x] = xdot(x, row, 1);
  }
  sync();
  constexpr int rows[3] = {0, 1, 7};
  for (int t = lane; t < 8; t += lanes) {
    auto XX = [&](int x, int y) { return xdot(y, GX + x, kNX); };     // <X, Y>
    const double cp = ec.cplus, cx = ec.ccross;
    switch (t) {
      case 0:
        ae.g3[0] = gb(0, 0); ae.g3[1] = gb(0, 1); ae.g3[2] = gb(0, 7);
        ae.g3[3] = gb(1, 1); ae.g3[4] = gb(1, 7); ae.g3[5] = gb(7, 7);
        break;
      case 1:
        for (int b = 0; b < 3; ++b)
          for (int x = 0; x < kNX; ++x) ae.bx[b][x] = GX[rows[b] * kNX + x];
        break;
      case 2:
        ae.cpl = cp;
        ae.ccr = cx;
        ae.cpp = cp * cp;
        ae.cxx = cx * cx;
        ae.cc4 = 4.0 * cp * cx;
        ae.pad = 0;
        break;
      case 3: ae.h00c = XX(kXv0, kXv0) + 4.0 * cx * cx * XX(kXe6, kXe6); break;
      case 4: ae.h11c = XX(kXw1, kXw1) + 4.0 * cp * cp * XX(kXe6, kXe6); break;
      case 5: ae.h01c = 2.0 * cp * XX(kXe6, kXv0) - 2.0 * cx * XX(kXe6, kXw1); break;
      case 6: ae.cp2x36 = 2.0 * cp * XX(kXe3, kXe6); break;
      default: ae.cx2x36 = 2.0 * cx * XX(kXe3, kXe6);
    }
  }
  for (int t = lane; t < kNX * kMaxNpi; t += lanes) {
    const int x = t / kMaxNpi, i = t - x * kMaxNpi;
    ae.cx[x][i] = i < NPI ? GX[(8 + i) * kNX + x] : 0.0;
  }
  for (int t = lane; t < 3 * kMaxNpi; t += lanes) {
    const int b = t / kMaxNpi, i = t - b * kMaxNpi;
    ae.cb[b][i] = i < NPI ? gb(b == 2 ? 7 : b, 8 + i) : 0.0;
  }
  for (int t = lane; t < kMaxNpi * kMaxNpi; t += lanes) {
    const int i = t / kMaxNpi, j = t - i * kMaxNpi;
    if (i <= j) ae.cq[cc_index(i, j)] = (i < NPI && j < NPI) ? (i == j ? 1.0 : 2.0) * gb(8 + i, 8 + j) : 0.0;
  }
  for (int t = lane; t < kNX * kNX; t += lanes) {
    const int x = t / kNX, y = t - x * kNX;
    if (x <= y) ae.xx[xx_index(x, y)] = xdot(y, GX + x, kNX);
  }
}

// By one caller.
template <int NPI, class GB>
__host__ __device__ inline void adj_event_setup(const EventC& ec, const GB& gb, AdjEventC& ae) {
  double GX[(8 + NPI) * kNX];
  adj_event_setup<NPI>(ec, gb, ae, GX, 0, 1, [] {});
}

// Accumulator slots of one site: sum Gbar dGamma along (lat, lon, gamma,
// ln S0), dSNR^2 along (lat, lon, gamma), and SNR^2 itself (its ln S0
// derivative is minus that).
enum { kAdjT = 0, kAdjS = 4, kAdjW = 7, kAdjN = 8 };

// ------------------------------------------------------ one grid point
// The point quantities shared by all sites: the coefficients of the quadratic
// form in (y0, y1, Z, Y), with r = 2 c+ e6 - cx pi and m = c+ pi - 2 cx e6
// (<e3,v0>, <e3,w1> and <e3,e3> are the event's).
struct AdjPoint {
  Point q;
  double k00, k11, k01;        // <v0,v0> + <m,m>, <w1,w1> + <r,r>, <v0,r> + <m,w1>
  double gv0, gr, gm, gw1;     // <gamma, v0>, <gamma, r>, <gamma, m>, <gamma, w1>
  double er, em;               // <e3, r>, <e3, m>
  double gg, g3;               // <gamma, gamma>, <gamma, e3>
};

// Marks memory as changed: what is read behind it is read there (scalar loads
// of an event's constants), not held in registers from before.
__host__ __device__ inline void constants_again() {
#if defined(__HIP_DEVICE_COMPILE__)
  __asm__ volatile("" ::: "memory");
#endif
}

// The NQ points k of an event; vrec: v, 1/v and v^-12.42 at each (GridWalk), or
// NULL.  Each group of constants is read once for all points.
template <int NPI, bool ROT, int NQ>
__host__ __device__ inline void adjoint_point_setup(const EventC& ec, const AdjEventC& ae, const int32_t (&k)[NQ],
                                                    AdjPoint (&ap)[NQ], const double (*vrec)[3] = nullptr) {
  double c[NQ][NPI];
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    constants_again();
    point_setup<false, PhaseOnly<NPI>::ecc>(ec, k[n], true, ROT, ap[n].q, kPsdF64, vrec ? vrec[n] : nullptr);
    phase_only_coefficients<NPI>(ec, ap[n].q, c[n]);
  }
  constants_again();
  // u_b = <e_b, C>, C = sum c_i e_{8+i}; pp = <C, C>
  //   = sum_i c_i (Gbar_ii c_i + 2 sum_{j > i} Gbar_ij c_j)
  double u[NQ][3], pp[NQ];
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      double t = 0.0;
#pragma unroll
      for (int i = 0; i < NPI; ++i) t = fma(ae.cb[b][i], c[n][i], t);
      u[n][b] = t;
    }
    pp[n] = 0.0;
#pragma unroll
    for (int i = 0; i < NPI; ++i) {
      double t = 0.0;
#pragma unroll
      for (int j = i; j < NPI; ++j) t = fma(ae.cq[cc_index(i, j)], c[n][j], t);
      pp[n] = fma(c[n][i], t, pp[n]);
    }
  }
  constants_again();
  // pi = pMc e0 + pEta e1 + tf e7 + C; pe: <pi, e0> and <pi, e1>
  double pX[NQ][kNX], pe[NQ][2];
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    const double a = ap[n].q.pMc, b = ap[n].q.pEta, tf = ap[n].q.tf;
    pe[n][0] = fma(a, ae.g3[0], fma(b, ae.g3[1], fma(tf, ae.g3[2], u[n][0])));
    pe[n][1] = fma(a, ae.g3[1], fma(b, ae.g3[3], fma(tf, ae.g3[4], u[n][1])));
    const double pe7 = fma(a, ae.g3[2], fma(b, ae.g3[4], fma(tf, ae.g3[5], u[n][2])));
    pp[n] = fma(a, pe[n][0], fma(b, pe[n][1], fma(tf, pe7, fma(a, u[n][0], fma(b, u[n][1], fma(tf, u[n][2], pp[n]))))));
#pragma unroll
    for (int x = 0; x < kNX; ++x) pX[n][x] = fma(a, ae.bx[0][x], fma(b, ae.bx[1][x], tf * ae.bx[2][x]));
  }
  constants_again();
#pragma unroll
  for (int n = 0; n < NQ; ++n)
#pragma unroll
    for (int x = 0; x < kNX; ++x)
#pragma unroll
      for (int i = 0; i < NPI; ++i) pX[n][x] = fma(c[n][i], ae.cx[x][i], pX[n][x]);
  constants_again();
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    AdjPoint& p = ap[n];
    // gamma = gMc e0 + gEta e1 + gamma0 (gMc = gEta = 0 without rotation)
    const double gm = p.q.gMc, ge = p.q.gEta;
    double gX[4];                                // <gamma, X>
#pragma unroll
    for (int x = 0; x < 4; ++x) gX[x] = fma(gm, ae.bx[0][x], fma(ge, ae.bx[1][x], ae.xx[xx_index(kXg0, x)]));
    const double pg = fma(gm, pe[n][0], fma(ge, pe[n][1], pX[n][kXg0]));
    const double ge0 = fma(gm, ae.g3[0], fma(ge, ae.g3[1], 2.0 * ae.bx[0][kXg0]));
    const double ge1 = fma(gm, ae.g3[1], fma(ge, ae.g3[3], 2.0 * ae.bx[1][kXg0]));
    const double cp = ae.cpl, cx = ae.ccr;
    const double c6 = -ae.cc4 * pX[n][kXe6];
    p.k00 = fma(ae.cpp, pp[n], ae.h00c + c6);
    p.k11 = fma(ae.cxx, pp[n], ae.h11c + c6);
    p.k01 = fma(-cx, pX[n][kXv0], fma(cp, pX[n][kXw1], ae.h01c));
    p.gv0 = gX[kXv0];
    p.gw1 = gX[kXw1];
    p.gr = fma(-cx, pg, 2.0 * cp * gX[kXe6]);
    p.gm = fma(cp, pg, -2.0 * cx * gX[kXe6]);
    p.er = fma(-cx, pX[n][kXe3], ae.cp2x36);
    p.em = fma(cp, pX[n][kXe3], -ae.cx2x36);
    p.gg = fma(gm, ge0, fma(ge, ge1, ae.xx[xx_index(kXg0, kXg0)]));
    p.g3 = gX[kXe3];
  }
}

// The sites' contributions at NQ points, out(s, t[kAdjN]) for each.  The basis
// carries the root weight (trig_basis), as in the forward pass.
template <int NQ, bool TAB, bool AHEAD, class OUT>
__host__ __device__ inline void adjoint_sites(const AdjEventC& ae, const SiteC* scs, const AdjSiteC* ass, int n_site,
                                              const AdjPoint (&ap)[NQ], OUT out) {
  SiteHead hd = site_head(scs[0]);
  for (int site = 0; site < n_site; ++site) {
    const SiteC& sc = scs[site];
    const AdjSiteC& as = ass[site];
    const double cp = ae.cpl, cx = ae.ccr;
    const double ev0 = ae.xx[xx_index(kXe3, kXv0)], ew1 = ae.xx[xx_index(kXe3, kXw1)];
    const double ee = ae.xx[xx_index(kXe3, kXe3)];
    const int n_eff = sc.n_eff;
    Poly4 c = poly4(sc.jk[0]);
    if (AHEAD) loads_ahead();
    SiteTrigR sp[NQ];
    double tc[NQ], ts[NQ], wu[NQ], ww[NQ];   // 2 pi f (cos H, sin H); adjoints of u and w (halved)
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const Point& q = ap[i].q;
      const double cH = q.cth * hd.cdl - q.sth * hd.sdl;
      const double sH = q.sth * hd.cdl + q.cth * hd.sdl;
      trig_basis(cH, sH, site_root<false, TAB>(sc, hd, q), sp[i]);
      tc[i] = q.tf * cH;
      ts[i] = q.tf * sH;
      sp[i].u = -hd.k1 * ts[i];
      sp[i].w = fma(hd.k1t, tc[i], q.tf * hd.k0t);
      wu[i] = ww[i] = 0.0;
    }
    double t[kAdjN] = {};
    for (int j = 0; j < n_eff; ++j) {      // none where the duty factor turns the whole site off
      if (j > 0) c = poly4(sc.jk[j]);
      Poly4 d = poly4(as.jl[j]);
      if (AHEAD) loads_ahead();
      // half the gradients of J in the coefficients of the four polynomials,
      // and of SNR^2/2 in those of the first two (over c+ and cx)
      double m[4][5] = {}, s[2][5] = {};
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const AdjPoint& a = ap[i];
        const SiteTrigR& b = sp[i];
        const double y0 = trig_val_r(c.c[0], b), y1 = trig_val_r(c.c[1], b);
        const double y2 = trig_dH_r(c.c[0], b), y3 = trig_dH_r(c.c[1], b);
        const double Qr = cp * y0, Qi = cx * y1;
        const double Zr = fma(cp, y2, -b.u * Qi);
        const double Zi = fma(cx, y3, b.u * Qr);
        const double Yr = fma(cp, trig_val_r(c.c[2], b), -b.w * Qi);
        const double Yi = fma(cx, trig_val_r(c.c[3], b), b.w * Qr);
        const double h0 = fma(a.k00, y0, fma(a.k01, y1, fma(a.gv0, Zr, fma(a.gm, Zi, fma(ev0, Yr, a.em * Yi)))));
        const double h1 = fma(a.k01, y0, fma(a.k11, y1, fma(a.gr, Zr, fma(a.gw1, Zi, fma(a.er, Yr, ew1 * Yi)))));
        const double hzr = fma(a.gv0, y0, fma(a.gr, y1, fma(a.gg, Zr, a.g3 * Yr)));
        const double hzi = fma(a.gm, y0, fma(a.gw1, y1, fma(a.gg, Zi, a.g3 * Yi)));
        const double hyr = fma(ev0, y0, fma(a.er, y1, fma(a.g3, Zr, ee * Yr)));
        const double hyi = fma(a.em, y0, fma(ew1, y1, fma(a.g3, Zi, ee * Yi)));
        t[kAdjT + 3] -= fma(y0, h0, fma(y1, h1, fma(Zr, hzr, fma(Zi, hzi, fma(Yr, hyr, Yi * hyi)))));
        t[kAdjW] = fma(Qr, Qr, fma(Qi, Qi, t[kAdjW]));
        wu[i] = fma(Qr, hzi, fma(-Qi, hzr, wu[i]));
        ww[i] = fma(Qr, hyi, fma(-Qi, hyr, ww[i]));
        const double g0 = fma(cp, fma(b.u, hzi, b.w * hyi), h0);
        const double g1 = fma(-cx, fma(b.u, hzr, b.w * hyr), h1);
        const double g2 = cp * hzr, g3 = cx * hzi, g4 = cp * hyr, g5 = cx * hyi;
        if (NQ == 1) {
          // one point: each direction's polynomials themselves
          auto along = [&](double l0, double l1, double l2, double l3, double l4, double l5, double& T, double& S) {
            T = fma(g0, l0, fma(g1, l1, fma(g2, l2, fma(g3, l3, fma(g4, l4, fma(g5, l5, T))))));
            S = fma(cp * Qr, l0, fma(cx * Qi, l1, S));
          };
          // the second H derivative: -(c1 cos H + c2 sin H + 4 (c3 cos 2H + c4 sin H cos H))
          auto dHH = [&](const double* C) {
            return -fma(4.0, fma(C[4], b.rsc, C[3] * b.rc2), fma(C[2], b.rs, C[1] * b.rc));
          };
          along(y2, y3, dHH(c.c[0]), dHH(c.c[1]), trig_dH_r(c.c[2], b), trig_dH_r(c.c[3], b), t[kAdjT + 1],
                t[kAdjS + 1]);
          along(trig_val_r(d.c[0], b), trig_val_r(d.c[1], b), trig_dH_r(d.c[0], b), trig_dH_r(d.c[1], b),
                trig_val_r(d.c[2], b), trig_val_r(d.c[3], b), t[kAdjT + 0], t[kAdjS + 0]);
          const Poly4 dg = poly4(as.jg[j]);
          along(trig_val_r(dg.c[0], b), trig_val_r(dg.c[1], b), trig_dH_r(dg.c[0], b), trig_dH_r(dg.c[1], b),
                trig_val_r(dg.c[2], b), trig_val_r(dg.c[3], b), t[kAdjT + 2], t[kAdjS + 2]);
          continue;
        }
        // two points or more: the coefficients' gradients, summed over them
        const double bv[5] = {b.r, b.rc, b.rs, b.rc2, b.rsc};
        const double bd[5] = {0.0, -b.rs, b.rc, b.rm4, b.rc2};
        m[0][0] = fma(g0, bv[0], m[0][0]);
        m[1][0] = fma(g1, bv[0], m[1][0]);
#pragma unroll
        for (int k = 1; k < 5; ++k) {
          m[0][k] = fma(g0, bv[k], fma(g2, bd[k], m[0][k]));
          m[1][k] = fma(g1, bv[k], fma(g3, bd[k], m[1][k]));
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) {
          m[2][k] = fma(g4, bv[k], m[2][k]);
          m[3][k] = fma(g5, bv[k], m[3][k]);
          s[0][k] = fma(Qr, bv[k], s[0][k]);
          s[1][k] = fma(Qi, bv[k], s[1][k]);
        }
      }
      if (NQ == 1) continue;
      // longitude: d/dH of c0 + c1 cos H + c2 sin H + c3 cos 2H + c4 sin H cos H
      // has the coefficients (0, c2, -c1, c4, -4 c3)
      double S1[2];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        double& T = t[kAdjT + 1];
        const double* C = c.c[q];
        T = fma(C[2], m[q][1], fma(-C[1], m[q][2], fma(C[4], m[q][3], fma(C[3], -4.0 * m[q][4], T))));
        if (q < 2) S1[q] = fma(C[2], s[q][1], fma(-C[1], s[q][2], fma(C[4], s[q][3], C[3] * (-4.0 * s[q][4]))));
      }
      t[kAdjS + 1] = fma(cp, S1[0], fma(cx, S1[1], t[kAdjS + 1]));
      // latitude and gamma: the directions' coefficients
      auto along = [&](const Poly4& d, double& T, double& S) {
        double x = 0.0, y = 0.0;
#pragma unroll
        for (int k = 0; k < 5; ++k) {
#pragma unroll
          for (int q = 0; q < 4; ++q) T = fma(d.c[q][k], m[q][k], T);
          x = fma(d.c[0][k], s[0][k], x);
          y = fma(d.c[1][k], s[1][k], y);
        }
        S = fma(cp, x, fma(cx, y, S));
      };
      const Poly4 dg = poly4(as.jg[j]);
      if (AHEAD) loads_ahead();
      along(d, t[kAdjT + 0], t[kAdjS + 0]);
      along(dg, t[kAdjT + 2], t[kAdjS + 2]);
    }
    // arrival-time derivatives: dDelta/dH = -k1 sin H, dDelta/dth = k1t cos H + k0t
    //   d/dH:   d(dDelta/dH) = -k1 cos H,      d(dDelta/dth) = -k1t sin H
    //   d/dlat: d(dDelta/dH) = -k1l sin H,     d(dDelta/dth) = k1tl cos H + k0tl
    const double k1 = sc.k1, k1t = sc.k1t, k1l = as.k1l, k1tl = as.k1tl, k0tl = as.k0tl;
    hd = site_head(scs[site + 1 < n_site ? site + 1 : site]);
    if (AHEAD) loads_ahead();
    double uc = 0.0, us = 0.0, wc = 0.0, ws = 0.0, w1 = 0.0;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      uc = fma(wu[i], tc[i], uc);
      us = fma(wu[i], ts[i], us);
      wc = fma(ww[i], tc[i], wc);
      ws = fma(ww[i], ts[i], ws);
      w1 = fma(ww[i], ap[i].q.tf, w1);
    }
    t[kAdjT + 1] = fma(-k1, uc, fma(-k1t, ws, t[kAdjT + 1]));
    t[kAdjT + 0] = fma(-k1l, us, fma(k1tl, wc, fma(k0tl, w1, t[kAdjT + 0])));
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      t[kAdjT + i] *= 2.0;
      t[kAdjS + i] *= 2.0;
    }
    out(site, t);
  }
}

// One grid point and one site (host checks).
template <int NPI, bool ROT>
__host__ __device__ inline void adjoint_point(const EventC& ec, const AdjEventC& ae, const SiteC& sc,
                                              const AdjSiteC& as, int32_t k, double* acc) {
  AdjPoint ap[1];
  adjoint_point_setup<NPI, ROT, 1>(ec, ae, {k}, ap);
  adjoint_sites<1, true, false>(ae, &sc, &as, 1, ap, [&](int, const double (&t)[kAdjN]) {
    for (int i = 0; i < kAdjN; ++i) acc[i] += t[i];
  });
}

}  // namespace gwf
