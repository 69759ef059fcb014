// gwf_model.hpp -- per-event, per-site and per-frequency mathematics of the
// Fisher/SNR path, shared by the HIP kernels of libgwf.
//
// The strain at interferometer i is h_i = A(f) Q_i(f) exp(i Psi_i(f)) with
//   A      restricted (Newtonian) amplitude, |h~| = sqrt(5/24) pi^{-2/3}
//          (G Mc/c^3)^{5/6} f^{-7/6} c/dL                          (sec. 2.2)
//   Q_i    F+_i (1+cos^2 iota)/2 + i Fx_i cos iota, the pattern-weighted
//          polarisations (sec. 3.1, GWAmplitudes)
//   Psi_i  2 pi f (tc + Delta_i) - Phic - pi/4 + Psi_PN, with Delta_i the
//          arrival-time offset of the site (Doppler term of the Earth-motion
//          footnote of sec. 3) and Psi_PN the TaylorF2 phase (sec. 2.2).
// Patterns and Delta_i are evaluated at the sidereal angle of t(f) = tc -
// tau*(f) when the Earth rotates (sec. 2.2, tau_star).
//
// Because every product entering SNR^2 and the Fisher matrix has the form
// d_a h d_b h^*, the common factor exp(i Psi_i) cancels:
//   d_a h_i = A (D_a + ...) exp(i Psi_i),  D_a = d_a Q_i + Q_i d_a ln A + i Q_i d_a Psi_i,
// so no sine or cosine of the (large) phase is ever needed here, only its
// derivatives.  Those of the PN phase are polynomials in v = (pi G M f/c^3)^{1/3}
// and ln v whose per-event coefficients are built once (PhaseSeries).
//
// Antenna patterns are written in closed form in the hour angle H of the
// source at the site: with E, N the local East/North unit vectors and the
// polarisation frame (e_phi, e_theta) of the source,
//   EX = E.e_phi = cos H,           EY = E.e_theta = -cos th sin H,
//   NX = N.e_phi = -sin lat sin H,  NY = N.e_theta = -sin lat cos th cos H - cos lat sin th,
// the detector tensor (sin zeta/2)[sin 2g (EE-NN) - cos 2g (EN+NE)] gives
//   F+ = sin z [a cos 2psi + b sin 2psi],  Fx = sin z [b cos 2psi - a sin 2psi],
//   a = sin2g P1 - cos2g P2,  b = sin2g P3 - cos2g P4,
//   P1 = (EX^2 - NX^2 - EY^2 + NY^2)/2, P2 = EX NX - EY NY,
//   P3 = EX EY - NX NY,  P4 = EX NY + NX EY,
// a derivation of this library (equivalent to the tensor contraction).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "gwf_arith.hpp"

namespace gwf {

// ----------------------------------------------------------- constants
// IAU 2015 nominal values (the paper fixes none numerically).
constexpr double kPi = 3.14159265358979323846;
constexpr double kTwoPi = 2.0 * kPi;
constexpr double kC = 299792458.0;
constexpr double kGMsun = 1.3271244e20;
constexpr double kTsun = kGMsun / (kC * kC * kC);           // s
constexpr double kAU = 149597870700.0;
constexpr double kPc = kAU * 648000.0 / kPi;                 // m
constexpr double kGpcS = 1e9 * kPc / kC;                     // s
constexpr double kSiderealDay = 86164.0905;                  // s
constexpr double kOmegaE = kTwoPi / kSiderealDay;            // rad/s
constexpr double kREarthS = 6.371e6 / kC;                    // s
constexpr double kEulerGamma = 0.5772156649015329;
constexpr double kLn2 = 0.69314718055994530942;

constexpr int kMaxSites = 8;
constexpr int kMaxPar = 14;     // Fisher rows with tides and eccentricity
constexpr int kMaxIfo = 16;
constexpr uint32_t kFlagRot = 1;
constexpr uint32_t kFlagTidal = 2;
constexpr uint32_t kFlagMixed = 4;
constexpr uint32_t kFlagEcc = 8;
constexpr int kNparIn = 15;      // event inputs: the 13 parameters, e0, f_ref (0: the grid start)

enum : int32_t { kEvInvalid = 1, kEvNotPD = 2, kEvIllCond = 4, kEvNonFinite = 8, kEvSkipped = 16, kEvSvd = 32 };

// ------------------------------------------------------------ series
// Per-event coefficients of a PN-phase derivative:
//   s(v) = v^-5 (c0 + c1 v + ... + c7 v^7) + ln v (l5 + l6 v) + v^5 (t10 + t12 v^2)
struct PhaseSeries {
  double c[8];
  double l5, l6, t10, t12;
};
// Per-event coefficients of a tau*-type series:
//   s(v) = v^-8 (c0 + c1 v + ... + c7 v^7) + l6 ln v v^-2
struct TauSeries {
  double c[8];
  double l6;
};

// Index of the phase-derivative series in EventC::ps.
enum { kPsMc = 0, kPsEta, kPsChi1, kPsChi2, kPsL1, kPsL2 };
// Index of the tau-type series in EventC::ts: the rotation angle offset
// -Omega tau*, and the derivatives of the sidereal angle w.r.t. Mc and eta.
enum { kTsTheta = 0, kTsMc, kTsEta };

struct EventC {
  // grid: v_k = exp(lnv0 + k dlnv), f_k = v_k^3 / (pi M), trapezoid weights
  double lnv0, dlnv, inv_piM, piM, wint, wfirst, wlast;
  // sqrt(w KA4 / (pi M)) for the three weights: sqrt(4 w_k A_k^2) = rw v_k^-2
  // (the Fisher kernels' root weight).  Kernels holding the struct in LDS read
  // the fields in 16-byte pairs
  double rwint, rwfirst, rwlast;
  // work-item kernels: the ratios of a workgroup's step along the log grid
  // (GridWalk), here and in place of the explicit grid's
  double walk_v;
  // explicit grid: the event's frequencies (NULL on a log grid) and ln(pi M),
  // v_k = exp((ln(pi M) + ln f_k)/3), weights (f_{k+1} - f_{k-1})/2
  union {
    const double* fx;
    double walk_iv;
  };
  union {
    double lnpiM;
    double walk_psd;
  };
  int32_t n;
  int32_t status;              // of the event; status_circ: with e0 left out of it
  // amplitude: A^2 = KA v^-7 (factor 4 of the inner product included)
  double KA4;
  double dlnA_dMc, inv_dL;
  // sky/orientation
  double thc;                  // sidereal angle at coalescence, 2 pi tcoal
  double cplus, ccross, dcplus, dcross;   // (1+cos^2 i)/2, cos i and d/d iota
  // their products in the per-point rows of iota, psi and the SNR density:
  // c+^2, cx^2, c+ dcx - cx dc+, -2 c+ cx
  double cp2, cx2, u_iota, u_psi;
  PhaseSeries ps[6];
  TauSeries ts[3];
  // waveform only: Psi_PN / (2 pi) in cycles, ln of the amplitude factor
  // (A = exp(lnA - 3.5 ln v)), and -(Phic + pi/4)/(2 pi)
  PhaseSeries cyc;
  double lnA, cyc0;
  // moderate eccentricity (ecc != 0): the phase gains ecc_psi v^-5 r with
  // r = (v_ref/v)^{19/3} = exp((19/3)(ecc_lnvr - ln v)); ecc_mc v^-5 r joins
  // dPsi/dMc and ecc_e0 v^-5 r is dPsi/de0 (eta does not enter at fixed Mc)
  double ecc_lnvr, ecc_psi, ecc_mc, ecc_e0, ecc_cyc;
  int32_t ecc, status_circ;
};

struct SiteC {
  double cdl, sdl;             // cos, sin of (site longitude - phi)
  double k1, k0, k1t, k0t;     // Delta = k1 cos H + k0;  dDelta/dth = k1t cos H + k0t
  // (f0/f)^2 = ix2_fac v^-6; (f/f0)^2 = x2_fac v^6; a sampled curve has the
  // two coefficients of its interval guess here (see table_setup)
  union { double ix2_fac, tab_a; };
  union { double x2_fac, tab_b; };
  double xp_fac;               // (f/f0)^-4.14 = xp_fac v^-12.42
  // S0 times the PSD shape's coefficients of v^-12.42, v^-6 and the rational
  // part (the root weight's form, see psd_root_weight), and sqrt(1/S0)
  // (a sampled curve: the ends of its range)
  double xpS0;
  union { double m5S0, tab_lo; };
  union { double k111S0, tab_hi; };
  double rS0inv;
  double alpha[2][4], beta[2][4], weff[2];  // effective interferometers (pattern maps)
  // the effective interferometers' F+, Fx and their theta derivatives as
  // trigonometric polynomials in the hour angle H: coefficients of
  // (1, cos H, sin H, cos 2H, sin H cos H), each scaled by sqrt(weff)
  double jk[2][4][5];
  int32_t n_eff, n_arm;
  // sampled noise curve (tab_kind 1: PSD, 2: ASD; 0: the analytic PSD above)
  const double* tab_f;
  const double* tab_S;
  int64_t tab_n;
  int32_t tab_kind, tab_guess;
};

// Site description as passed at the boundary (radians); psd_kind 0 is the
// analytic PSD (S0, f0), 1 and 2 a sampled PSD or ASD (tab_f, tab_S,
// tab_n, scaled by S0).
struct SiteDesc {
  double lat, lon, gamma, zeta, S0, f0;
  int32_t shape, psd_kind;
  const double* tab_f;
  const double* tab_S;
  int64_t tab_n;
};

struct NetDesc {
  SiteDesc site[kMaxSites];
  int32_t n_site, n_ifo;
};

// Whether any site of the network has a sampled noise curve (the kernels
// without one leave the check out).
__host__ __device__ inline bool net_has_tables(const NetDesc& nd) {
  for (int s = 0; s < nd.n_site; ++s)
    if (nd.site[s].psd_kind != 0) return true;
  return false;
}

// The set-up below is compiled into many kernels, and an event has to get the
// same constants, bit for bit, in all of them: products and sums are fused by
// how they are written here, not as each kernel's code generation finds best.
#pragma clang fp contract(on)

// ------------------------------------------------ per-event coefficients
// Coefficients a_k (k = 0..7), b_5, b_6 (ln v parts) and tidal a_10, a_12 of
// the TaylorF2 phase Psi_PN = 3/(128 eta) v^-5 sum_k (a_k + b_k ln v) v^k,
// together with their partial derivatives with respect to eta (at fixed
// component spins and deformabilities), chi_s, chi_a, Lambda1, Lambda2.
// Point-particle terms to 3.5PN, aligned-spin spin-orbit terms to 3.5PN and
// 2PN spin-spin terms, tidal terms at 5PN/6PN through the combinations of
// eq. (LamTdelLam_def) (refs. of sec. 2.2).
struct PNCoef {
  double a[8], ae[8], as[8], aa[8];   // value, d/deta, d/dchi_s, d/dchi_a
  double b5, b5e, b5s, b5a, b6;
  double a10, a10e, a10_1, a10_2, a12, a12e, a12_1, a12_2;
};

__host__ __device__ inline void pn_coefficients(double eta, double chi1, double chi2, double L1,
                                                double L2, bool tidal, PNCoef& p) {
  const double pi = kPi, pi2 = kPi * kPi;
  const double e2 = eta * eta, e3 = e2 * eta;
  const double dl = sqrt(1.0 - 4.0 * eta);
  const double ddl = -2.0 / dl;     // d delta / d eta
  const double xs = 0.5 * (chi1 + chi2), xa = 0.5 * (chi1 - chi2);
  for (int k = 0; k < 8; ++k) { p.a[k] = 0.0; p.ae[k] = 0.0; p.as[k] = 0.0; p.aa[k] = 0.0; }
  p.a[0] = 1.0;
  // 1PN
  p.a[2] = 3715.0 / 756.0 + (55.0 / 9.0) * eta;
  p.ae[2] = 55.0 / 9.0;
  // 1.5PN: tail and spin-orbit
  p.a[3] = -16.0 * pi + (113.0 / 3.0) * dl * xa + (113.0 / 3.0 - (76.0 / 3.0) * eta) * xs;
  p.ae[3] = (113.0 / 3.0) * ddl * xa - (76.0 / 3.0) * xs;
  p.as[3] = 113.0 / 3.0 - (76.0 / 3.0) * eta;
  p.aa[3] = (113.0 / 3.0) * dl;
  // 2PN: point particle and spin-spin
  p.a[4] = 15293365.0 / 508032.0 + (27145.0 / 504.0) * eta + (3085.0 / 72.0) * e2 +
           (-405.0 / 8.0 + 200.0 * eta) * xa * xa - (405.0 / 4.0) * dl * xa * xs +
           (-405.0 / 8.0 + 2.5 * eta) * xs * xs;
  p.ae[4] = 27145.0 / 504.0 + (3085.0 / 36.0) * eta + 200.0 * xa * xa -
            (405.0 / 4.0) * ddl * xa * xs + 2.5 * xs * xs;
  p.as[4] = -(405.0 / 4.0) * dl * xa + 2.0 * (-405.0 / 8.0 + 2.5 * eta) * xs;
  p.aa[4] = 2.0 * (-405.0 / 8.0 + 200.0 * eta) * xa - (405.0 / 4.0) * dl * xs;
  // 2.5PN: X5 (1 + 3 ln v)
  const double q5 = 732985.0 / 2268.0 + (140.0 / 9.0) * eta;
  const double r5 = -732985.0 / 2268.0 + (24260.0 / 81.0) * eta + (340.0 / 9.0) * e2;
  const double X5 = pi * (38645.0 / 756.0 - (65.0 / 9.0) * eta) - q5 * dl * xa + r5 * xs;
  const double X5e = -(65.0 / 9.0) * pi - (140.0 / 9.0) * dl * xa - q5 * ddl * xa +
                     (24260.0 / 81.0 + (680.0 / 9.0) * eta) * xs;
  const double X5s = r5;
  const double X5a = -q5 * dl;
  p.a[5] = X5; p.ae[5] = X5e; p.as[5] = X5s; p.aa[5] = X5a;
  p.b5 = 3.0 * X5; p.b5e = 3.0 * X5e; p.b5s = 3.0 * X5s; p.b5a = 3.0 * X5a;
  // 3PN: Y6 - (6848/21) ln(4 v)
  const double Y6 = 11583231236531.0 / 4694215680.0 - (640.0 / 3.0) * pi2 -
                    (6848.0 / 21.0) * kEulerGamma +
                    (-15737765635.0 / 3048192.0 + (2255.0 / 12.0) * pi2) * eta +
                    (76055.0 / 1728.0) * e2 - (127825.0 / 1296.0) * e3 +
                    pi * ((2270.0 / 3.0) * dl * xa + (2270.0 / 3.0 - 520.0 * eta) * xs);
  const double Y6e = (-15737765635.0 / 3048192.0 + (2255.0 / 12.0) * pi2) +
                     (76055.0 / 864.0) * eta - (127825.0 / 432.0) * e2 +
                     pi * ((2270.0 / 3.0) * ddl * xa - 520.0 * xs);
  p.a[6] = Y6 - (6848.0 / 21.0) * (2.0 * kLn2);
  p.ae[6] = Y6e;
  p.as[6] = pi * (2270.0 / 3.0 - 520.0 * eta);
  p.aa[6] = pi * (2270.0 / 3.0) * dl;
  p.b6 = -6848.0 / 21.0;
  // 3.5PN
  const double u7 = -25150083775.0 / 3048192.0 + (26804935.0 / 6048.0) * eta - (1985.0 / 48.0) * e2;
  const double w7 = -25150083775.0 / 3048192.0 + (10566655595.0 / 762048.0) * eta -
                    (1042165.0 / 3024.0) * e2 + (5345.0 / 36.0) * e3;
  p.a[7] = pi * (77096675.0 / 254016.0 + (378515.0 / 1512.0) * eta - (74045.0 / 756.0) * e2) +
           u7 * dl * xa + w7 * xs;
  p.ae[7] = pi * (378515.0 / 1512.0 - (74045.0 / 378.0) * eta) +
            (26804935.0 / 6048.0 - (1985.0 / 24.0) * eta) * dl * xa + u7 * ddl * xa +
            (10566655595.0 / 762048.0 - (1042165.0 / 1512.0) * eta + (5345.0 / 12.0) * e2) * xs;
  p.as[7] = w7;
  p.aa[7] = u7 * dl;
  // tides: a10 = -(39/2) Lt, a12 = -(3115/64) Lt + (6595/364) delta dLt
  p.a10 = p.a10e = p.a10_1 = p.a10_2 = 0.0;
  p.a12 = p.a12e = p.a12_1 = p.a12_2 = 0.0;
  if (tidal) {
    const double s = L1 + L2, d = L1 - L2;
    const double q1 = 1.0 + 7.0 * eta - 31.0 * e2, q1e = 7.0 - 62.0 * eta;
    const double q2 = 1.0 + 9.0 * eta - 11.0 * e2, q2e = 9.0 - 22.0 * eta;
    const double Lt = (8.0 / 13.0) * (q1 * s + dl * q2 * d);
    const double Lte = (8.0 / 13.0) * (q1e * s + (ddl * q2 + dl * q2e) * d);
    const double Lt1 = (8.0 / 13.0) * (q1 + dl * q2), Lt2 = (8.0 / 13.0) * (q1 - dl * q2);
    const double r1 = 1.0 - (13272.0 / 1319.0) * eta + (8944.0 / 1319.0) * e2;
    const double r1e = -13272.0 / 1319.0 + (17888.0 / 1319.0) * eta;
    const double r2 = 1.0 - (15910.0 / 1319.0) * eta + (32850.0 / 1319.0) * e2 + (3380.0 / 1319.0) * e3;
    const double r2e = -15910.0 / 1319.0 + (65700.0 / 1319.0) * eta + (10140.0 / 1319.0) * e2;
    const double dLt = 0.5 * (dl * r1 * s + r2 * d);
    const double dLte = 0.5 * ((ddl * r1 + dl * r1e) * s + r2e * d);
    const double dLt1 = 0.5 * (dl * r1 + r2), dLt2 = 0.5 * (dl * r1 - r2);
    p.a10 = -19.5 * Lt; p.a10e = -19.5 * Lte; p.a10_1 = -19.5 * Lt1; p.a10_2 = -19.5 * Lt2;
    const double k12 = 6595.0 / 364.0;
    p.a12 = -(3115.0 / 64.0) * Lt + k12 * dl * dLt;
    p.a12e = -(3115.0 / 64.0) * Lte + k12 * (ddl * dLt + dl * dLte);
    p.a12_1 = -(3115.0 / 64.0) * Lt1 + k12 * dl * dLt1;
    p.a12_2 = -(3115.0 / 64.0) * Lt2 + k12 * dl * dLt2;
  }
}

// tau*(f) = 5 M/(256 eta) v^-8 sum_k (t_k + l_k ln v) v^k at 3.5PN, non-spinning
// (the paper cites Buonanno et al. 2009, eq. 3.8b); t_k and d t_k/d eta.
__host__ __device__ inline void tau_coefficients(double eta, double t[8], double te[8], double& l6) {
  const double pi = kPi, pi2 = kPi * kPi, e2 = eta * eta, e3 = e2 * eta;
  for (int k = 0; k < 8; ++k) { t[k] = 0.0; te[k] = 0.0; }
  t[0] = 1.0;
  t[2] = 743.0 / 252.0 + (11.0 / 3.0) * eta;               te[2] = 11.0 / 3.0;
  t[3] = -32.0 * pi / 5.0;
  t[4] = 3058673.0 / 508032.0 + (5429.0 / 504.0) * eta + (617.0 / 72.0) * e2;
  te[4] = 5429.0 / 504.0 + (617.0 / 36.0) * eta;
  t[5] = pi * (-7729.0 / 252.0 + (13.0 / 3.0) * eta);     te[5] = pi * 13.0 / 3.0;
  // (3424/105) ln(16 v^2) = (3424/105) (4 ln 2 + 2 ln v)
  t[6] = -10052469856691.0 / 23471078400.0 + (128.0 / 3.0) * pi2 + (6848.0 / 105.0) * kEulerGamma +
         (3147553127.0 / 3048192.0 - (451.0 / 12.0) * pi2) * eta - (15211.0 / 1728.0) * e2 +
         (25565.0 / 1296.0) * e3 + (3424.0 / 105.0) * 4.0 * kLn2;
  te[6] = (3147553127.0 / 3048192.0 - (451.0 / 12.0) * pi2) - (15211.0 / 864.0) * eta +
          (25565.0 / 432.0) * e2;
  t[7] = pi * (-15419335.0 / 127008.0 - (75703.0 / 756.0) * eta + (14809.0 / 378.0) * e2);
  te[7] = pi * (-75703.0 / 756.0 + (14809.0 / 189.0) * eta);
  l6 = 2.0 * 3424.0 / 105.0;
}

// Cut frequency: twice the ISCO orbital frequency, 1/(6^{3/2} pi G M/c^3)
// (sec. 2.2 footnote).
__host__ __device__ inline double cut_frequency_of(double M_s) {
  return 1.0 / (6.0 * sqrt(6.0) * kPi * M_s);
}

// x is neither infinite nor NaN (x - x is 0 exactly for finite x).
__host__ __device__ inline bool finite(double x) { return (x - x) == 0.0; }


// Rows of event e's Fisher matrix (bit r: row r; NULL: every row).
__host__ __device__ inline uint32_t event_rows(const uint32_t* par_mask, int64_t e) {
  return par_mask ? par_mask[e] : ~0u;
}

__host__ __device__ inline bool rows_in(uint32_t m, int r, int c) { return ((m >> r) & (m >> c) & 1u) != 0; }

// Parameter validity; returns the status bits of an event.
__host__ __device__ inline int32_t check_event(const double* p, bool tidal, double fmin, double fmax,
                                               int32_t n, bool ecc = false) {
  int32_t st = 0;
  const int np = tidal ? 13 : 11;
  for (int i = 0; i < np; ++i)
    if (!finite(p[i])) st |= kEvNonFinite;
  if (ecc && (!finite(p[13]) || !finite(p[14]))) st |= kEvNonFinite;
  if (!finite(fmin) || !finite(fmax)) st |= kEvNonFinite;
  if (st) return st;
  if (!(p[0] > 0.0) || !(p[1] > 0.0) || !(p[1] <= 0.25) || !(p[2] > 0.0)) st |= kEvInvalid;
  if (fabs(p[9]) > 1.0 || fabs(p[10]) > 1.0) st |= kEvInvalid;
  if (tidal && (p[11] < 0.0 || p[12] < 0.0)) st |= kEvInvalid;
  if (n < 2 || !(fmin > 0.0) || !(fmax > fmin)) st |= kEvInvalid;
  if (ecc && (!(p[13] >= 0.0) || !(p[13] < 1.0) || p[14] < 0.0)) st |= kEvInvalid;
  return st;
}

// Build the per-event constants.  p[13] are the parameters in boundary
// order; fmax <= 0 selects the cut frequency.
// The binary's total mass in seconds, M = Mc eta^(-3/5) G/c^3 (pi M sets the
// grid's v = (pi M f)^(1/3) and the PSD's x = f/f0 of every site).
__host__ __device__ inline double total_mass_s(const double* p) { return p[0] * pow(p[1], -0.6) * kTsun; }

// The constants fall into three parts that share nothing but p, so that the
// kernels can form them side by side, one wavefront or workgroup each (the
// chain of one lane doing all of them is 7 us).  An event whose status is set
// gets the other parts all the same; nothing reads them.
enum { kSetupGrid = 1, kSetupPhase = 2, kSetupAngle = 4, kSetupAll = 7 };

// The grid, the weights, the amplitude and the status.
__host__ __device__ inline void event_grid_setup(const double* p, double fmin, double fmax, int32_t n,
                                                 uint32_t flags, EventC& ec) {
  const double Mc = p[0], dL = p[2];
  const double Ms = total_mass_s(p);
  if (!(fmax > 0.0)) fmax = cut_frequency_of(Ms);
  ec.n = n;
  ec.fx = nullptr;
  // the SNR does not know e0: it is there for an event whose e0 alone is refused
  ec.status = ec.status_circ = check_event(p, (flags & kFlagTidal) != 0, fmin, fmax, n);
  if (flags & kFlagEcc) ec.status = check_event(p, (flags & kFlagTidal) != 0, fmin, fmax, n, true);
  if (ec.status_circ) return;
  // grid
  const double D = log(fmax / fmin) / (double)(n - 1);
  ec.piM = kPi * Ms;
  ec.inv_piM = 1.0 / ec.piM;
  ec.lnpiM = log(ec.piM);
  ec.lnv0 = (ec.lnpiM + log(fmin)) / 3.0;
  ec.dlnv = D / 3.0;
  ec.wint = sinh(D);                  // interior weight / f_k
  ec.wfirst = 0.5 * expm1(D);         // (f_1 - f_0)/2 / f_0
  ec.wlast = -0.5 * expm1(-D);        // (f_{n-1} - f_{n-2})/2 / f_{n-1}
  // amplitude: 4 A^2 = 4 (5/24) pi^{-4/3} (G Mc/c^3)^{5/3} f^{-7/3} (c/dL)^2, f^{-7/3} = (pi M)^{7/3} v^{-7}
  const double Mcs = Mc * kTsun, dLs = dL * kGpcS;
  ec.KA4 = 4.0 * (5.0 / 24.0) * pow(kPi, -4.0 / 3.0) * pow(Mcs, 5.0 / 3.0) * pow(ec.piM, 7.0 / 3.0) /
           (dLs * dLs);
  ec.rwint = sqrt(ec.wint * ec.KA4 * ec.inv_piM);
  ec.rwfirst = sqrt(ec.wfirst * ec.KA4 * ec.inv_piM);
  ec.rwlast = sqrt(ec.wlast * ec.KA4 * ec.inv_piM);
  ec.walk_v = 0.0;
  ec.dlnA_dMc = 5.0 / (6.0 * Mc);
  ec.inv_dL = 1.0 / dL;
  ec.lnA = 0.5 * log(0.25 * ec.KA4);
}

// The orientation, the eccentric terms and the sidereal-angle series.
__host__ __device__ inline void event_angle_setup(const double* p, double fmin, uint32_t flags, EventC& ec) {
  const bool rot = (flags & kFlagRot) != 0, ecc = (flags & kFlagEcc) != 0;
  const double Mc = p[0], eta = p[1], Ms = total_mass_s(p);
  // 2 pi tcoal reduced to [0, 2 pi)
  const double tfrac = p[7] - floor(p[7]);
  ec.thc = kTwoPi * tfrac;
  const double ci = cos(p[5]), si = sin(p[5]);
  ec.cplus = 0.5 * (1.0 + ci * ci);
  ec.ccross = ci;
  ec.dcplus = -ci * si;
  ec.dcross = -si;
  ec.cp2 = ec.cplus * ec.cplus;
  ec.cx2 = ec.ccross * ec.ccross;
  ec.u_iota = ec.cplus * ec.dcross - ec.ccross * ec.dcplus;
  ec.u_psi = -2.0 * ec.cplus * ec.ccross;

  // ---- moderate eccentricity (sec. 2.2, is_eccentric): the leading-order
  // correction -(2355/1462) e0^2 (v_ref/v)^{19/3} relative to the Newtonian
  // phase 3/(128 eta v^5) (the model the paper cites, Moore et al. 2016),
  // e0 given where the GW frequency is f_ref (the grid's first frequency
  // unless given, sec. 2.1).  At fixed f and f_ref it is proportional to
  // eta^-1 v^-5, i.e. to Mc^{-5/3} alone.
  ec.ecc = 0;
  ec.ecc_lnvr = ec.ecc_psi = ec.ecc_mc = ec.ecc_e0 = ec.ecc_cyc = 0.0;
  if (ecc) {
    const double e0 = p[13], fref = p[14] > 0.0 ? p[14] : fmin;
    const double K = (3.0 / (128.0 * eta)) * (-2355.0 / 1462.0);
    ec.ecc = 1;
    ec.ecc_lnvr = (log(kPi * Ms) + log(fref)) / 3.0;
    ec.ecc_psi = K * e0 * e0;
    ec.ecc_mc = -5.0 / (3.0 * Mc) * ec.ecc_psi;
    ec.ecc_e0 = 2.0 * K * e0;
    ec.ecc_cyc = ec.ecc_psi / kTwoPi;
  }
  ec.cyc0 = -(p[8] + 0.25 * kPi) / kTwoPi;

  // ---- rotation: sidereal-angle offset -Omega tau* and its Mc, eta derivatives
  double t[8], te[8], l6;
  tau_coefficients(eta, t, te, l6);
  const double Kt = 5.0 * Ms / (256.0 * eta);
  const double om = rot ? kOmegaE : 0.0;
  double lk[8] = {0, 0, 0, 0, 0, 0, l6, 0};
  for (int k = 0; k < 8; ++k) {
    ec.ts[kTsTheta].c[k] = -om * Kt * t[k];
    // d tau*/d Mc = (Kt/Mc) sum [(t_k + l_k L)(1 + (k-8)/3) + l_k/3] v^(k-8)
    ec.ts[kTsMc].c[k] = -om * (Kt / Mc) * ((1.0 + (k - 8) / 3.0) * t[k] + lk[k] / 3.0);
    // d tau*/d eta = Kt sum [t_k' - (k t_k + l_k)/(5 eta)] v^(k-8) + log part
    ec.ts[kTsEta].c[k] = -om * Kt * (te[k] - (k * t[k] + lk[k]) / (5.0 * eta));
  }
  ec.ts[kTsEta].c[0] = 0.0;   // leading tau* does not depend on eta at fixed Mc
  ec.ts[kTsTheta].l6 = -om * Kt * l6;
  ec.ts[kTsMc].l6 = -om * (Kt / Mc) * (1.0 + (6 - 8) / 3.0) * l6;
  ec.ts[kTsEta].l6 = -om * Kt * (-6.0 * l6 / (5.0 * eta));
}

// The phase series.
__host__ __device__ inline void event_phase_setup(const double* p, uint32_t flags, EventC& ec) {
  const bool tidal = (flags & kFlagTidal) != 0;
  const double Mc = p[0], eta = p[1];
  // ---- phase-derivative series
  PNCoef c;
  pn_coefficients(eta, p[9], p[10], tidal ? p[11] : 0.0, tidal ? p[12] : 0.0, tidal, c);
  const double A = 3.0 / (128.0 * eta);
  double b[8] = {0, 0, 0, 0, 0, c.b5, c.b6, 0};
  double be[8] = {0, 0, 0, 0, 0, c.b5e, 0.0, 0};
  // d Psi/d Mc = (1/(3 Mc)) v dPsi/dv
  {
    PhaseSeries& s = ec.ps[kPsMc];
    const double K = A / (3.0 * Mc);
    for (int k = 0; k < 8; ++k) s.c[k] = K * ((k - 5) * c.a[k] + b[k]);
    s.l5 = 0.0;
    s.l6 = K * c.b6;
    s.t10 = K * 5.0 * c.a10;
    s.t12 = K * 7.0 * c.a12;
  }
  // d Psi/d eta = explicit eta dependence - (1/(5 eta)) v dPsi/dv (v ~ eta^{-1/5})
  {
    PhaseSeries& s = ec.ps[kPsEta];
    const double K = A / (5.0 * eta);
    for (int k = 0; k < 8; ++k) s.c[k] = A * (c.ae[k] - c.a[k] / eta) - K * ((k - 5) * c.a[k] + b[k]);
    s.c[0] = 0.0;   // the leading term does not depend on eta at fixed Mc
    s.l5 = A * (be[5] - b[5] / eta);
    s.l6 = A * (-c.b6 / eta) - K * c.b6;
    s.t10 = A * (c.a10e - c.a10 / eta) - K * 5.0 * c.a10;
    s.t12 = A * (c.a12e - c.a12 / eta) - K * 7.0 * c.a12;
  }
  // spins: d/dchi1 = (d/dchi_s + d/dchi_a)/2, d/dchi2 = (d/dchi_s - d/dchi_a)/2
  for (int j = 0; j < 2; ++j) {
    PhaseSeries& s = ec.ps[kPsChi1 + j];
    const double sg = j == 0 ? 1.0 : -1.0;
    for (int k = 0; k < 8; ++k) s.c[k] = 0.5 * A * (c.as[k] + sg * c.aa[k]);
    s.l5 = 0.5 * A * (c.b5s + sg * c.b5a);
    s.l6 = 0.0;
    s.t10 = 0.0;
    s.t12 = 0.0;
  }
  // tides
  for (int j = 0; j < 2; ++j) {
    PhaseSeries& s = ec.ps[kPsL1 + j];
    for (int k = 0; k < 8; ++k) s.c[k] = 0.0;
    s.l5 = s.l6 = 0.0;
    s.t10 = A * (j == 0 ? c.a10_1 : c.a10_2);
    s.t12 = A * (j == 0 ? c.a12_1 : c.a12_2);
  }

  // Psi_PN itself, in cycles, for the strain output
  {
    PhaseSeries& s = ec.cyc;
    const double K = A / kTwoPi;
    for (int k = 0; k < 8; ++k) s.c[k] = K * c.a[k];
    s.l5 = K * c.b5;
    s.l6 = K * c.b6;
    s.t10 = K * c.a10;
    s.t12 = K * c.a12;
  }
}

__host__ __device__ inline void event_setup(const double* p, double fmin, double fmax, int32_t n,
                                            uint32_t flags, EventC& ec, int parts = kSetupAll) {
  if (parts & kSetupGrid) event_grid_setup(p, fmin, fmax, n, flags, ec);
  if (parts & kSetupAngle) event_angle_setup(p, fmin, flags, ec);
  if (parts & kSetupPhase) event_phase_setup(p, flags, ec);
}

// event_setup on event e's grid: the log descriptors, or an explicit grid
// (gf non-NULL; event e's npts[e] frequencies from gf + goff[e]) bounded by
// its first and last frequency, which must be positive and increasing (the
// event is flagged invalid otherwise, before any other frequency is read).
__host__ __device__ inline void event_setup_grid(const double* p, const double* fmin, const double* fmax,
                                                 const int32_t* npts, const int64_t* goff, const double* gf,
                                                 int64_t e, uint32_t flags, EventC& ec, int parts = kSetupAll) {
  const int32_t n = npts[e];
  if (gf) {
    const double* fx = gf + goff[e];
    const bool ok = n >= 2 && fx[0] > 0.0 && fx[n - 1] > fx[0];
    event_setup(p, ok ? fx[0] : 0.0, ok ? fx[n - 1] : 0.0, n, flags, ec, parts);
    if (parts & kSetupGrid) ec.fx = fx;
  } else {
    event_setup(p, fmin[e], fmax ? fmax[e] : 0.0, n, flags, ec, parts);
  }
}

// A function u + v cos H + w sin H of the hour angle H.
struct TrigLin {
  double u, v, w;
};

// Adds k a b to out, the coefficients of (1, cos H, sin H, cos 2H, sin H cos H).
__host__ __device__ inline void trig_mul_add(const TrigLin& a, const TrigLin& b, double k, double out[5]) {
  out[0] += k * fma(a.u, b.u, 0.5 * fma(a.v, b.v, a.w * b.w));
  out[1] += k * fma(a.u, b.v, a.v * b.u);
  out[2] += k * fma(a.u, b.w, a.w * b.u);
  out[3] += k * 0.5 * fma(a.v, b.v, -a.w * b.w);
  out[4] += k * fma(a.v, b.w, a.w * b.v);
}

// The pattern vector P(H) and its theta derivative as
// trigonometric polynomials of degree two in the hour angle: the frame
// components EX = cos H, EY = -cos th sin H, NX = -sin lat sin H,
// NY = -(sin lat cos th cos H + cos lat sin th) are linear in (cos H, sin H),
// and every component of P is a quadratic form in them.
__host__ __device__ inline void pattern_trig(double ct, double st, double sl, double cl, double pc[4][5],
                                             double ptc[4][5]) {
  const TrigLin EX{0.0, 1.0, 0.0}, EY{0.0, 0.0, -ct}, NX{0.0, 0.0, -sl}, NY{-cl * st, -sl * ct, 0.0};
  const TrigLin EYt{0.0, 0.0, st}, NYt{-cl * ct, sl * st, 0.0};    // theta derivatives (EX, NX do not move)
  for (int i = 0; i < 4; ++i)
    for (int m = 0; m < 5; ++m) pc[i][m] = ptc[i][m] = 0.0;
  trig_mul_add(EX, EX, 0.5, pc[0]);
  trig_mul_add(NX, NX, -0.5, pc[0]);
  trig_mul_add(EY, EY, -0.5, pc[0]);
  trig_mul_add(NY, NY, 0.5, pc[0]);
  trig_mul_add(EX, NX, 1.0, pc[1]);
  trig_mul_add(EY, NY, -1.0, pc[1]);
  trig_mul_add(EX, EY, 1.0, pc[2]);
  trig_mul_add(NX, NY, -1.0, pc[2]);
  trig_mul_add(EX, NY, 1.0, pc[3]);
  trig_mul_add(NX, EY, 1.0, pc[3]);
  trig_mul_add(EY, EYt, -1.0, ptc[0]);
  trig_mul_add(NY, NYt, 1.0, ptc[0]);
  trig_mul_add(EYt, NY, -1.0, ptc[1]);
  trig_mul_add(EY, NYt, -1.0, ptc[1]);
  trig_mul_add(EX, EYt, 1.0, ptc[2]);
  trig_mul_add(NX, NYt, -1.0, ptc[2]);
  trig_mul_add(EX, NYt, 1.0, ptc[3]);
  trig_mul_add(NX, EYt, 1.0, ptc[3]);
}

// Pattern maps of one interferometer: F+ = alpha.P, Fx = beta.P.
__host__ __device__ inline void pattern_map(double gamma, double zeta, double c2p, double s2p,
                                            double al[4], double be[4]) {
  const double sz = sin(zeta), s2g = sin(2.0 * gamma), c2g = cos(2.0 * gamma);
  al[0] = sz * s2g * c2p; al[1] = -sz * c2g * c2p; al[2] = sz * s2g * s2p; al[3] = -sz * c2g * s2p;
  be[0] = -sz * s2g * s2p; be[1] = sz * c2g * s2p; be[2] = sz * s2g * c2p; be[3] = -sz * c2g * c2p;
}

// A sampled curve's range (its end samples cover frequencies within a relative
// 1e-12 of them, so a grid starting on a sampled frequency keeps its first
// point whatever the rounding of f) and the guess of a frequency's interval:
// curve files are most often spaced evenly in ln f or in f, where the
// interval's number is linear in ln v (tab_guess 1: ln f = 3 ln v - ln(pi M))
// or in f (2).  Three samples decide; a guess is verified at every point, and a
// curve that follows neither (0) is searched by bisection.
__host__ __device__ inline void table_setup(const SiteDesc& sd, double piM, SiteC& sc) {
  constexpr double eps = 1e-12;
  const int64_t n = sd.tab_n, m = n - 1;
  const double fa = sd.tab_f[0], fb = sd.tab_f[m];
  sc.tab_lo = fa * (1.0 - eps);
  sc.tab_hi = fb * (1.0 + eps);
  sc.tab_a = sc.tab_b = 0.0;
  if (n < 4) return;
  const double la = log(fa), sl = (double)m / (log(fb) - la), sf = (double)m / (fb - fa);
  bool by_ln = true, by_f = true;
  for (int i = 1; i <= 3; ++i) {
    const int64_t j = (m * i) >> 2;
    const double fj = sd.tab_f[j];
    by_ln = by_ln && fabs((log(fj) - la) * sl - (double)j) < 0.5;
    by_f = by_f && fabs((fj - fa) * sf - (double)j) < 0.5;
  }
  if (by_ln) {
    sc.tab_guess = 1;
    sc.tab_a = 3.0 * sl;
    sc.tab_b = -(log(piM) + la) * sl;
  } else if (by_f) {
    sc.tab_guess = 2;
    sc.tab_a = sf;
    sc.tab_b = -fa * sf;
  }
}

// Per (event, site) constants.  A triangle (shape 1) is three 60-degree
// interferometers with bisectors at gamma + 30 deg + k 120 deg; since the
// third arm's response is minus the sum of the other two (closed loop,
// sec. 3.3), the Gram sum over its arms a a^T + b b^T + (a+b)(a+b)^T equals
// (3/2)(a+b)(a+b)^T + (1/2)(a-b)(a-b)^T: two effective interferometers.
// arm_on: bit k set where arm k of the site takes part (the duty factor).
// A triangle with all three arms uses the closure form (two effective
// interferometers with weights 3/2 and 1/2); with some arms off, every arm
// that is on is its own effective interferometer.  A site with no arm on has
// none (its patterns are still set for the strain).
// piM: pi times the event's total mass in seconds (EventC::piM, the only
// event constant a site needs).
__host__ __device__ inline void site_setup(const double* p, const SiteDesc& sd, double piM, SiteC& sc,
                                           uint32_t arm_on = 7u) {
  const double th = p[3], ph = p[4], psi = p[6];
  const double c2p = cos(2.0 * psi), s2p = sin(2.0 * psi);
  sc.cdl = cos(sd.lon - ph);
  sc.sdl = sin(sd.lon - ph);
  const double ct = cos(th), st = sin(th), sl = sin(sd.lat), cl = cos(sd.lat);
  // arrival-time offset -(n . r)/c with n.r/R = sin th cos lat cos H + cos th sin lat
  sc.k1 = -kREarthS * cl * st;
  sc.k0 = -kREarthS * sl * ct;
  sc.k1t = -kREarthS * cl * ct;
  sc.k0t = kREarthS * sl * st;
  const double lnx_off = -log(piM) - log(sd.f0);      // ln(f/f0) = 3 ln v + lnx_off
  sc.xp_fac = exp(-4.14 * lnx_off);
  const double ix_fac = sd.f0 * piM;          // f0/f = ix_fac v^-3
  sc.ix2_fac = ix_fac * ix_fac;
  sc.x2_fac = 1.0 / sc.ix2_fac;
  sc.xpS0 = sd.S0 * sc.xp_fac;
  sc.m5S0 = -5.0 * sd.S0 * sc.ix2_fac;
  sc.k111S0 = 111.0 * sd.S0;
  sc.rS0inv = sqrt(1.0 / sd.S0);
  sc.tab_f = sd.tab_f;
  sc.tab_S = sd.tab_S;
  sc.tab_n = sd.tab_n;
  sc.tab_kind = sd.psd_kind;
  sc.tab_guess = 0;
  if (sd.psd_kind) table_setup(sd, piM, sc);
  if (sd.shape == 1) {
    double al[3][4], be[3][4];
    for (int k = 0; k < 3; ++k)
      pattern_map(sd.gamma + kPi / 6.0 + kTwoPi * k / 3.0, kPi / 3.0, c2p, s2p, al[k], be[k]);
    sc.n_arm = 3;
    if ((arm_on & 7u) == 7u) {
      for (int j = 0; j < 4; ++j) {
        sc.alpha[0][j] = al[0][j] + al[1][j]; sc.beta[0][j] = be[0][j] + be[1][j];
        sc.alpha[1][j] = al[0][j] - al[1][j]; sc.beta[1][j] = be[0][j] - be[1][j];
      }
      sc.weff[0] = 1.5; sc.weff[1] = 0.5;
      sc.n_eff = 2;
    } else {
      int m = 0;
      for (int k = 0; k < 3; ++k)
        if (arm_on >> k & 1u) {
          for (int j = 0; j < 4; ++j) { sc.alpha[m][j] = al[k][j]; sc.beta[m][j] = be[k][j]; }
          sc.weff[m] = 1.0;
          ++m;
        }
      for (int r = m; r < 2; ++r) {
        for (int j = 0; j < 4; ++j) { sc.alpha[r][j] = 0.0; sc.beta[r][j] = 0.0; }
        sc.weff[r] = 0.0;
      }
      sc.n_eff = m;
    }
  } else {
    pattern_map(sd.gamma, sd.zeta, c2p, s2p, sc.alpha[0], sc.beta[0]);
    for (int j = 0; j < 4; ++j) { sc.alpha[1][j] = 0.0; sc.beta[1][j] = 0.0; }
    sc.weff[0] = 1.0; sc.weff[1] = 0.0;
    sc.n_eff = (arm_on & 1u) ? 1 : 0; sc.n_arm = 1;
  }
  double pc[4][5], ptc[4][5];
  pattern_trig(ct, st, sl, cl, pc, ptc);
  for (int j = 0; j < 2; ++j) {
    const double w = sqrt(sc.weff[j]);
    for (int m = 0; m < 5; ++m) {
      double fp = 0.0, fx = 0.0, fpt = 0.0, fxt = 0.0;
      for (int i = 0; i < 4; ++i) {
        fp = fma(sc.alpha[j][i], pc[i][m], fp);
        fx = fma(sc.beta[j][i], pc[i][m], fx);
        fpt = fma(sc.alpha[j][i], ptc[i][m], fpt);
        fxt = fma(sc.beta[j][i], ptc[i][m], fxt);
      }
      sc.jk[j][0][m] = w * fp;
      sc.jk[j][1][m] = w * fx;
      sc.jk[j][2][m] = w * fpt;
      sc.jk[j][3][m] = w * fxt;
    }
  }
}

__host__ __device__ inline void site_setup(const double* p, const SiteDesc& sd, const EventC& ec, SiteC& sc,
                                           uint32_t arm_on = 7u) {
  site_setup(p, sd, ec.piM, sc, arm_on);
}

// The arm mask of site s for event e from the per-interferometer flags
// active[ifo][ld] (NULL: every arm on); interferometers are numbered site
// by site, three for a triangle, one for an L.
__host__ __device__ inline uint32_t site_arms_on(const uint8_t* active, int64_t ld, int64_t e,
                                                 const NetDesc& net, int s) {
  if (!active) return 7u;
  int ifo0 = 0;
  for (int u = 0; u < s; ++u) ifo0 += net.site[u].shape == 1 ? 3 : 1;
  const int na = net.site[s].shape == 1 ? 3 : 1;
  uint32_t m = 0;
  for (int k = 0; k < na; ++k)
    if (active[(int64_t)(ifo0 + k) * ld + e]) m |= 1u << k;
  return m;
}

// site_setup's arm mask for a site's arms on their own: the first two of a
// triangle (the third response is minus their sum) or an L's one.
constexpr uint32_t kArmsPlain = 3u;

// The arms of site s that take part when only interferometer ifo_sel - 1 is
// wanted (ifo_sel = 0: every arm in `arms`).
__host__ __device__ inline uint32_t select_ifo(uint32_t arms, const NetDesc& net, int s, int ifo_sel) {
  if (ifo_sel <= 0) return arms;
  int ifo0 = 0;
  for (int u = 0; u < s; ++u) ifo0 += net.site[u].shape == 1 ? 3 : 1;
  const int k = ifo_sel - 1 - ifo0;
  const int na = net.site[s].shape == 1 ? 3 : 1;
  return (k >= 0 && k < na) ? (arms & (1u << k)) : 0u;
}

#pragma clang fp contract(fast)

// ---------------------------------------------------------- sin and cos
// sin and cos of a moderate angle (|x| < 1e5): Cody-Waite reduction by pi/2
// with a three-part constant, then the Taylor series of sin (to x^17) and
// cos (to x^18) on [-pi/4, pi/4], whose truncation errors (< 1e-19) are far
// below one ulp.  Used for the sidereal angle, which stays within tens of
// radians, instead of a general routine built for arbitrary arguments.
__host__ __device__ inline void sincos_moderate(double x, double* s, double* c) {
  // pi/2 = C1 + C2 + C3 (+1e-37): C1 and C2 are pi/2 and its remainder
  // rounded to 33 significant bits, so k*C1 and k*C2 are exact for |k| < 2^20
  constexpr double kInvPio2 = 0.63661977236758134308;
  constexpr double C1 = 1.5707963267341256e+00;
  constexpr double C2 = 6.077100506303966e-11;
  constexpr double C3 = 2.0222662487959506e-21;
  const double kf = rint(x * kInvPio2);
  double r = fma(-kf, C1, x);
  r = fma(-kf, C2, r);
  r = fma(-kf, C3, r);
  const double r2 = r * r;
  // sin r = r (1 - r^2/3! + r^4/5! - ...), cos r = 1 - r^2/2! + r^4/4! - ...
  double ps = -1.0 / 355687428096000.0;          // -1/17!
  ps = fma(ps, r2, 1.0 / 1307674368000.0);       //  1/15!
  ps = fma(ps, r2, -1.0 / 6227020800.0);         // -1/13!
  ps = fma(ps, r2, 1.0 / 39916800.0);            //  1/11!
  ps = fma(ps, r2, -1.0 / 362880.0);             // -1/9!
  ps = fma(ps, r2, 1.0 / 5040.0);                //  1/7!
  ps = fma(ps, r2, -1.0 / 120.0);                // -1/5!
  ps = fma(ps, r2, 1.0 / 6.0);                   //  1/3!
  const double sr = fma(-r * r2, ps, r);
  double pc = 1.0 / 6402373705728000.0;          //  1/18!
  pc = fma(pc, r2, -1.0 / 20922789888000.0);     // -1/16!
  pc = fma(pc, r2, 1.0 / 87178291200.0);         //  1/14!
  pc = fma(pc, r2, -1.0 / 479001600.0);          // -1/12!
  pc = fma(pc, r2, 1.0 / 3628800.0);             //  1/10!
  pc = fma(pc, r2, -1.0 / 40320.0);              // -1/8!
  pc = fma(pc, r2, 1.0 / 720.0);                 //  1/6!
  pc = fma(pc, r2, -1.0 / 24.0);                 // -1/4!
  pc = fma(pc, r2, 0.5);                         //  1/2!
  const double cr = fma(-r2, pc, 1.0);
  const int q = (int)kf & 3;
  const double ss = (q & 1) ? cr : sr;
  const double cc = (q & 1) ? sr : cr;
  *s = (q & 2) ? -ss : ss;
  *c = ((q + 1) & 2) ? -cc : cc;
}

// ------------------------------------------------------ per-point pieces
// Powers of v at one grid point, shared by every PN series of the point.
struct VPow {
  double p1, p2, p3, p4, p5, p6, p7;   // v^1 .. v^7
  double L, Lv;                        // ln v and v ln v
};

__host__ __device__ inline void vpow(double v, double L, VPow& w) {
  w.p1 = v;
  w.p2 = v * v;
  w.p3 = w.p2 * v;
  w.p4 = w.p2 * w.p2;
  w.p5 = w.p4 * v;
  w.p6 = w.p3 * w.p3;
  w.p7 = w.p4 * w.p3;
  w.L = L;
  w.Lv = L * v;
}

// c0 + c2 v^2 + ... + c7 v^7 as a sum of products with the powers, lowest
// order first and c0 last (no series has a term c1 v: there is no 0.5PN
// order); FIRST = 2 for a series without c0 as well, 3 for one that starts
// at c3 v^3, where c0 and c2 are zero by construction too.  Each fused multiply-add keeps the running sum as
// its addend, so per-event coefficients held in scalar registers enter every
// step directly (a Horner recurrence makes the coefficient the addend, which
// costs two register copies per step on this ISA).
template <int FIRST = 0>
__host__ __device__ inline double series7(const double c[8], const VPow& w) {
  double h;
  if (FIRST == 3) {
    h = c[3] * w.p3;
  } else {
    h = c[2] * w.p2;
    h = fma(c[3], w.p3, h);
  }
  h = fma(c[4], w.p4, h);
  h = fma(c[5], w.p5, h);
  h = fma(c[6], w.p6, h);
  h = fma(c[7], w.p7, h);
  return FIRST == 0 ? h + c[0] : h;
}

// A phase series (PhaseSeries) at v: v^-5 (sum c_k v^k) + (l5 + l6 v) ln v
// + t10 v^5 + t12 v^7.
__host__ __device__ inline double eval_phase(const PhaseSeries& s, const VPow& w, double iv5) {
  const double rest = fma(s.l6, w.Lv, fma(s.l5, w.L, fma(s.t12, w.p7, s.t10 * w.p5)));
  return fma(series7(s.c, w), iv5, rest);
}
// The Mc series, whose l5 is zero, the eta series, whose c0 is (at fixed Mc
// the leading order does not depend on eta), and the spin series, which
// start at 1.5PN and whose l6, t10 and t12 are zero, all by construction.
__host__ __device__ inline double eval_phase_mc(const PhaseSeries& s, const VPow& w, double iv5) {
  return fma(series7(s.c, w), iv5, fma(s.l6, w.Lv, fma(s.t12, w.p7, s.t10 * w.p5)));
}
__host__ __device__ inline double eval_phase_eta(const PhaseSeries& s, const VPow& w, double iv5) {
  const double rest = fma(s.l6, w.Lv, fma(s.l5, w.L, fma(s.t12, w.p7, s.t10 * w.p5)));
  return fma(series7<2>(s.c, w), iv5, rest);
}
__host__ __device__ inline double eval_phase_spin(const PhaseSeries& s, const VPow& w, double iv5) {
  return fma(series7<3>(s.c, w), iv5, s.l5 * w.L);
}
// The deformability series, which only have the tidal terms.
__host__ __device__ inline double eval_phase_tidal(const PhaseSeries& s, const VPow& w) {
  return fma(s.t12, w.p7, s.t10 * w.p5);
}
// A tau*-type series at v: v^-8 (sum c_k v^k) + l6 ln v v^-2 (FIRST = 2: the
// eta series, whose c0 is zero as that of the phase).
template <int FIRST = 0>
__host__ __device__ inline double eval_tau(const TauSeries& s, const VPow& w, double iv8, double iv2) {
  return fma(series7<FIRST>(s.c, w), iv8, s.l6 * (w.L * iv2));
}

// Frequency-point quantities shared by all sites.
struct Point {
  double v, iv, L, f, tf, w4A2;   // tf = 2 pi f; w4A2 = 4 w A^2 (PSD not yet applied)
  double rw;                      // sqrt(w4A2)
  double cth, sth;                // cos, sin of the sidereal angle at t(f)
  double gMc, gEta;               // d(sidereal angle)/dMc, /deta
  double pMc, pEta;               // dPsi_PN/dMc, /deta
  double vpsd;                    // v^-12.42: the PSD's power law, shared by all sites
  double v6, iv6;                 // v^6 and v^-6 (proportional to f^2 and f^-2), shared by all sites
  double ecv;                     // v^-5 (v_ref/v)^{19/3} (eccentric forms, else 0)
};

// v = exp(ln v), 1/v and the PSD's power law v^-12.42 at the points k,
// k + stride, k + 2 stride, ... of a log grid (ln v linear in k): evaluated
// once at the first point, then multiplied by the ratios exp(stride dlnv),
// exp(-stride dlnv), exp(-12.42 stride dlnv) per step.  After m steps each
// value carries a relative error of at most about (2m + 1) u (u = 2^-53) on
// top of that of its first evaluation: 1.4e-14 for the 63 steps of a
// 16384-point work item walked by 256 lanes, far inside the Fisher and SNR
// tolerances, for three multiplications per point instead of two
// exponentials and a reciprocal.
__host__ __device__ inline void grid_values(const EventC& ec, int32_t k, double* val) {
  const double L = fma((double)k, ec.dlnv, ec.lnv0);
  val[0] = exp(L);
  val[1] = exp(-L);
  val[2] = exp(-12.42 * L);
}

struct GridWalk {
  double val[3];      // v, 1/v, v^-12.42 at the current point
  double ratio[3];
  __host__ __device__ inline void start(const EventC& ec, int32_t k, int32_t stride) {
    grid_values(ec, k, val);
    set_ratios(ec, stride);
  }
  __host__ __device__ inline void set_ratios(const EventC& ec, int32_t stride) {
    const double D = (double)stride * ec.dlnv;
    ratio[0] = exp(D);
    ratio[1] = exp(-D);
    ratio[2] = exp(-12.42 * D);
  }
  // start with the ratios that keep_ratios has left in ec: three exponentials less
  // in every workgroup (SNR of 3000 neutron-star pairs 248 -> 242 us, 500 pairs'
  // matrices of five interferometers 479 -> 473 us)
  __host__ __device__ inline void start_kept(const EventC& ec, int32_t k) {
    grid_values(ec, k, val);
    ratio[0] = ec.walk_v;
    ratio[1] = ec.walk_iv;
    ratio[2] = ec.walk_psd;
  }
  __host__ __device__ static inline void keep_ratios(EventC& ec, int32_t stride) {
    GridWalk gw;
    gw.set_ratios(ec, stride);
    ec.walk_v = gw.ratio[0];
    ec.walk_iv = gw.ratio[1];
    ec.walk_psd = gw.ratio[2];
  }
  __host__ __device__ inline void step() {
    val[0] *= ratio[0];
    val[1] *= ratio[1];
    val[2] *= ratio[2];
  }
  // the values at point k evaluated directly again (ratios kept)
  __host__ __device__ inline void anchor(const EventC& ec, int32_t k) { grid_values(ec, k, val); }
};

// Number of phase-only Fisher parameters (Phic, chi1z, chi2z, then Lambda1,
// Lambda2 with tides, then e0 with eccentricity) and what it implies.
template <int NPI>
struct PhaseOnly {
  static_assert(NPI >= 3 && NPI <= 6, "3 to 6 phase-only parameters");
  static constexpr bool tidal = NPI >= 5;
  static constexpr bool ecc = (NPI & 1) == 0;
  static constexpr int P = 8 + NPI;
};

// How point_setup forms the PSD's power law v^-12.42 shared by all sites:
// not at all, in FP64, or in FP32 (the mixed form's weight).
enum PsdPow { kPsdNone = 0, kPsdF64 = 1, kPsdF32 = 2 };

// Keeps the compiler from turning the uniform branch it stands in into
// selects that every lane pays for.
__host__ __device__ inline void keep_branch() {
#if defined(__HIP_DEVICE_COMPILE__)
  __asm__ volatile("");
#endif
}

// The point's derivatives of the PN phase and of the sidereal angle with
// respect to Mc and eta, from the v, 1/v and ln v of point_setup.
template <bool ECC>
__host__ __device__ inline void point_derivatives(const EventC& ec, bool rot, Point& q) {
  const double iv2 = q.iv * q.iv, iv4 = iv2 * iv2, iv5 = iv4 * q.iv, iv8 = iv4 * iv4;
  VPow pw;
  vpow(q.v, q.L, pw);
  q.gMc = rot ? eval_tau(ec.ts[kTsMc], pw, iv8, iv2) : 0.0;
  q.gEta = rot ? eval_tau<2>(ec.ts[kTsEta], pw, iv8, iv2) : 0.0;
  q.pMc = eval_phase_mc(ec.ps[kPsMc], pw, iv5);
  q.pEta = eval_phase_eta(ec.ps[kPsEta], pw, iv5);
  q.ecv = 0.0;
  if (ECC) {
    q.ecv = iv5 * exp((19.0 / 3.0) * (ec.ecc_lnvr - q.L));
    q.pMc = fma(ec.ecc_mc, q.ecv, q.pMc);
  }
}

// EXPL: the point of an explicit grid (ec.fx) rather than of the log grid.
// vrec (log grids only, NULL: evaluate directly): v, 1/v and v^-12.42 at the
// point, carried by the caller from an earlier point (see GridWalk).
// inner: the caller knows that k is neither end of the grid (a uniform value,
// so that the end weights cost a wavefront inside the grid nothing).
template <bool EXPL = false, bool ECC = false>
__host__ __device__ inline void point_setup(const EventC& ec, int32_t k, bool need_derivs, bool rot,
                                            Point& q, int psd = kPsdF64, const double* vrec = nullptr,
                                            bool inner = false) {
  double L, v, f, wf;               // wf: the trapezoid weight
  double rwe = 0.0;                 // log grid: sqrt(w KA4 / (pi M)) of the point's weight
  if (EXPL) {
    f = ec.fx[k];
    L = (ec.lnpiM + log(f)) / 3.0;
    v = exp(L);
    wf = 0.5 * (ec.fx[k < ec.n - 1 ? k + 1 : k] - ec.fx[k > 0 ? k - 1 : k]);
  } else {
    L = fma((double)k, ec.dlnv, ec.lnv0);
    v = vrec ? vrec[0] : exp(L);
    f = (v * v * v) * ec.inv_piM;
    double w = ec.wint;
    rwe = ec.rwint;
    if (!inner) {
      keep_branch();
      if (k == 0) {
        w = ec.wfirst;
        rwe = ec.rwfirst;
      }
      if (k == ec.n - 1) {
        w = ec.wlast;
        rwe = ec.rwlast;
      }
    }
    wf = w * f;
  }
  const double iv = (!EXPL && vrec) ? vrec[1] : recip(v);
  const double iv2 = iv * iv, iv4 = iv2 * iv2, iv5 = iv4 * iv, iv7 = iv5 * iv2, iv8 = iv4 * iv4;
  q.v = v; q.iv = iv; q.L = L; q.f = f;
  const double v3 = v * v * v;
  q.v6 = v3 * v3;
  q.iv6 = iv4 * iv2;
  q.tf = kTwoPi * f;
  q.w4A2 = wf * ec.KA4 * iv7;
  q.rw = EXPL ? sqrt(q.w4A2) : rwe * iv2;
  q.vpsd = 0.0;
  if (!EXPL && vrec && psd != kPsdNone) {
    q.vpsd = vrec[2];
  } else if (psd == kPsdF64) {
    q.vpsd = exp(-12.42 * L);
  } else if (psd == kPsdF32) {   // 2^y with the integer part of y split off exactly
    const double y = (-12.42 / kLn2) * L, ny = rint(y);
    q.vpsd = (double)ldexpf(exp2f((float)(y - ny)), (int)ny);
  }
  VPow pw;
  vpow(v, L, pw);
  const double th = rot ? ec.thc + eval_tau(ec.ts[kTsTheta], pw, iv8, iv2) : ec.thc;
  sincos_moderate(th, &q.sth, &q.cth);
  if (need_derivs) point_derivatives<ECC>(ec, rot, q);
}

// The phase-only derivative coefficients of a point: c = (-1, dPsi/dchi1,
// dPsi/dchi2[, dPsi/dLambda1, dPsi/dLambda2][, dPsi/de0]).
template <int NPI>
__host__ __device__ inline void phase_only_coefficients(const EventC& ec, const Point& q, double* c) {
  using PO = PhaseOnly<NPI>;
  const double iv = q.iv, iv2 = iv * iv, iv5 = iv2 * iv2 * iv;
  VPow pw;
  vpow(q.v, q.L, pw);
  c[0] = -1.0;
  c[1] = eval_phase_spin(ec.ps[kPsChi1], pw, iv5);
  c[2] = eval_phase_spin(ec.ps[kPsChi2], pw, iv5);
  if (PO::tidal) {
    c[3] = eval_phase_tidal(ec.ps[kPsL1], pw);
    c[4] = eval_phase_tidal(ec.ps[kPsL2], pw);
  }
  if (PO::ecc) c[NPI - 1] = ec.ecc_e0 * q.ecv;
}

// A sampled noise curve at f (sec. 3.1, a PSD or ASD file): the PSD between
// two samples on the straight line through them (an ASD squared at the samples
// first), not yet scaled by S0; false outside the sampled range.  Where the
// curve has a guess for f's interval (table_setup), the four samples about it
// and their values are read at once, and the interval among their three that
// holds f is taken: one round of memory latency for any number of samples.
// Otherwise, or if f is in none of the three, the interval is found by
// bisection, a chain of log2(n) dependent reads.  Measured on 3000 neutron-star
// binaries with curves of 900-3200 samples evenly spaced in ln f: SNR 2.03 ms
// by bisection, 0.71 ms with the guess.
__host__ __device__ inline bool table_psd(const SiteC& sc, const Point& q, double& S) {
  const double f = q.f;
  if (!(f >= sc.tab_lo) || !(f <= sc.tab_hi)) return false;
  const double* __restrict__ tf = sc.tab_f;
  const double* __restrict__ tS = sc.tab_S;
  const int64_t n = sc.tab_n;
  double f0, f1, s0, s1;
  bool found = false;
  if (sc.tab_guess) {
    const double x = fma(sc.tab_a, sc.tab_guess == 1 ? q.L : f, sc.tab_b);
    int32_t g = (int32_t)fmin(fmax(x, 1.0), (double)(n - 3));     // 1 <= g <= n - 3
    const double fm = tf[g - 1], fg = tf[g], fp = tf[g + 1], fq = tf[g + 2];
    const double sm = tS[g - 1], sg = tS[g], sp = tS[g + 1], sq = tS[g + 2];
    const bool below = f < fg, above = f >= fp;
    f0 = below ? fm : above ? fp : fg;
    f1 = below ? fg : above ? fq : fp;
    s0 = below ? sm : above ? sp : sg;
    s1 = below ? sg : above ? sq : sp;
    found = (f >= f0 || (below && g == 1)) && (f < f1 || (above && g == n - 3));
  }
  if (!found) {
    int64_t lo = 0, hi = n - 1;
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1;
      if (tf[mid] <= f) lo = mid;
      else hi = mid;
    }
    f0 = tf[lo];
    f1 = tf[hi];
    s0 = tS[lo];
    s1 = tS[hi];
  }
  if (sc.tab_kind == 2) {
    s0 *= s0;
    s1 *= s1;
  }
  const double t = fmin(fmax((f - f0) * recip(f1 - f0), 0.0), 1.0);
  S = fma(t, s1 - s0, s0);
  return true;
}

// The square root of the weight 4 w A^2 / S_n(f) with a sampled curve; zero
// outside the sampled range and where the curve is infinite.
__host__ __device__ inline double table_root_weight(const SiteC& sc, const Point& q) {
  double S;
  return table_psd(sc, q, S) ? (q.rw * sc.rS0inv) * rsqrt_inf_d(S) : 0.0;
}

// The square root of the weight, r = sqrt(4 w A^2 / S_n(f)), which the
// Fisher kernels fold into the pattern values: every Fisher entry is a sum of
// w Re(D_a D_b^*), bilinear in the derivative vectors, and those are linear
// in the pattern values, so the weighted sums follow from r D with no
// per-entry weight product.  S_n = S0 [x^-4.14 - 5 x^-2
// + 111 (1 - x^2 + x^4/2)/(1 + x^2/2)], x = f/f0, = S0 top / den, and
// r = sqrt(4 w A^2) den / sqrt(den S0 top); S0 top is formed from the site's
// S0-scaled coefficients, so 1/S0 costs nothing per point.  A sampled curve
// takes the root of the full weight.  TAB = false: instantiations for networks
// without sampled curves, which leave the check out of the per-point code.
__host__ __device__ inline double psd_root_of(double x2_fac, double xpS0, double m5S0, double k111S0, const Point& q) {
  const double x2 = x2_fac * q.v6;                 // (f/f0)^2
  const double num = fma(fma(0.5, x2, -1.0), x2, 1.0);
  const double den = fma(0.5, x2, 1.0);
  const double topS = fma(fma(m5S0, q.iv6, xpS0 * q.vpsd), den, k111S0 * num);
  return (q.rw * den) * rsqrt_d(den * topS);
}

template <bool TAB = true>
__host__ __device__ inline double psd_root_weight(const SiteC& sc, const Point& q) {
  if (TAB && sc.tab_kind)
    return table_root_weight(sc, q);
  return psd_root_of(sc.x2_fac, sc.xpS0, sc.m5S0, sc.k111S0, q);
}

// The weight w / S_n(f) itself, for w = 4 w A^2, as the SNR kernels take it: it
// enters their sums as it is, so that a sampled value that is zero, negative or
// infinite gives an infinite, negative or no contribution.
template <bool TAB = true>
__host__ __device__ inline double psd_weight(const SiteC& sc, const Point& q, double w) {
  if (TAB && sc.tab_kind) {
    double S;
    return table_psd(sc, q, S) ? w * (sc.rS0inv * sc.rS0inv) / S : 0.0;
  }
  const double x2 = sc.x2_fac * q.v6;
  const double num = fma(fma(0.5, x2, -1.0), x2, 1.0);
  const double den = fma(0.5, x2, 1.0);
  const double topS = fma(fma(sc.m5S0, q.iv6, sc.xpS0 * q.vpsd), den, sc.k111S0 * num);
  return w * den * recip(topS);
}

// The same root with the PSD shape in FP32 (mixed form).  The weight is a
// positive factor per grid point, so a relative error e in it keeps the
// Fisher matrix between (1 - e) Gamma and (1 + e) Gamma in the
// positive-semidefinite order: SNR^2 moves by at most e and every sigma_i by
// at most about e/2, whatever the condition number.  Errors in the response
// vectors or in the sums have no such bound, which is why they stay FP64.
// x^-4.14 = xp_fac v^-12.42, the power of v taken once per point; x^2 and x^-2
// are FP64 products rounded once; sqrt(den / top) in FP32 (den/top = S0/S_n
// stays within FP32's range), so a relative error e in r is one of about 2e in
// the weight.  Measured on sampled events of the BNS catalogue: Fisher within
// 4.2e-8 of sqrt(Gamma_aa Gamma_bb), SNR within 1.9e-8.
template <bool TAB = true>
__host__ __device__ inline double psd_root_weight_f32(const SiteC& sc, const Point& q) {
  if (TAB && sc.tab_kind)
    return table_root_weight(sc, q);
  const float xp = (float)(sc.xp_fac * q.vpsd);
  const float x2 = (float)(sc.x2_fac * q.v6), ix2 = (float)(sc.ix2_fac * q.iv6);
  const float num = fmaf(0.5f * x2, x2, 1.0f - x2);
  const float den = fmaf(0.5f, x2, 1.0f);
  const float top = fmaf(fmaf(-5.0f, ix2, xp), den, 111.0f * num);
  return (q.rw * sc.rS0inv) * (double)sqrtf_hw(den * recipf(top));
}

// The Fisher kernels' site quantities: the patterns' trigonometric basis
// scaled by the root weight r (psd_root_weight), so that SiteC::jk's
// polynomials give r F+, r Fx and their derivatives directly, and the
// arrival-time derivatives.
struct SiteTrigR {
  double r, rc, rs, rc2, rsc;   // r (1, cos H, sin H, cos 2H, sin H cos H)
  double rm4;                   // -4 r sin H cos H
  double u, w;                  // 2 pi f dDelta/dH, 2 pi f dDelta/dtheta
};

// cos and sin of the hour angle from a site's (cos, sin) of its longitude less
// phi, every product's rounding written out: left to the compiler, which of the
// two products of a sum is fused changes from kernel to kernel, and the same
// point would have other bits in each.
__host__ __device__ inline void hour_angle(const Point& q, double cdl, double sdl, double& cH, double& sH) {
  cH = fma(q.cth, cdl, -(q.sth * sdl));
  sH = fma(q.sth, cdl, q.cth * sdl);
}

__host__ __device__ inline void trig_basis(double cH, double sH, double r, SiteTrigR& sp) {
  sp.r = r;
  sp.rc = r * cH;
  sp.rs = r * sH;
  sp.rc2 = fma(sp.rc, cH, -sp.rs * sH);
  sp.rsc = sp.rs * cH;
  sp.rm4 = -4.0 * sp.rsc;
}

template <bool MIXED = false, bool TAB = true>
__host__ __device__ inline void site_trig_root(const SiteC& sc, const Point& q, SiteTrigR& sp) {
  double cH, sH;
  hour_angle(q, sc.cdl, sc.sdl, cH, sH);
  trig_basis(cH, sH, MIXED ? psd_root_weight_f32<TAB>(sc, q) : psd_root_weight<TAB>(sc, q), sp);
  sp.u = q.tf * (-sc.k1 * sH);
  sp.w = fma(q.tf, sc.k1t * cH, q.tf * sc.k0t);
}

// r times a trigonometric polynomial of SiteC::jk, and r times its H
// derivative (the constant term last: the coefficients sit in scalar registers,
// and as the first addend it would need copying into vector registers).
__host__ __device__ inline double trig_val_r(const double c[5], const SiteTrigR& sp) {
  return fma(c[0], sp.r, fma(c[4], sp.rsc, fma(c[3], sp.rc2, fma(c[2], sp.rs, c[1] * sp.rc))));
}
__host__ __device__ inline double trig_dH_r(const double c[5], const SiteTrigR& sp) {
  return fma(c[4], sp.rc2, fma(c[3], sp.rm4, fma(c[2], sp.rc, -c[1] * sp.rs)));
}

// The event's amplitude factors that enter the derivative vectors.
struct AmpFactors {
  double cplus, ccross, dcp, dcx, dlnA, idL;
};

__host__ __device__ inline AmpFactors amp_factors(const EventC& ec) {
  return AmpFactors{ec.cplus, ec.ccross, ec.dcplus, ec.dcross, ec.dlnA_dMc, ec.inv_dL};
}

// Marks v and 1/v as unknown to the compiler, so that their powers are formed
// again where they are needed next instead of being held in registers.
__host__ __device__ inline void reread(double& v, double& iv) {
#if defined(__HIP_DEVICE_COMPILE__)
  __asm__("" : "+v"(v), "+v"(iv));
#endif
}

// ------------------------------------------------ one frequency point
// With Q = (c+ F+, cx Fx) and its hour-angle and theta derivatives Q_H, Q_t as
// (re, im) pairs, u = 2 pi f dDelta/dH and w = 2 pi f dDelta/dtheta, put
//   Z = Q_H + i u Q,   Y = Q_t + i w Q.
// Then the derivative vectors of every interferometer are combinations of Q,
// iQ, Z and Y with coefficients that no site or interferometer changes:
//   D_Mc = dlnA Q + gMc Z + pMc iQ,   D_eta = gEta Z + pEta iQ,
//   D_theta = Y,   D_phi = -Z,   D_tc = Omega Z + 2 pi f iQ,
//   D_dL = -Q/dL,  D_iota = (dc+ F+, dcx Fx),  D_psi = (2 c+ Fx, -2 cx F+)
// (the phase derivatives' shares of the delay sit in Z and Y).  So a point's
// whole 8x8 block follows from 14 sums over its interferometers (NetSums): the
// loop over them takes 17 multiply-adds each instead of the 63 of a rank-2
// update of the five rows and their pattern moments, and the coefficients are
// applied once per point.
struct NetSums {
  double spp, spx, sxx;                // F+^2, F+ Fx, Fx^2
  double pzr, pzi, xzr, xzi;           // (F+, Fx) x (Re Z, Im Z)
  double pyr, pyi, xyr, xyi;           // (F+, Fx) x (Re Y, Im Y)
  double zz, yy, zy;                   // |Z|^2, |Y|^2, Re(Z Y^*)
};

// What a site's trigonometry and noise weight take from its constants.
struct SiteHead {
  double cdl, sdl, k1, k1t, k0t, x2_fac, xpS0, m5S0, k111S0;
};

__host__ __device__ inline SiteHead site_head(const SiteC& sc) {
  return SiteHead{sc.cdl, sc.sdl, sc.k1, sc.k1t, sc.k0t, sc.x2_fac, sc.xpS0, sc.m5S0, sc.k111S0};
}

// The constants read before this line are asked for here, ahead of the work
// behind it: scalar loads complete out of order, so a use waits for every load
// in flight, and left alone the compiler puts each group right before its use.
__host__ __device__ inline void loads_ahead() {
#if defined(__HIP_DEVICE_COMPILE__)
  __asm__ volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// The root weight from the head, or from the site's other constants where the
// head has not all it takes.
template <bool MIXED, bool TAB>
__host__ __device__ inline double site_root(const SiteC& sc, const SiteHead& hd, const Point& q) {
  if (TAB || MIXED) return MIXED ? psd_root_weight_f32<TAB>(sc, q) : psd_root_weight<TAB>(sc, q);
  return psd_root_of(hd.x2_fac, hd.xpS0, hd.m5S0, hd.k111S0, q);
}

struct Poly4 {
  double c[4][5];
};

__host__ __device__ inline Poly4 poly4(const double (&p)[4][5]) {
  Poly4 r;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int k = 0; k < 5; ++k) r.c[q][k] = p[q][k];
  return r;
}

// Adds one site's n_eff = 1 or 2 effective interferometers to the sums of NQ
// points (of one event).  The patterns are trigonometric polynomials in H whose
// coefficients carry sqrt(weff), and the basis carries the root weight r, so
// every product of two of the values below is weighted by weff r^2.
// hd: the site's, left as next's (the site taken after this one).
// AHEAD: the constants sit in scalar registers, and a site's polynomials and
// the next site's head are asked for ahead of their use, two waits for scalar
// loads per site where there were four.  Plans of 10^4 BNS on three sites
// 2.111 and 2.104 ms, 5000 of all kinds with sampled curves 1.555 and 1.526,
// 5000 mixed pairs on five sites 1.475 and 1.460 (FP32 weights 1.470 and
// 1.437).  With eccentricity it is slower (2000 events 0.565 and 0.571 ms),
// and with the constants in LDS there is nothing to wait for.
template <int NQ, bool MIXED = false, bool TAB = true, bool AHEAD = false>
__host__ __device__ inline void site_sums(const AmpFactors& am, const Point (&q)[NQ], const SiteC& st, int n_eff,
                                          SiteHead& hd, const SiteC& next, NetSums (&net)[NQ]) {
  SiteTrigR sp[NQ];
  Poly4 p;
  if (AHEAD) {
    p = poly4(st.jk[0]);
    loads_ahead();
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      double cH, sH;
      hour_angle(q[i], hd.cdl, hd.sdl, cH, sH);
      trig_basis(cH, sH, site_root<MIXED, TAB>(st, hd, q[i]), sp[i]);
      sp[i].u = q[i].tf * (-hd.k1 * sH);
      sp[i].w = fma(q[i].tf, hd.k1t * cH, q[i].tf * hd.k0t);
    }
    hd = site_head(next);
    loads_ahead();
  } else {
#pragma unroll
    for (int i = 0; i < NQ; ++i) site_trig_root<MIXED, TAB>(st, q[i], sp[i]);
  }
  int j = 0;
  do {
    if (AHEAD && j > 0) p = poly4(st.jk[j]);
    const double(*c)[5] = AHEAD ? p.c : st.jk[j];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      NetSums& n = net[i];
      const double Fp = trig_val_r(c[0], sp[i]), Fx = trig_val_r(c[1], sp[i]);
      const double Qr = am.cplus * Fp, Qi = am.ccross * Fx;
      const double Zr = fma(am.cplus, trig_dH_r(c[0], sp[i]), -sp[i].u * Qi);
      const double Zi = fma(am.ccross, trig_dH_r(c[1], sp[i]), sp[i].u * Qr);
      const double Yr = fma(am.cplus, trig_val_r(c[2], sp[i]), -sp[i].w * Qi);
      const double Yi = fma(am.ccross, trig_val_r(c[3], sp[i]), sp[i].w * Qr);
      n.spp = fma(Fp, Fp, n.spp);
      n.spx = fma(Fp, Fx, n.spx);
      n.sxx = fma(Fx, Fx, n.sxx);
      n.pzr = fma(Fp, Zr, n.pzr);
      n.pzi = fma(Fp, Zi, n.pzi);
      n.xzr = fma(Fx, Zr, n.xzr);
      n.xzi = fma(Fx, Zi, n.xzi);
      n.pyr = fma(Fp, Yr, n.pyr);
      n.pyi = fma(Fp, Yi, n.pyi);
      n.xyr = fma(Fx, Yr, n.xyr);
      n.xyi = fma(Fx, Yi, n.xyi);
      n.zz = fma(Zr, Zr, fma(Zi, Zi, n.zz));
      n.yy = fma(Yr, Yr, fma(Yi, Yi, n.yy));
      n.zy = fma(Zr, Yr, fma(Zi, Yi, n.zy));
    }
  } while (++j < n_eff);
}

// Slots of the accumulator G[kGramAcc]: the sums over points of
//   the pattern products S, the products of (F+, Fx) with Z and with Y;
//   2 pi f times W = |Q|^2, U_iota and U_psi;
//   for b = Mc and eta, with D'_b = D_b - dlnA_b Q: U_b = Re(iQ D'_b^*),
//   g_b Re(Q Z^*), Re(D_iota D'_b^*), Re(D_psi D'_b^*);
//   the products of D'_Mc, D'_eta, Y, Z and 2 pi f iQ among each other.
enum {
  kGSpp = 0, kGSpx, kGSxx, kGPzr, kGPzi, kGXzr, kGXzi, kGPyr, kGPyi, kGXyr, kGXyi, kGTW, kGTI, kGTP,
  kGMu, kGMd, kGMi, kGMp, kGEu, kGEd, kGEi, kGEp,
  kGMM, kGME, kGEE, kGMY, kGEY, kGMZ, kGEZ, kGMt, kGEt, kGYY, kGZY, kGZZ, kGtY, kGtZ, kGtt,
  kGramAcc
};

// Adds a point's sums n to G[kGramAcc] and returns its phase-only quantities:
//   U[8]   U_b = sum_i w_i Re(i Q_i D_b,i^*)
//   W      sum_i w_i |Q_i|^2 (the SNR^2 density).
// The phase-only derivative vectors are i Q c(f) with the same real c(f) at
// every interferometer, so the blocks they span are
//   Gamma_{b, 8+i} += U_b c_i,   Gamma_{8+i, 8+j} += W c_i c_j,
// which the caller accumulates (see add_phase_blocks).
template <bool ROT>
__host__ __device__ inline void accumulate_sums(const EventC& ec, const Point& q, const NetSums& n, double* G,
                                                double* U, double& W) {
  const AmpFactors am = amp_factors(ec);
  const double pm = q.pMc, pe = q.pEta, gm = q.gMc, ge = q.gEta, tf = q.tf;
  G[kGSpp] += n.spp;
  G[kGSpx] += n.spx;
  G[kGSxx] += n.sxx;
  G[kGPzr] += n.pzr;
  G[kGPzi] += n.pzi;
  G[kGXzr] += n.xzr;
  G[kGXzi] += n.xzi;
  G[kGPyr] += n.pyr;
  G[kGPyi] += n.pyi;
  G[kGXyr] += n.xyr;
  G[kGXyi] += n.xyi;
  G[kGYY] += n.yy;
  G[kGZY] += n.zy;
  G[kGZZ] += n.zz;
  W = fma(ec.cp2, n.spp, ec.cx2 * n.sxx);
  const double ui = ec.u_iota * n.spx, up = ec.u_psi * (n.spp + n.sxx);
  const double iqz = fma(am.cplus, n.pzi, -am.ccross * n.xzr);    // Re(iQ Z^*)
  const double iqy = fma(am.cplus, n.pyi, -am.ccross * n.xyr);    // Re(iQ Y^*)
  const double tW = tf * W;
  G[kGTW] += tW;
  G[kGTI] = fma(tf, ui, G[kGTI]);
  G[kGTP] = fma(tf, up, G[kGTP]);
  G[kGtY] = fma(tf, iqy, G[kGtY]);
  G[kGtZ] = fma(tf, iqz, G[kGtZ]);
  G[kGtt] = fma(tf, tW, G[kGtt]);
  double mu, eu, mz, ez;               // Re(iQ D'^*), Re(Z D'^*) of D'_Mc and D'_eta
  if (ROT) {
    const double qz = fma(am.cplus, n.pzr, am.ccross * n.xzi);             // Re(Q Z^*)
    const double iz = fma(am.dcp, n.pzr, am.dcx * n.xzi);                  // Re(D_iota Z^*)
    const double pz = 2.0 * fma(am.cplus, n.xzr, -am.ccross * n.pzi);      // Re(D_psi Z^*)
    mu = fma(pm, W, gm * iqz);
    eu = fma(pe, W, ge * iqz);
    mz = fma(pm, iqz, gm * n.zz);
    ez = fma(pe, iqz, ge * n.zz);
    G[kGMd] = fma(gm, qz, G[kGMd]);
    G[kGMi] = fma(pm, ui, fma(gm, iz, G[kGMi]));
    G[kGMp] = fma(pm, up, fma(gm, pz, G[kGMp]));
    G[kGEd] = fma(ge, qz, G[kGEd]);
    G[kGEi] = fma(pe, ui, fma(ge, iz, G[kGEi]));
    G[kGEp] = fma(pe, up, fma(ge, pz, G[kGEp]));
    G[kGMM] = fma(pm, mu, fma(gm, mz, G[kGMM]));
    G[kGME] = fma(pe, mu, fma(ge, mz, G[kGME]));
    G[kGEE] = fma(pe, eu, fma(ge, ez, G[kGEE]));
    G[kGMY] = fma(pm, iqy, fma(gm, n.zy, G[kGMY]));
    G[kGEY] = fma(pe, iqy, fma(ge, n.zy, G[kGEY]));
  } else {                             // the sidereal angle does not move: gMc = gEta = 0
    mu = pm * W;
    eu = pe * W;
    mz = pm * iqz;
    ez = pe * iqz;
    G[kGMi] = fma(pm, ui, G[kGMi]);
    G[kGMp] = fma(pm, up, G[kGMp]);
    G[kGEi] = fma(pe, ui, G[kGEi]);
    G[kGEp] = fma(pe, up, G[kGEp]);
    G[kGMM] = fma(pm, mu, G[kGMM]);
    G[kGME] = fma(pe, mu, G[kGME]);
    G[kGEE] = fma(pe, eu, G[kGEE]);
    G[kGMY] = fma(pm, iqy, G[kGMY]);
    G[kGEY] = fma(pe, iqy, G[kGEY]);
  }
  G[kGMu] += mu;
  G[kGEu] += eu;
  G[kGMZ] += mz;
  G[kGEZ] += ez;
  G[kGMt] = fma(tf, mu, G[kGMt]);
  G[kGEt] = fma(tf, eu, G[kGEt]);
  U[0] = mu;
  U[1] = eu;
  U[2] = 0.0;
  U[3] = iqy;
  U[4] = -iqz;
  U[5] = ui;
  U[6] = up;
  U[7] = fma(kOmegaE, iqz, tW);
}

// The sites of an event that have an interferometer on, in order: four bits
// each, the site's number and (bit 3) whether it has two effective ones.
struct ActiveSites {
  uint32_t list;
  int32_t n;
};

__host__ __device__ inline ActiveSites active_sites(const SiteC* sc, int n_site) {
  ActiveSites a{0u, 0};
  for (int s = 0; s < n_site; ++s)
    if (sc[s].n_eff > 0) {
      a.list |= ((uint32_t)s | (sc[s].n_eff > 1 ? 8u : 0u)) << (4 * a.n);
      ++a.n;
    }
  return a;
}

// Whether the point k + d is kend or past it, without a sign: a grid may end
// within a workgroup's points of 2^31.
__host__ __device__ inline bool point_past(int32_t k, int32_t d, int32_t kend) {
  return (uint32_t)k + (uint32_t)d >= (uint32_t)kend;
}

// The grid values, weights and sidereal angles of NQ points k, k + stride, ...
// of an event, from vrec[NQ][3] (GridWalk; NULL: evaluated directly).  Points
// at or past kend stand for the point kend - 1 (whose grid values the caller
// gives) and get zero weight; inner says that no point is an end of the grid
// or past kend.
template <int NQ, bool MIXED, bool ROT, bool ECC, bool EXPL>
__host__ __device__ inline void point_block(const EventC& ec, int32_t k, int32_t stride, int32_t kend, bool inner,
                                            const double (*vrec)[3], Point (&q)[NQ]) {
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const bool past = !inner && point_past(k, i * stride, kend);
    int32_t ki = (int32_t)((uint32_t)k + (uint32_t)(i * stride));
    if (!inner) {
      keep_branch();
      if (past) ki = kend - 1;
    }
    point_setup<EXPL, ECC>(ec, ki, false, ROT, q[i], MIXED ? kPsdF32 : kPsdF64, vrec ? vrec[i] : nullptr, inner);
    if (!inner) {
      keep_branch();
      if (past) q[i].rw = q[i].w4A2 = 0.0;
    }
  }
}

// The grid values of a lane's next NQ points (k and on, the walk's stride
// apart) from its walk, those of the point k1 - 1 where a point is past it.
template <int NQ>
__host__ __device__ inline void walk_points(const EventC& ec, GridWalk& gw, int32_t k, int32_t stride, int32_t k1,
                                            bool inner, double (&vv)[NQ][3]) {
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
#pragma unroll
    for (int c = 0; c < 3; ++c) vv[i][c] = gw.val[c];
    gw.step();
  }
  if (!inner) {
    keep_branch();
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      if (point_past(k, i * stride, k1)) grid_values(ec, k1 - 1, vv[i]);
  }
}

// The sums over the network's interferometers at the points of point_block
// (q, net).  This part needs the points' grid values and sidereal angle only;
// the phase and angle derivatives follow it (finish_point), so that they and
// the sums are not held at the same time as the sites' values.
template <int NQ, int NPI, bool ROT, bool MIXED, bool EXPL, bool TAB>
__host__ __device__ inline void network_sums(const EventC& ec, const SiteC* sc, const ActiveSites& act, int32_t k,
                                             int32_t stride, int32_t kend, bool inner, const double (*vrec)[3],
                                             Point (&q)[NQ], NetSums (&net)[NQ]) {
  const AmpFactors am = amp_factors(ec);
  point_block<NQ, MIXED, ROT, PhaseOnly<NPI>::ecc, EXPL>(ec, k, stride, kend, inner, vrec, q);
#pragma unroll
  for (int i = 0; i < NQ; ++i) net[i] = NetSums{};
  if (act.n == 0) return;
  // one loop without a way round its body: a site skipped inside the loop
  // would have the compiler copy every sum where the two ways meet
  uint32_t list = act.list;
  int left = act.n;
  constexpr bool AHEAD = NQ > 1 && !PhaseOnly<NPI>::ecc;
  SiteHead hd{};
  if (AHEAD) hd = site_head(sc[list & 7u]);
  do {
    const uint32_t l = list;
    if (!AHEAD || left > 1) list >>= 4;
    site_sums<NQ, MIXED, TAB, AHEAD>(am, q, sc[l & 7u], 1 + (int)(l >> 3 & 1u), hd, sc[list & 7u], net);
  } while (--left > 0);
}

// The rest of a point whose network sums are n: its derivatives, its share of
// G[kGramAcc], U[8], W (accumulate_sums) and its phase-only coefficients
// c[NPI] = (-1, dPsi/dchi1, dPsi/dchi2[, dPsi/dLambda1, dPsi/dLambda2]
// [, dPsi/de0]).
template <int NPI, bool ROT>
__host__ __device__ inline void finish_point(const EventC& ec, Point& q, const NetSums& n, double* G, double* U,
                                             double& W, double* cph) {
  reread(q.v, q.iv);
  point_derivatives<PhaseOnly<NPI>::ecc>(ec, ROT, q);
  accumulate_sums<ROT>(ec, q, n, G, U, W);
  phase_only_coefficients<NPI>(ec, q, cph);
}

// One grid point k of an event as a whole.
template <int NPI, bool ROT, bool MIXED = false, bool EXPL = false, bool TAB = true>
__host__ __device__ inline void accumulate_point(const EventC& ec, const SiteC* sc, const ActiveSites& act,
                                                 int32_t k, double* G, double* U, double& W,
                                                 double* cph, const double (*vrec)[3] = nullptr) {
  Point q[1];
  NetSums n[1];
  network_sums<1, NPI, ROT, MIXED, EXPL, TAB>(ec, sc, act, k, 0, k + 1, false, vrec, q, n);
  finish_point<NPI, ROT>(ec, q[0], n[0], G, U, W, cph);
}
template <int NPI, bool ROT, bool MIXED = false, bool EXPL = false, bool TAB = true>
__host__ __device__ inline void accumulate_point(const EventC& ec, const SiteC* sc, int n_site,
                                                 int32_t k, double* G, double* U, double& W,
                                                 double* cph) {
  accumulate_point<NPI, ROT, MIXED, EXPL, TAB>(ec, sc, active_sites(sc, n_site), k, G, U, W, cph);
}

// The 8x8 upper-triangle block of (Mc, eta, dL, theta, phi, iota, psi, tc)
// (row-major, 36 values) from the accumulator of accumulate_point.
__host__ __device__ inline void gram_finish(const EventC& ec, const double* G, double* F) {
  const AmpFactors am = amp_factors(ec);
  auto at = [](int r, int c) { return r <= c ? 8 * r - (r * (r - 1)) / 2 + (c - r)
                                             : 8 * c - (c * (c - 1)) / 2 + (r - c); };
  const double cp = am.cplus, cx = am.ccross, a = am.dlnA;
  const double spp = G[kGSpp], spx = G[kGSpx], sxx = G[kGSxx];
  const double si2 = (1.0 - cx) * (1.0 + cx);                     // c+^2 - cx^2 = sin^4(iota)/4
  const double W = fma(cp * cp, spp, cx * cx * sxx);
  const double qi = fma(cp * am.dcp, spp, cx * am.dcx * sxx);     // Re(Q D_iota^*)
  const double qp = 0.5 * si2 * si2 * spx;                        // Re(Q D_psi^*)
  // Re(X Z^*) and Re(X Y^*) for X = Q, D_iota, D_psi
  const double qz = fma(cp, G[kGPzr], cx * G[kGXzi]), qy = fma(cp, G[kGPyr], cx * G[kGXyi]);
  const double iz = fma(am.dcp, G[kGPzr], am.dcx * G[kGXzi]), iy = fma(am.dcp, G[kGPyr], am.dcx * G[kGXyi]);
  const double pz = 2.0 * fma(cp, G[kGXzr], -cx * G[kGPzi]), py = 2.0 * fma(cp, G[kGXyr], -cx * G[kGPyi]);
  // Mc and eta
  F[at(0, 0)] = fma(a, fma(a, W, 2.0 * G[kGMd]), G[kGMM]);
  F[at(0, 1)] = fma(a, G[kGEd], G[kGME]);
  F[at(1, 1)] = G[kGEE];
  F[at(0, 3)] = fma(a, qy, G[kGMY]);
  F[at(1, 3)] = G[kGEY];
  const double mz = fma(a, qz, G[kGMZ]);
  F[at(0, 4)] = -mz;
  F[at(1, 4)] = -G[kGEZ];
  F[at(0, 7)] = fma(kOmegaE, mz, G[kGMt]);
  F[at(1, 7)] = fma(kOmegaE, G[kGEZ], G[kGEt]);
  // theta, phi, tc
  F[at(3, 3)] = G[kGYY];
  F[at(3, 4)] = -G[kGZY];
  F[at(3, 7)] = fma(kOmegaE, G[kGZY], G[kGtY]);
  F[at(4, 4)] = G[kGZZ];
  F[at(4, 7)] = -fma(kOmegaE, G[kGZZ], G[kGtZ]);
  F[at(7, 7)] = fma(kOmegaE, fma(kOmegaE, G[kGZZ], 2.0 * G[kGtZ]), G[kGtt]);
  // dL
  F[at(0, 2)] = -am.idL * fma(a, W, G[kGMd]);
  F[at(1, 2)] = -am.idL * G[kGEd];
  F[at(2, 2)] = am.idL * am.idL * W;
  F[at(2, 3)] = -am.idL * qy;
  F[at(2, 4)] = am.idL * qz;
  F[at(2, 5)] = -am.idL * qi;
  F[at(2, 6)] = -am.idL * qp;
  F[at(2, 7)] = -am.idL * (kOmegaE * qz);
  // iota
  F[at(0, 5)] = fma(a, qi, G[kGMi]);
  F[at(1, 5)] = G[kGEi];
  F[at(3, 5)] = iy;
  F[at(4, 5)] = -iz;
  F[at(5, 5)] = fma(am.dcp * am.dcp, spp, am.dcx * am.dcx * sxx);
  F[at(5, 6)] = 2.0 * fma(cp, am.dcp, -cx * am.dcx) * spx;
  F[at(5, 7)] = fma(kOmegaE, iz, G[kGTI]);
  // psi
  F[at(0, 6)] = fma(a, qp, G[kGMp]);
  F[at(1, 6)] = G[kGEp];
  F[at(3, 6)] = py;
  F[at(4, 6)] = -pz;
  F[at(6, 6)] = 4.0 * fma(cp * cp, sxx, cx * cx * spp);
  F[at(6, 7)] = fma(kOmegaE, pz, G[kGTP]);
}

// The Phic column from the accumulator: -sum U_b of the rows Mc, eta, theta,
// phi, iota, psi, tc (the dL row is zero), then sum W (= Gamma_{Phic,Phic}).
__host__ __device__ inline void gram_phic(const EventC& ec, const double* G, double xc[8]) {
  const AmpFactors am = amp_factors(ec);
  const double iqz = fma(am.cplus, G[kGPzi], -am.ccross * G[kGXzr]);
  xc[0] = -G[kGMu];
  xc[1] = -G[kGEu];
  xc[2] = fma(am.ccross, G[kGXyr], -am.cplus * G[kGPyi]);
  xc[3] = iqz;
  xc[4] = -(am.cplus * am.dcx - am.ccross * am.dcp) * G[kGSpx];
  xc[5] = 2.0 * am.cplus * am.ccross * (G[kGSpp] + G[kGSxx]);
  xc[6] = -fma(kOmegaE, iqz, G[kGTW]);
  xc[7] = fma(am.cplus * am.cplus, G[kGSpp], am.ccross * am.ccross * G[kGSxx]);
}

// Plain accumulation of the phase-only blocks of one point into
// xy[(b*NPI + i)*xs] (b < 8) and then the upper triangle of W c_i c_j.
__host__ __device__ inline void add_phase_blocks(int NPI, const double* U, double W, const double* cph,
                                                 double* xy, int xs) {
  for (int b = 0; b < 8; ++b)
    for (int i = 0; i < NPI; ++i) xy[(b * NPI + i) * xs] = fma(U[b], cph[i], xy[(b * NPI + i) * xs]);
  int y = 8 * NPI;
  for (int i = 0; i < NPI; ++i) {
    const double wc = W * cph[i];
    for (int j = i; j < NPI; ++j) {
      xy[y * xs] = fma(wc, cph[j], xy[y * xs]);
      ++y;
    }
  }
}

// Position (r, c) in the P x P Fisher matrix of accumulator slot t, with
// slots ordered as: 36 entries of the 8x8 upper block (row-major), then the
// 8 x NPI block, then the NPI x NPI upper block.
__host__ __device__ inline void slot_position(int t, int NPI, int& r, int& c) {
  if (t < 36) {
    int i = t;
    r = 0;
    while (i >= 8 - r) { i -= 8 - r; ++r; }
    c = r + i;
  } else if (t < 36 + 8 * NPI) {
    const int i = t - 36;
    r = i / NPI;
    c = 8 + i % NPI;
  } else {
    int i = t - 36 - 8 * NPI;
    r = 0;
    while (i >= NPI - r) { i -= NPI - r; ++r; }
    c = 8 + r + i;
    r = 8 + r;
  }
}

}  // namespace gwf
