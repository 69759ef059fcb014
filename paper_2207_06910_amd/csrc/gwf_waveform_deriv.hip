// gwf_waveform_deriv.hip -- the strain's derivatives with respect to the
// Fisher parameters at every interferometer and grid point (the d h / d theta
// arrays the paper's Fisher matrices are built from, sec. 3.2), phase in
// cycles as for the strain (gwf_waveform.hip).
#include "gwf_waveform.hpp"

namespace gwf {

namespace {

// The strain's derivatives with respect to the P parameters, in the rows and
// units of the Fisher matrix (whose entries are 4 Re sum w d_a h d_b h^* / S_n):
//   d_a h_i = A exp(2 pi i cyc_i) D_a,i,
// D the phase-free derivative vector of the Fisher kernels for (Mc, eta, dL,
// theta, phi, iota, psi, tc) and i Q c_a for the phase-only parameters
// (Phic, chi1z, chi2z[, Lambda1, Lambda2][, e0]); the phase in cycles exactly as
// for the strain.  D is a combination of Q, iQ, Z and Y (NetSums), so a point
// turns those three complex numbers by the phase and the rows follow by real
// coefficients.  One or several workgroups per event (wave_part), lanes over
// grid points; row (a, i) of dh holds parameter a at interferometer i,
// consecutive lanes on consecutive complex values.  FP64 only.
// What bounds it: the output's writes, 4.9 TB/s on 3.0 GB of 300 neutron-star
// pairs (616 us; every arm's rows from its own derivative vector, one
// workgroup per event: 960 us).
// One arm at one point: its patterns, and Q, Z and Y turned by A exp(i Psi).
struct Response {
  double Fp, Fx, qr, qi, zr, zi, yr, yi;
};

__device__ inline void arm_response(const AmpFactors& am, const double (*c)[5], const SiteTrigR& tr, double u,
                                    double w, double ca, double sa, Response& r) {
  r.Fp = trig_val_r(c[0], tr);
  r.Fx = trig_val_r(c[1], tr);
  const double Qr = am.cplus * r.Fp, Qi = am.ccross * r.Fx;
  const double Zr = fma(am.cplus, trig_dH_r(c[0], tr), -u * Qi), Zi = fma(am.ccross, trig_dH_r(c[1], tr), u * Qr);
  const double Yr = fma(am.cplus, trig_val_r(c[2], tr), -w * Qi), Yi = fma(am.ccross, trig_val_r(c[3], tr), w * Qr);
  r.qr = fma(Qr, ca, -Qi * sa); r.qi = fma(Qr, sa, Qi * ca);
  r.zr = fma(Zr, ca, -Zi * sa); r.zi = fma(Zr, sa, Zi * ca);
  r.yr = fma(Yr, ca, -Yi * sa); r.yi = fma(Yr, sa, Yi * ca);
}

// The P rows of one arm at one point (see NetSums), those outside the event's
// set pm as zeros.
template <int NPI>
__device__ inline void write_rows(const AmpFactors& am, const Point& q, const double* cph, double ca, double sa,
                                  const Response& r, uint32_t pm, int64_t prow, double2* o) {
  auto put = [&](int row, double x, double y) {
    const bool in = (pm >> row) & 1u;
    o[row * prow] = make_double2(in ? x : 0.0, in ? y : 0.0);
  };
  put(0, fma(am.dlnA, r.qr, fma(q.gMc, r.zr, -q.pMc * r.qi)), fma(am.dlnA, r.qi, fma(q.gMc, r.zi, q.pMc * r.qr)));
  put(1, fma(q.gEta, r.zr, -q.pEta * r.qi), fma(q.gEta, r.zi, q.pEta * r.qr));
  put(2, -am.idL * r.qr, -am.idL * r.qi);
  put(3, r.yr, r.yi);
  put(4, -r.zr, -r.zi);
  const double ir = am.dcp * r.Fp, ii = am.dcx * r.Fx;
  put(5, fma(ir, ca, -ii * sa), fma(ir, sa, ii * ca));
  const double pr = 2.0 * am.cplus * r.Fx, pi = -2.0 * am.ccross * r.Fp;
  put(6, fma(pr, ca, -pi * sa), fma(pr, sa, pi * ca));
  put(7, fma(kOmegaE, r.zr, -q.tf * r.qi), fma(kOmegaE, r.zi, q.tf * r.qr));
#pragma unroll
  for (int i = 0; i < NPI; ++i) put(8 + i, -r.qi * cph[i], r.qr * cph[i]);
}

template <bool ROT, int NPI, bool EXPL>
__global__ __launch_bounds__(kWBlock) void waveform_deriv_kernel(WaveformArgs a) {
  using PO = PhaseOnly<NPI>;
  constexpr bool TIDAL = PO::tidal;
  constexpr uint32_t flags = (TIDAL ? kFlagTidal : 0u) | (ROT ? kFlagRot : 0u) | (PO::ecc ? kFlagEcc : 0u);
  __shared__ EventC ec;
  __shared__ SiteC sc[kMaxSites];
  __shared__ int32_t ok;
  const int64_t e = a.base + blockIdx.x;
  const int tid = threadIdx.x;
  const int n_site = a.net.n_site;
  int32_t k0 = 0, k1 = 0;
  const bool some = wave_setup(a, e, TIDAL, flags, ec, ok, k0, k1, [&](int s, const double* p) {
    SiteDesc sd = a.net.site[s];
    sd.psd_kind = 0;                     // the noise curve plays no part, nor does pi M
    site_setup(p, sd, 1.0, sc[s], kArmsPlain);
  });
  if (!some) return;

  const uint32_t pm = event_rows(a.par_mask, e);
  const double tc = a.tc_s ? a.tc_s[e] : 0.0;
  const double amp0 = exp(ec.lnA);
  const AmpFactors am = amp_factors(ec);
  double2* __restrict__ out = reinterpret_cast<double2*>(a.dh) + a.offsets[e];
  const int64_t row = a.total;
  const int64_t prow = (int64_t)a.net.n_ifo * row;     // one parameter's block of rows
  // (counted in 32 bits without a sign: a grid may end within a run of 2^31)
  for (uint32_t u = tid, end = (uint32_t)k1 - (uint32_t)k0; u < end; u += kWBlock) {
    const int k = (int)((uint32_t)k0 + u);
    if (k < 0) continue;
    // the event and site constants are re-read from LDS (uniform broadcast
    // reads) rather than held in registers across iterations
    asm volatile("" ::: "memory");
    Point q;
    point_setup<EXPL, PO::ecc>(ec, k, true, ROT, q, kPsdNone);
    VPow pw;
    vpow(q.v, q.L, pw);
    const double iv = q.iv, iv2 = iv * iv, iv5 = iv2 * iv2 * iv;
    const double amp = amp0 * iv2 * iv * sqrt(iv);
    double pnc = eval_phase(ec.cyc, pw, iv5);
    if (PO::ecc) pnc = fma(ec.ecc_cyc, q.ecv, pnc);
    const double pn = frac_center(pnc);
    const double ftr = fma(q.f, tc, -rint(q.f * tc));
    const double cyc = frac_center(pn + ftr + ec.cyc0);
    double cph[NPI];
    phase_only_coefficients<NPI>(ec, q, cph);
    double2* o = out + k;
    for (int s = 0; s < n_site; ++s) {
      asm volatile("" ::: "memory");
      const SiteC& st = sc[s];
      const double cH = q.cth * st.cdl - q.sth * st.sdl;
      const double sH = q.sth * st.cdl + q.cth * st.sdl;
      double sn, cs;
      sincos_cycles<false>(frac_center(fma(q.f, fma(st.k1, cH, st.k0), cyc)), &sn, &cs);
      const double ca = amp * cs, sa = amp * sn;
      SiteTrigR tr;                      // the patterns' basis, unweighted
      trig_basis(cH, sH, 1.0, tr);
      const double u = q.tf * (-st.k1 * sH), w = q.tf * fma(st.k1t, cH, st.k0t);
      Response a0, a1;
      arm_response(am, st.jk[0], tr, u, w, ca, sa, a0);
      write_rows<NPI>(am, q, cph, ca, sa, a0, pm, prow, o);
      o += row;
      if (st.n_arm == 3) {               // closed triangle: third arm = -(first + second)
        arm_response(am, st.jk[1], tr, u, w, ca, sa, a1);
        write_rows<NPI>(am, q, cph, ca, sa, a1, pm, prow, o);
        o += row;
        a0.Fp = -(a0.Fp + a1.Fp); a0.Fx = -(a0.Fx + a1.Fx);
        a0.qr = -(a0.qr + a1.qr); a0.qi = -(a0.qi + a1.qi);
        a0.zr = -(a0.zr + a1.zr); a0.zi = -(a0.zi + a1.zi);
        a0.yr = -(a0.yr + a1.yr); a0.yi = -(a0.yi + a1.yi);
        write_rows<NPI>(am, q, cph, ca, sa, a0, pm, prow, o);
        o += row;
      }
    }
  }
}

}  // namespace

template <int NPI, bool EXPL>
void launch_deriv_n(const WaveformArgs& a, bool rot, dim3 grid, dim3 block, hipStream_t stream) {
  if (rot) hipLaunchKernelGGL((waveform_deriv_kernel<true, NPI, EXPL>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((waveform_deriv_kernel<false, NPI, EXPL>), grid, block, 0, stream, a);
}

template <bool EXPL>
void launch_deriv_t(const WaveformArgs& a, int npi, bool rot, dim3 grid, dim3 block, hipStream_t stream) {
  switch (npi) {
    case 6: launch_deriv_n<6, EXPL>(a, rot, grid, block, stream); break;
    case 5: launch_deriv_n<5, EXPL>(a, rot, grid, block, stream); break;
    case 4: launch_deriv_n<4, EXPL>(a, rot, grid, block, stream); break;
    default: launch_deriv_n<3, EXPL>(a, rot, grid, block, stream);
  }
}

hipError_t launch_waveform_deriv(const WaveformArgs& args, int npi, bool rot, hipStream_t stream) {
  WaveformArgs a0 = args;
  a0.share = a0.n < 512 ? wave_share(a0.n, 2048) : 1;
  a0.longest = 4;
  return launch_slices(a0, a0.n, 1, kWBlock, [&](const WaveformArgs& a, dim3 grid, dim3 block) {
    grid.y = a.n < 512 ? (unsigned)a.share : (unsigned)((8192 + a.n - 1) / a.n);
    if (a.gf) launch_deriv_t<true>(a, npi, rot, grid, block, stream);
    else launch_deriv_t<false>(a, npi, rot, grid, block, stream);
  });
}

}  // namespace gwf
