// gwf_fisher.hip -- SNR and Fisher-matrix kernels (plain FP64 form).
//
// One workgroup of 256 lanes per event.  The workgroup first builds the
// event's constants (PN-series coefficients, grid, amplitude) and each
// site's constants (pattern polynomials, delay and PSD factors) in LDS, three
// parts of the event and the sites side by side; every lane then walks a stretch
// of the event's frequency grid with stride 256, sums the products of all
// interferometers' response vectors at its frequency in registers (NetSums) and
// adds the point's share of the noise-weighted Gram matrix; a fixed-order
// wavefront + LDS reduction produces the stretch's matrix, and the stretches
// are added in order.  Nothing is atomically added, so results are bitwise
// reproducible, and the split form (gwf_split.hip), a workgroup per stretch,
// gives the same bits.
//
// The accumulation itself (gwf_fisher_body.hpp) is shared with the batched
// work-item form (gwf_batched.hip).
//
// Gram structure exploited (exact algebra, no approximation): the derivative
// vectors with respect to Phic, chi1, chi2, Lambda1, Lambda2 are i Q c_a(f)
// with the same real c_a(f) for every interferometer, so their blocks follow
// from per-frequency network sums W = sum_i w_i |Q_i|^2 and
// U_b = sum_i w_i Re(i Q_i D_b,i^*):
//   Gamma_ab += W c_a c_b   (a, b phase-only),   Gamma_ba += U_b c_a,
// and the 8x8 block of (Mc, eta, dL, theta, phi, iota, psi, tc) follows from the
// same point's 14 sums by coefficients that no interferometer changes
// (accumulate_sums).
#include "gwf_fisher_body.hpp"
#include "gwf_snr_body.hpp"

namespace gwf {

// Two workgroups per compute unit (256 registers; 43 KB of LDS each with
// tides: 37 KB of FisherLds, the event's 1.2 KB of constants and 4.9 KB for
// eight sites) hide the latency of the LDS constant reads and of the
// transcendental sequences.
static_assert(64 + kMaxSites <= 128, "site set-up lanes in the second wavefront");

template <int NPI_, bool ROT, bool EXPL, bool TAB>
__global__ __launch_bounds__(kBlock, 2) void fisher_kernel(FisherArgs a) {
  using Dm = FisherDims<NPI_>;
  using PO = PhaseOnly<NPI_>;
  constexpr int P = Dm::P, NPI = Dm::NPI, NACC = Dm::NACC;
  constexpr uint32_t flags = (PO::tidal ? kFlagTidal : 0u) | (ROT ? kFlagRot : 0u) | (PO::ecc ? kFlagEcc : 0u);

  __shared__ EventC ec;
  __shared__ SiteC sc[kMaxSites];
  __shared__ FisherLds<NPI, 1> L;
  __shared__ int32_t skip, bad;

  const int64_t e = a.base + blockIdx.x;
  const int tid = threadIdx.x;
  const int n_site = a.net.n_site;
  double p[kNparIn];
  load_par(a.par, a.ld, e, PO::tidal, PO::ecc ? a.ecc : nullptr, a.fref, p);
  // the three parts of the event's constants and the sites' on a wavefront each,
  // at the same time (a site needs only the parameters and pi M)
  if (tid == 0) {
    event_setup_grid(p, a.fmin, a.fmax, a.npts, a.goff, a.gf, e, flags, ec, kSetupGrid);
    int32_t sk = ec.status;
    if (!sk && a.snr_pre && !(a.snr_pre[e] > a.snr_th)) sk = kEvSkipped;
    skip = sk;
    bad = 0;
  } else if (tid >= 64 && tid < 64 + n_site) {
    const int s = tid - 64;
    site_setup(p, a.net.site[s], kPi * total_mass_s(p), sc[s],
               select_ifo(site_arms_on(a.active, a.ld, e, a.net, s), a.net, s, a.ifo_sel));
  } else if (tid == 128) {
    event_setup_grid(p, a.fmin, a.fmax, a.npts, a.goff, a.gf, e, flags, ec, kSetupPhase);
  } else if (tid == 192) {
    event_setup_grid(p, a.fmin, a.fmax, a.npts, a.goff, a.gf, e, flags, ec, kSetupAngle);
  }
  __syncthreads();
  if (skip) {
    for (int i = tid; i < P * P; i += kBlock) a.fisher[(int64_t)i * a.n + e] = 0.0;
    if (tid == 0) {
      if (!a.snr_pre && a.snr) a.snr[e] = 0.0;
      a.status[e] = skip;
    }
    return;
  }

  double t = 0.0;
  // an explicit grid has one form only
  const int len = EXPL ? ec.n : stretch_length(ec.n, a.ifo_sel > 0 ? kIfoStretch : kFisherStretch);
  if (ec.n <= len) {
    double x = 0.0;
    fisher_sums<NPI, 1, ROT, false, EXPL, TAB>(ec, sc, n_site, 0, ec.n, L, &x);
    t += x;
  } else if (!EXPL) {                    // on its own: a loop around it costs short grids 2 %
    for (int k0 = 0;; k0 += len) {
      double x = 0.0;
      fisher_sums<NPI, 1, ROT, false, EXPL, TAB>(ec, sc, n_site, k0, k0 + min(ec.n - k0, len), L, &x);
      t += x;
      if (ec.n - k0 <= len) break;
      __syncthreads();                   // the next stretch's sums take the same LDS
    }
  }
  if (tid < NACC) {
    int r, c;
    slot_position(tid, NPI, r, c);
    if (r == 8 && c == 8 && a.snr) a.snr[e] = sqrt(t);     // Gamma_{Phic,Phic} = SNR^2
    const double v = rows_in(event_rows(a.par_mask, e), r, c) ? t : 0.0;
    if (!isfinite(v)) atomicOr(&bad, 1);
    a.fisher[((int64_t)r * P + c) * a.n + e] = v;
    a.fisher[((int64_t)c * P + r) * a.n + e] = v;
  }
  __syncthreads();
  // one launch per interferometer (ifo_sel > 1 after the first) adds its bit
  if (tid == 0) {
    const int32_t f = bad ? kEvNonFinite : 0;
    a.status[e] = a.ifo_sel > 1 ? (a.status[e] | f) : f;
  }
}

// SNR only, with the SNR of every interferometer.  Same grid, weights and
// patterns as the Fisher kernel; no derivatives.
template <bool ROT, bool EXPL>
__global__ __launch_bounds__(kBlock) void snr_kernel(SnrArgs a) {
  constexpr uint32_t flags = ROT ? kFlagRot : 0u;
  __shared__ EventC ec;
  __shared__ SiteC sc[kMaxSites];
  __shared__ double red[kWaves][kMaxIfo], ifo[kMaxIfo];
  const int64_t e = a.base + blockIdx.x;
  const int tid = threadIdx.x;
  const int n_site = a.net.n_site, n_ifo = a.net.n_ifo;
  double p[kNparIn];
  load_par(a.par, a.ld, e, a.tidal, nullptr, nullptr, p);
  // the event's grid and angle constants and the sites', on a wavefront each at
  // once (no phase series here)
  const uint32_t ef = flags | (a.tidal ? kFlagTidal : 0u);
  if (tid == 0)
    event_setup_grid(p, a.fmin, a.fmax, a.npts, a.goff, a.gf, e, ef, ec, kSetupGrid);
  else if (tid == 192)
    event_setup_grid(p, a.fmin, a.fmax, a.npts, a.goff, a.gf, e, ef, ec, kSetupAngle);
  else if (tid >= 64 && tid < 64 + n_site)
    site_setup(p, a.net.site[tid - 64], kPi * total_mass_s(p), sc[tid - 64], kArmsPlain);
  __syncthreads();
  if (ec.status) {
    if (tid == 0) {
      a.snr[e] = 0.0;
      if (a.status) a.status[e] = ec.status;
    }
    if (a.snr_ifo)
      for (int i = tid; i < n_ifo; i += kBlock) a.snr_ifo[(int64_t)i * a.n + e] = 0.0;
    return;
  }
  const uint32_t shapes = site_shapes(a.net);
  double t = 0.0;
  const int len = EXPL ? ec.n : stretch_length(ec.n, kSnrStretch);
  for (int k0 = 0;; k0 += len) {
    double acc[kSnrSlots], x = 0.0;
#pragma unroll
    for (int i = 0; i < kSnrSlots; ++i) acc[i] = 0.0;
    snr_sums<ROT, EXPL, true>(ec, sc, n_site, k0, k0 + min(ec.n - k0, len), acc);
    snr_reduce(acc, n_site, n_ifo, shapes, red, &x);
    t += x;
    if (EXPL || ec.n - k0 <= len) break;
    __syncthreads();                     // the next stretch's sums take the same LDS
  }
  if (tid < n_ifo) {
    if (a.active && !a.active[(int64_t)tid * a.ld + e]) t = 0.0;   // off for this event
    if (a.snr_ifo) a.snr_ifo[(int64_t)tid * a.n + e] = sqrt(t);
    ifo[tid] = t;
  }
  __syncthreads();
  if (tid == 0) {
    double tot = 0.0;
    for (int i = 0; i < n_ifo; ++i) tot += ifo[i];
    a.snr[e] = sqrt(tot);
    if (a.status) a.status[e] = isfinite(tot) ? 0 : kEvNonFinite;
  }
}

template <int NPI, bool EXPL>
void launch_fisher_n(const FisherArgs& a, bool rot, dim3 grid, dim3 block, hipStream_t stream) {
  const bool tab = net_has_tables(a.net);
  if (rot && tab) hipLaunchKernelGGL((fisher_kernel<NPI, true, EXPL, true>), grid, block, 0, stream, a);
  else if (rot) hipLaunchKernelGGL((fisher_kernel<NPI, true, EXPL, false>), grid, block, 0, stream, a);
  else if (tab) hipLaunchKernelGGL((fisher_kernel<NPI, false, EXPL, true>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((fisher_kernel<NPI, false, EXPL, false>), grid, block, 0, stream, a);
}

template <bool EXPL>
void launch_fisher_t(const FisherArgs& a, int npi, bool rot, dim3 grid, dim3 block, hipStream_t stream) {
  switch (npi) {
    case 6: launch_fisher_n<6, EXPL>(a, rot, grid, block, stream); break;
    case 5: launch_fisher_n<5, EXPL>(a, rot, grid, block, stream); break;
    case 4: launch_fisher_n<4, EXPL>(a, rot, grid, block, stream); break;
    default: launch_fisher_n<3, EXPL>(a, rot, grid, block, stream);
  }
}

// An explicit grid (a.gf set) selects the instantiations that read it.
hipError_t launch_fisher(const FisherArgs& a0, int npi, bool rot, hipStream_t stream) {
  return launch_slices(a0, a0.n, 1, kBlock, [&](const FisherArgs& a, dim3 grid, dim3 block) {
    if (a.gf) launch_fisher_t<true>(a, npi, rot, grid, block, stream);
    else launch_fisher_t<false>(a, npi, rot, grid, block, stream);
  });
}

hipError_t launch_snr(const SnrArgs& a0, bool rot, hipStream_t stream) {
  return launch_slices(a0, a0.n, 1, kBlock, [&](const SnrArgs& a, dim3 grid, dim3 block) {
    if (a.gf) {
      if (rot) hipLaunchKernelGGL((snr_kernel<true, true>), grid, block, 0, stream, a);
      else hipLaunchKernelGGL((snr_kernel<false, true>), grid, block, 0, stream, a);
    } else {
      if (rot) hipLaunchKernelGGL((snr_kernel<true, false>), grid, block, 0, stream, a);
      else hipLaunchKernelGGL((snr_kernel<false, false>), grid, block, 0, stream, a);
    }
  });
}

}  // namespace gwf
