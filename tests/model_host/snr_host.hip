// snr_host.hip -- TEST ONLY: the SNR kernels' per-lane sums (snr_lane of
// gwf_snr_body.hpp) run on the host.
#include "../../paper_2207_06910_amd/csrc/gwf_snr_body.hpp"

using namespace gwf;

// SNR^2 sums [3 n_site] of the points lane tid takes of an event's grid from point
// k0 on, walked (direct = 0), or of the same points one by one, each evaluated
// directly; sites[s][7] = lat, lon, gamma, zeta, shape, S0, f0; tab_n > 0: every
// site has the sampled curve (tab_f, tab_S) of that kind, scaled by its S0.
extern "C" int snr_lane_host(const double* par, double fmin, double fmax, int32_t n, int n_site, const double* sites,
                             int tid, int direct, int32_t k0, int64_t tab_n, const double* tab_f, const double* tab_S,
                             int kind, double* out) {
  EventC ec;
  event_setup(par, fmin, fmax, n, kFlagRot, ec);
  if (ec.status) return ec.status;
  SiteC sc[kMaxSites];
  for (int s = 0; s < n_site; ++s) {
    const double* r = sites + 7 * s;
    SiteDesc sd{r[0], r[1], r[2], r[3], r[5], r[6], (int32_t)r[4], 0};
    if (tab_n > 0) {
      sd.psd_kind = kind;
      sd.tab_n = tab_n;
      sd.tab_f = tab_f;
      sd.tab_S = tab_S;
    }
    site_setup(par, sd, ec, sc[s], kArmsPlain);
  }
  double acc[kSnrSlots] = {};
  if (!direct) {
    snr_lane<true, false, true>(ec, sc, n_site, k0, ec.n, tid, acc);
  } else {
    for (int64_t k = (int64_t)k0 + tid; k < ec.n; k += kBlock)
      snr_lane<true, false, true>(ec, sc, n_site, (int)k, (int)k + 1, 0, acc);
  }
  for (int i = 0; i < 3 * n_site; ++i) out[i] = acc[i];
  return 0;
}
