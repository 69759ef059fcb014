// gwf_split.hip -- gwf_*_split: the plain calls (SNR, Fisher, per-interferometer
// Fisher matrices) with each event's grid split over several workgroups, in a
// workspace of the caller's.
//
// The one-workgroup-per-event kernels need no memory of their own, but one
// event's grid is then one workgroup's serial loop, the constants are formed
// in every workgroup and read from LDS, and a ragged catalogue ends with a few
// long events on an idle chip.  Here the set-up kernel of the batched form
// writes every event's constants once, the work-item kernel (gwf_batched.hip)
// takes (event, part, matrix) from its workgroup's number -- no item table,
// so nothing is read back or built -- with scalar loads of the constants, and
// the parts' sums are combined in order.  More events than the workspace holds
// are taken in slices, one after the other on the stream.  A part is a stretch of the grid that
// the one-workgroup form sums on its own as well (stretch_length), so both
// forms give the same bits.  Measured before there was a split form and now: one
// neutron-star pair 165 and 41 us, 1000 pairs 512 and 290 us, 1501 events with
// their SNR threshold 1043 and 487 us, 500 pairs' matrices of five
// interferometers 945 and 468 us, SNR of 3000 pairs 578 and 237 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "../../include/gwf.h"
#include "gwf_api_internal.hpp"
#include "gwf_batched.hpp"

using namespace gwf;

static_assert(kFisherStretch == GWF_FISHER_STRETCH && kSnrStretch == GWF_SNR_STRETCH && kIfoStretch == GWF_IFO_STRETCH &&
              kMaxStretches == GWF_SPLIT_PARTS_MAX, "stretches as declared");

namespace {

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// The parts of the workspace, each 256-byte aligned.
struct Layout {
  size_t sic = 0, partial = 0, total = 0;
  size_t per_event = 0;      // bytes of one event in the three parts together
  int32_t sets = kSetsSites, n_set = 0, set0 = 0, n_mat = 0;
  bool snr = false;
};
constexpr size_t kAlignSlack = 3 * 256;

// what: the SNR alone (0), Fisher matrices (1), after an SNR pass (2), one per
// interferometer (3)
enum { kWhatSnr = 0, kWhatFisher = 1, kWhatSnrFisher = 2, kWhatIfos = 3 };

Layout layout(int64_t n, const NetDesc& nd, uint32_t flags, int what, int32_t parts) {
  Layout l;
  l.snr = what == kWhatSnr || what == kWhatSnrFisher;
  l.n_mat = what == kWhatSnr ? 0 : what == kWhatIfos ? nd.n_ifo : 1;
  l.sets = what == kWhatSnr ? kSetsArms : what == kWhatFisher ? kSetsSites : what == kWhatIfos ? kSetsIfos : kSetsSitesArms;
  l.n_set = what == kWhatIfos ? nd.n_ifo : what == kWhatSnrFisher ? 2 * nd.n_site : nd.n_site;
  l.set0 = what == kWhatSnrFisher ? nd.n_site : 0;
  l.sic = align256((size_t)n * sizeof(EventC));
  l.partial = l.sic + align256((size_t)n * l.n_set * sizeof(SiteC));
  // the SNR pass and the matrices use the partial sums one after the other
  const size_t per = std::max<size_t>(l.snr ? nd.n_ifo : 0, (size_t)l.n_mat * fisher_nacc(api_npi(flags)));
  l.total = l.partial + align256((size_t)n * parts * per * sizeof(double));
  l.per_event = sizeof(EventC) + l.n_set * sizeof(SiteC) + parts * per * sizeof(double);
  return l;
}

// The events of a slice for which `bytes` hold the layout l, up to n; their
// workgroups are numbered in 32 bits.
int64_t slice_events(int64_t n, const Layout& l, int32_t parts, size_t bytes) {
  if (bytes < l.total) n = std::min<int64_t>(n, (int64_t)((bytes - kAlignSlack) / l.per_event));
  return std::min<int64_t>(n, 0x7fffffffLL / ((int64_t)parts * std::max(l.n_mat, 1)));
}

// What n events need: all of them at once up to GWF_SPLIT_SLICE_BYTES, and
// beyond that a slice of as many as that holds.  That is 30000 neutron-star
// pairs' matrices (7 ms), beside which a slice's ragged end does not show: 36000
// and 60000 pairs 9.5 and 16.0 ms, where one workgroup per event takes 12.6 and
// 21.0; matrices of five interferometers of 12000 pairs 10.4 and 15.1 ms.
size_t needed(int64_t n, const NetDesc& nd, uint32_t flags, int what, int32_t parts) {
  const Layout l = layout(n, nd, flags, what, parts);
  if (l.total <= GWF_SPLIT_SLICE_BYTES) return l.total;
  return layout(slice_events(n, l, parts, GWF_SPLIT_SLICE_BYTES), nd, flags, what, parts).total;
}

gwf_status check(const gwf_events* ev, const gwf_network* net, const gwf_grid* grid, uint32_t flags, int32_t parts,
                 int what, const void* work, int64_t work_bytes, NetDesc& nd) {
  gwf_status st = api_check_common(ev, grid, flags);
  if (st) return st;
  if (flags & GWF_MIXED) return api_fail(GWF_E_UNSUPPORTED, "the mixed form runs through a plan");
  if (grid->kind == GWF_GRID_EXPLICIT)
    return api_fail(GWF_E_UNSUPPORTED, "the split form generates log grids; use the plain call for explicit grids");
  if (parts < 1 || parts > GWF_SPLIT_PARTS_MAX)
    return api_fail(GWF_E_INVALID_ARG, "parts=%d outside 1..%d", parts, GWF_SPLIT_PARTS_MAX);
  if ((st = api_pack_network(net, nd))) return st;
  const size_t need = needed(ev->n, nd, flags, what, parts);
  if (!work || ((uintptr_t)work & 255) || work_bytes < (int64_t)need)
    return api_fail(GWF_E_INVALID_ARG, "the split form needs %zu bytes of 256-byte aligned workspace, got %lld",
                    need, (long long)work_bytes);
  return GWF_OK;
}

// The events [e0, e0 + n) of ev; snr, status and the rows of fisher and snr_ifo
// are those of all of ev.
gwf_status run_slice(const gwf_events* ev, const gwf_grid* grid, int64_t e0, int64_t n, uint32_t flags, double snr_th,
                     int32_t parts, const NetDesc& nd, const Layout& l, void* work, double* fisher, double* snr,
                     double* snr_ifo, int32_t* status, hipStream_t s) {
  const uint8_t* active = ev->active ? ev->active + e0 : nullptr;
  if (fisher) fisher += e0;
  if (snr) snr += e0;
  if (snr_ifo) snr_ifo += e0;
  if (status) status += e0;
  unsigned char* w = static_cast<unsigned char*>(work);
  EventC* evc = reinterpret_cast<EventC*>(w);
  SiteC* sic = reinterpret_cast<SiteC*>(w + l.sic);
  double* partial = reinterpret_cast<double*>(w + l.partial);
  const bool rot = (flags & GWF_EARTH_ROT) != 0, tab = net_has_tables(nd);
  const int npi = api_npi(flags);
  SetupArgs sa{};
  sa.par = ev->par + e0; sa.ld = ev->ld; sa.n = n;
  sa.fmin = grid->fmin + e0; sa.fmax = grid->fmax ? grid->fmax + e0 : nullptr;
  sa.npts = grid->npts + e0; sa.npts_plan = grid->npts + e0;
  sa.npts_max = 0x7fffffff;
  sa.ecc = ev->ecc ? ev->ecc + e0 : nullptr; sa.fref = ev->f_ref_ecc ? ev->f_ref_ecc + e0 : nullptr;
  sa.flags = flags;
  sa.net = nd; sa.evc = evc; sa.sic = sic; sa.status = status; sa.active = active;
  sa.sets = l.sets; sa.n_set = l.n_set; sa.no_phase = l.n_mat == 0;
  hipError_t err = launch_setup(sa, s);
  if (err == hipSuccess && l.snr) {
    SnrPartsArgs pa{};
    pa.evc = evc; pa.sic = sic; pa.n_set = l.n_set; pa.set0 = l.set0; pa.parts = parts; pa.n = (int32_t)n;
    pa.net = nd; pa.partial = partial;
    err = launch_snr_parts(pa, rot, tab, s);
    if (err == hipSuccess) {
      SnrCombineArgs ca{};
      ca.n = n; ca.ld = ev->ld; ca.ldo = ev->n; ca.parts = parts; ca.n_ifo = nd.n_ifo; ca.active = active; ca.evc = evc;
      ca.partial = partial; ca.snr_th = snr_th; ca.snr = snr; ca.snr_ifo = snr_ifo;
      ca.status = l.n_mat && !(snr_th > 0.0) ? nullptr : status;
      err = launch_snr_combine(ca, s);
    }
  }
  if (err == hipSuccess && l.n_mat) {
    const int32_t unit = l.sets == kSetsIfos ? kIfoStretch : kFisherStretch;
    ItemsArgs ia{};
    ia.evc = evc; ia.sic = sic; ia.n_site = l.n_mat > 1 || l.sets == kSetsIfos ? 1 : nd.n_site;
    ia.partial = partial; ia.parts = parts; ia.unit = unit; ia.n = (int32_t)n; ia.n_mat = l.n_mat; ia.n_set = l.n_set;
    err = launch_items(ia, npi, rot, false, tab, n * parts * l.n_mat, s);
    if (err == hipSuccess) {
      CombineArgs ca{};
      ca.n = n; ca.ldo = ev->n; ca.evc = evc; ca.partial = partial; ca.parts = parts; ca.unit = unit; ca.n_mat = l.n_mat;
      ca.fisher = fisher; ca.snr = snr; ca.status = status; ca.par_mask = ev->par_mask ? ev->par_mask + e0 : nullptr;
      ca.keep_snr = snr_th > 0.0;
      err = launch_combine(ca, npi, s);
    }
  }
  if (err != hipSuccess) return api_hip_fail(err, "split launch");
  return GWF_OK;
}

// The events in slices of even length, as many as the workspace holds.
gwf_status run(const gwf_events* ev, const gwf_grid* grid, uint32_t flags, double snr_th, int32_t parts, int what,
               const NetDesc& nd, void* work, int64_t work_bytes, double* fisher, double* snr, double* snr_ifo,
               int32_t* status, hipStream_t s) {
  const int64_t most = slice_events(ev->n, layout(ev->n, nd, flags, what, parts), parts, (size_t)work_bytes);
  const int64_t slices = (ev->n - 1) / most + 1, len = (ev->n - 1) / slices + 1;
  const Layout l = layout(len, nd, flags, what, parts);
  for (int64_t e0 = 0; e0 < ev->n; e0 += len) {
    const gwf_status st = run_slice(ev, grid, e0, std::min(len, ev->n - e0), flags, snr_th, parts, nd, l, work, fisher,
                                    snr, snr_ifo, status, s);
    if (st) return st;
  }
  return GWF_OK;
}

}  // namespace

extern "C" {

int64_t gwf_split_bytes(int64_t n, const gwf_network* net, uint32_t flags, int32_t what, int32_t parts) {
  NetDesc nd;
  if (n < 1 || n > 0x7fffffffLL || what < kWhatSnr || what > kWhatIfos || parts < 1 || parts > GWF_SPLIT_PARTS_MAX) {
    api_fail(GWF_E_INVALID_ARG, "n=%lld, what=%d or parts=%d out of range", (long long)n, what, parts);
    return -1;
  }
  if (api_pack_network(net, nd)) return -1;
  return (int64_t)needed(n, nd, flags, what, parts);
}

gwf_status gwf_snr_split(const gwf_events* ev, const gwf_network* net, const gwf_grid* grid, uint32_t flags,
                         int32_t parts, double* snr, double* snr_ifo, int32_t* status, void* work,
                         int64_t work_bytes, void* stream) {
  NetDesc nd;
  gwf_status st = check(ev, net, grid, flags, parts, kWhatSnr, work, work_bytes, nd);
  if (st) return st;
  if (!snr) return api_fail(GWF_E_INVALID_ARG, "snr is NULL");
  return run(ev, grid, flags, 0.0, parts, kWhatSnr, nd, work, work_bytes, nullptr, snr, snr_ifo, status,
             (hipStream_t)stream);
}

gwf_status gwf_fisher_split(const gwf_events* ev, const gwf_network* net, const gwf_grid* grid, uint32_t flags,
                            double snr_th, int32_t parts, double* fisher, double* snr, double* snr_ifo,
                            int32_t* status, void* work, int64_t work_bytes, void* stream) {
  NetDesc nd;
  const int what = snr_ifo || snr_th > 0.0 ? kWhatSnrFisher : kWhatFisher;
  gwf_status st = check(ev, net, grid, flags, parts, what, work, work_bytes, nd);
  if (st) return st;
  if (!fisher || !snr || !status) return api_fail(GWF_E_INVALID_ARG, "fisher, snr and status are required");
  if (!std::isfinite(snr_th)) return api_fail(GWF_E_INVALID_ARG, "snr_th is not finite");
  return run(ev, grid, flags, snr_th, parts, what, nd, work, work_bytes, fisher, snr, snr_ifo, status,
             (hipStream_t)stream);
}

gwf_status gwf_fisher_ifo_split(const gwf_events* ev, const gwf_network* net, const gwf_grid* grid, uint32_t flags,
                                int32_t parts, double* fisher_ifo, int32_t* status, void* work,
                                int64_t work_bytes, void* stream) {
  NetDesc nd;
  gwf_status st = check(ev, net, grid, flags, parts, kWhatIfos, work, work_bytes, nd);
  if (st) return st;
  if (!fisher_ifo || !status) return api_fail(GWF_E_INVALID_ARG, "fisher_ifo and status are required");
  return run(ev, grid, flags, 0.0, parts, kWhatIfos, nd, work, work_bytes, fisher_ifo, nullptr, nullptr, status,
             (hipStream_t)stream);
}

}  // extern "C"
