// gwf_batched.hip -- batched form of the Fisher/SNR path for catalogues with
// uneven grid lengths.
//
//   setup_kernel    three lanes per event (the parts of its constants) and one
//                   per event x site, each on a row of workgroups of its own:
//                   written once to a workspace.
//   items_kernel    one workgroup per work item (event, point range [k0, k1),
//                   at most `chunk` points), dispatched in the plan's
//                   longest-first order, writes the item's partial sums to its
//                   own slot (the item's position in event order), so long
//                   and short events are spread evenly over the chip, the
//                   last items to start are the shortest, and the result
//                   does not depend on which workgroup took which item.  (A
//                   persistent form pulling items from a counter kept more
//                   values live across its outer loop: more register spills,
//                   1.7% slower.)  The event's constants are read from the
//                   workspace through the constant address space, i.e. by
//                   scalar loads into SGPRs, which costs neither LDS traffic
//                   nor vector registers.
//   combine_kernel  sums each event's item partials in item order and writes
//                   the Fisher matrix, SNR and status.
// Every step is an ordinary kernel on one stream, so the sequence can be
// captured in a HIP graph and replayed.
#include "gwf_batched.hpp"
#include "gwf_fisher_body.hpp"
#include "gwf_snr_body.hpp"

namespace gwf {

__global__ void fill_i32_kernel(int32_t* p, int32_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Lane e of the grid's row y: y = 0, 1, 2 form one part each of event e's
// constants (EventC; the first part its status), y = 3 + r its r-th site
// constants (SiteSets; with pi M formed from the parameters exactly as the
// event's grid part forms it); all write straight into the workspace.  A site of an
// event whose set-up fails is written anyway and never read.  The rows are
// independent workgroups, so a small catalogue's set-up takes as long as the
// longest of the parts, not their sum.
constexpr int kSetupRows = 3;

__global__ __launch_bounds__(64) void setup_kernel(SetupArgs a) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= a.n) return;
  const int row = blockIdx.y;
  const bool tidal = (a.flags & kFlagTidal) != 0;
  double p[kNparIn];
  for (int r = 0; r < 13; ++r) p[r] = (r < 11 || tidal) ? a.par[r * a.ld + e] : 0.0;
  p[13] = (a.flags & kFlagEcc) && a.ecc ? a.ecc[e] : 0.0;
  p[14] = (a.flags & kFlagEcc) && a.fref ? a.fref[e] : 0.0;
  if (row == 0) {
    EventC& ec = a.evc[e];
    event_grid_setup(p, a.fmin[e], a.fmax ? a.fmax[e] : 0.0, a.npts[e], a.flags, ec);
    if (!ec.status_circ) GridWalk::keep_ratios(ec, kBlock);
    if (!ec.status && (a.npts[e] != a.npts_plan[e] || a.npts[e] > a.npts_max))
      ec.status = ec.status_circ = kEvInvalid;   // grid changed since the items were built, or longer than they allow
    if (a.status) a.status[e] = ec.status;
  } else if (row == 1) {
    if (!a.no_phase) event_phase_setup(p, a.flags, a.evc[e]);
  } else if (row == 2) {
    event_angle_setup(p, a.fmin[e], a.flags, a.evc[e]);
  } else {
    const int r = row - kSetupRows;
    int s = r;                                   // the entry's site
    bool arms = a.sets == kSetsArms;
    int32_t ifo_sel = 0;
    if (a.sets == kSetsSitesArms && r >= a.net.n_site) {
      s = r - a.net.n_site;
      arms = true;
    } else if (a.sets == kSetsIfos) {
      ifo_sel = r + 1;
      int left = r;
      for (s = 0; left >= (a.net.site[s].shape == 1 ? 3 : 1); ++s) left -= a.net.site[s].shape == 1 ? 3 : 1;
    }
    const uint32_t on =
        arms ? kArmsPlain : select_ifo(site_arms_on(a.active, a.ld, e, a.net, s), a.net, s, ifo_sel);
    site_setup(p, a.net.site[s], kPi * total_mass_s(p), a.sic[e * a.n_set + r], on);
  }
}

template <int NPI, bool ROT, bool MIXED, bool TAB>
__global__ __launch_bounds__(kBlock, 2) void items_kernel(ItemsArgs a) {
  using Dm = FisherDims<NPI>;
  constexpr int NACC = Dm::NACC;
  __shared__ FisherLds<NPI, 2> L;
  const int tid = threadIdx.x;
  const int n_site = a.n_site;
  // workgroup b takes item b (the plan orders its items longest first, and
  // workgroups are dispatched in order); with the count on the device, the
  // grid is its upper bound and the surplus workgroups leave
  Item w;
  int32_t n_set = n_site, set0 = 0;
  if (a.items) {
    const int32_t n_items = a.n_items_dev ? *a.n_items_dev : a.n_items;
    const int64_t it = a.base + blockIdx.x;
    if (it >= n_items) return;
    w = a.items[it];
  } else {
    // part-major within a matrix: the first parts, which every event has, come
    // first, and the workgroups with nothing to do last
    const uint32_t u = (uint32_t)(a.base + blockIdx.x), n = (uint32_t)a.n;
    const uint32_t row = u / n, mat = row / (uint32_t)a.parts;
    const int32_t part = (int32_t)(row - mat * (uint32_t)a.parts);
    w.e = (int32_t)(u - row * n);
    const int32_t ne = a.evc[w.e].n, len = part_length(ne, a.parts, a.unit);
    w.k0 = part * len;
    if (a.evc[w.e].status || w.k0 >= ne) return;   // its sums are not read
    w.k1 = w.k0 + min(ne - w.k0, len);
    w.slot = ((int32_t)mat * a.n + w.e) * a.parts + part;
    n_set = a.n_set;
    if (a.n_mat > 1) set0 = (int32_t)mat;
  }
  const int32_t ew = __builtin_amdgcn_readfirstlane(w.e);
  const int32_t k0 = __builtin_amdgcn_readfirstlane(w.k0);
  const int32_t k1 = __builtin_amdgcn_readfirstlane(w.k1);
  set0 = __builtin_amdgcn_readfirstlane(set0);
  // constants read through the constant address space: uniform, never
  // written during the kernel, so the compiler may use scalar loads
  typedef const __attribute__((address_space(4))) EventC CEventC;
  typedef const __attribute__((address_space(4))) SiteC CSiteC;
  CEventC* ecp = (CEventC*)(a.evc) + ew;
  CSiteC* scp = (CSiteC*)(a.sic) + (int64_t)ew * n_set + set0;
  const EventC& ecg = *(const EventC*)ecp;
  const SiteC* scg = (const SiteC*)scp;
  double* out = a.partial + (int64_t)__builtin_amdgcn_readfirstlane(w.slot) * NACC;
  if (ecg.status) {
    if (tid < NACC) out[tid] = 0.0;
  } else {
    double t = 0.0;
    fisher_sums<NPI, 2, ROT, MIXED, false, TAB>(ecg, scg, n_site, k0, k1, L, &t);
    if (tid < NACC) out[tid] = t;
  }
}

template <int NPI_>
__global__ void combine_kernel(CombineArgs a) {
  using Dm = FisherDims<NPI_>;
  constexpr int P = Dm::P, NPI = Dm::NPI, NACC = Dm::NACC;
  const int64_t t = a.base + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t n_mat = a.item_first ? 1 : a.n_mat;
  if (t >= a.n * NACC * n_mat) return;
  const int64_t u = t / NACC;                      // (matrix, event)
  const int slot = (int)(t - u * NACC);
  const int64_t mat = n_mat > 1 ? u / a.n : 0, e = u - mat * a.n;
  const int32_t st0 = a.evc[e].status;
  double s = 0.0;
  if (!st0) {
    int64_t i0, i1;
    if (a.item_first) {
      i0 = a.item_first[e];
      i1 = a.item_first[e + 1];
    } else {
      const int32_t ne = a.evc[e].n;
      i0 = u * a.parts;
      i1 = i0 + (ne - 1) / part_length(ne, a.parts, a.unit) + 1;
    }
    for (int64_t i = i0; i < i1; ++i) s += a.partial[i * NACC + slot];
  }
  int r, c;
  slot_position(slot, NPI, r, c);
  if (r == 8 && c == 8 && a.snr && !(st0 && a.keep_snr)) a.snr[e] = sqrt(s);
  if (!rows_in(event_rows(a.par_mask, e), r, c)) s = 0.0;   // not one of the event's rows
  double* F = a.fisher + mat * ((int64_t)P * P * a.ldo);
  F[((int64_t)r * P + c) * a.ldo + e] = s;
  F[((int64_t)c * P + r) * a.ldo + e] = s;
  // the set-up kernel wrote the parameter status; a non-finite sum adds its bit
  if (!st0 && !finite(s)) atomicOr(a.status + e, (int32_t)kEvNonFinite);
}

constexpr int kScanBlock = 1024;

// One workgroup: item counts per event and their exclusive prefix sum, tile
// by tile of kScanBlock events (wavefront scans, then the wavefront totals,
// then the running carry of the earlier tiles).
__global__ __launch_bounds__(kScanBlock) void items_scan_kernel(const int32_t* __restrict__ npts, int64_t n,
                                                                int32_t chunk, int32_t npts_max,
                                                                int32_t* __restrict__ first,
                                                                int32_t* __restrict__ n_items) {
  __shared__ int32_t wtot[kScanBlock / 64];
  __shared__ int32_t carry;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) carry = 0;
  __syncthreads();
  for (int64_t base = 0; base < n; base += kScanBlock) {
    const int64_t e = base + tid;
    int32_t c = 0;
    if (e < n) {
      int32_t m = npts[e];
      if (m < 2 || m > npts_max) m = 2;
      c = (m - 1) / chunk + 1;
    }
    int32_t x = c;                                   // inclusive scan within the wavefront
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int32_t y = __shfl_up(x, off, 64);
      if (lane >= off) x += y;
    }
    if (lane == 63) wtot[wave] = x;
    __syncthreads();
    int32_t before = carry;                          // earlier tiles and earlier wavefronts
    for (int w = 0; w < wave; ++w) before += wtot[w];
    if (e < n) first[e] = before + x - c;
    __syncthreads();                                 // every lane has read carry and wtot
    if (tid == kScanBlock - 1) carry = before + x;
    __syncthreads();
  }
  if (tid == 0) {
    first[n] = carry;
    *n_items = carry;
  }
}

// One lane per event writes its items (slot = position in event order).
__global__ void items_fill_kernel(const int32_t* __restrict__ npts, int64_t n, int32_t chunk, int32_t npts_max,
                                  const int32_t* __restrict__ first, Item* __restrict__ items) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  int32_t m = npts[e];
  if (m < 2 || m > npts_max) m = 2;
  const int32_t f0 = first[e], f1 = first[e + 1];
  for (int32_t i = f0, k0 = 0; i < f1; ++i, k0 += chunk)
    items[i] = Item{(int32_t)e, k0, min(m, k0 + chunk), i};
}

hipError_t launch_items_build(const int32_t* npts, int64_t n, int32_t chunk, int32_t npts_max, int32_t* first,
                              int32_t* n_items, Item* items, hipStream_t s) {
  hipLaunchKernelGGL(items_scan_kernel, dim3(1), dim3(kScanBlock), 0, s, npts, n, chunk, npts_max, first, n_items);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(items_fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, npts, n, chunk, npts_max,
                     first, items);
  return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

hipError_t launch_setup(const SetupArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(setup_kernel, dim3((unsigned)((a.n + 63) / 64), (unsigned)(kSetupRows + a.n_set)), dim3(64), 0, s,
                     a);
  return hipGetLastError();
}

template <int NPI, bool MIXED>
void launch_items_n(const ItemsArgs& a, bool rot, bool tab, dim3 grid, dim3 block, hipStream_t s) {
  if (rot && tab) hipLaunchKernelGGL((items_kernel<NPI, true, MIXED, true>), grid, block, 0, s, a);
  else if (rot) hipLaunchKernelGGL((items_kernel<NPI, true, MIXED, false>), grid, block, 0, s, a);
  else if (tab) hipLaunchKernelGGL((items_kernel<NPI, false, MIXED, true>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((items_kernel<NPI, false, MIXED, false>), grid, block, 0, s, a);
}

template <bool MIXED>
void launch_items_t(const ItemsArgs& a, int npi, bool rot, bool tab, dim3 grid, dim3 block, hipStream_t s) {
  switch (npi) {
    case 6: launch_items_n<6, MIXED>(a, rot, tab, grid, block, s); break;
    case 5: launch_items_n<5, MIXED>(a, rot, tab, grid, block, s); break;
    case 4: launch_items_n<4, MIXED>(a, rot, tab, grid, block, s); break;
    default: launch_items_n<3, MIXED>(a, rot, tab, grid, block, s);
  }
}

hipError_t launch_items(const ItemsArgs& a0, int npi, bool rot, bool mixed, bool tab, int64_t n_wg, hipStream_t s) {
  return launch_slices(a0, n_wg, 1, kBlock, [&](const ItemsArgs& a, dim3 grid, dim3 block) {
    if (mixed) launch_items_t<true>(a, npi, rot, tab, grid, block, s);
    else launch_items_t<false>(a, npi, rot, tab, grid, block, s);
  });
}

int fisher_nacc(int npi) {
  switch (npi) {
    case 6: return FisherDims<6>::NACC;
    case 5: return FisherDims<5>::NACC;
    case 4: return FisherDims<4>::NACC;
    default: return FisherDims<3>::NACC;
  }
}

hipError_t launch_combine(const CombineArgs& a0, int npi, hipStream_t s) {
  return launch_slices(a0, a0.n * fisher_nacc(npi) * (a0.item_first ? 1 : a0.n_mat), 256, 256, [&](const CombineArgs& a, dim3 grid, dim3 block) {
    switch (npi) {
      case 6: hipLaunchKernelGGL((combine_kernel<6>), grid, block, 0, s, a); break;
      case 5: hipLaunchKernelGGL((combine_kernel<5>), grid, block, 0, s, a); break;
      case 4: hipLaunchKernelGGL((combine_kernel<4>), grid, block, 0, s, a); break;
      default: hipLaunchKernelGGL((combine_kernel<3>), grid, block, 0, s, a);
    }
  });
}

// The SNR sums of one part of one event's grid (split form), constants read by
// scalar loads as in items_kernel.
template <bool ROT, bool TAB>
__global__ __launch_bounds__(kBlock, 2) void snr_parts_kernel(SnrPartsArgs a) {
  __shared__ double red[kWaves][kMaxIfo];
  const uint32_t u = (uint32_t)(a.base + blockIdx.x), n = (uint32_t)a.n;
  const int32_t part = (int32_t)(u / n), e = (int32_t)(u - (uint32_t)part * n);
  typedef const __attribute__((address_space(4))) EventC CEventC;
  typedef const __attribute__((address_space(4))) SiteC CSiteC;
  const EventC& ec = *(const EventC*)((CEventC*)(a.evc) + e);
  const SiteC* sc = (const SiteC*)((CSiteC*)(a.sic) + (int64_t)e * a.n_set + a.set0);
  const int32_t len = part_length(ec.n, a.parts, kSnrStretch), k0 = part * len;
  if (ec.status_circ || k0 >= ec.n) return;        // its sums are not read
  double acc[kSnrSlots];
#pragma unroll
  for (int i = 0; i < kSnrSlots; ++i) acc[i] = 0.0;
  snr_sums<ROT, false, TAB, true>(ec, sc, a.net.n_site, k0, k0 + min(ec.n - k0, len), acc);
  double t;
  snr_reduce(acc, a.net.n_site, a.net.n_ifo, site_shapes(a.net), red, &t);
  if ((int)threadIdx.x < a.net.n_ifo) a.partial[((int64_t)e * a.parts + part) * a.net.n_ifo + threadIdx.x] = t;
}

__global__ __launch_bounds__(64) void snr_combine_kernel(SnrCombineArgs a) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= a.n) return;
  const int32_t st0 = a.evc[e].status_circ;
  const int32_t parts = st0 ? 0 : (a.evc[e].n - 1) / part_length(a.evc[e].n, a.parts, kSnrStretch) + 1;
  double tot = 0.0;
  for (int i = 0; i < a.n_ifo; ++i) {
    double t = 0.0;
    for (int32_t q = 0; q < parts; ++q) t += a.partial[(e * a.parts + q) * a.n_ifo + i];
    if (a.active && !a.active[(int64_t)i * a.ld + e]) t = 0.0;   // off for this event
    tot += t;
    if (a.snr_ifo) a.snr_ifo[(int64_t)i * a.ldo + e] = sqrt(t);
  }
  const double snr = sqrt(tot);
  a.snr[e] = snr;
  if (a.snr_th > 0.0) {                            // the pass before the matrices
    if (!a.evc[e].status && !(snr > a.snr_th)) {
      a.evc[e].status = kEvSkipped;
      if (a.status) a.status[e] = kEvSkipped;
    }
  } else if (a.status) {
    a.status[e] = st0 ? st0 : finite(tot) ? 0 : kEvNonFinite;
  }
}

hipError_t launch_snr_parts(const SnrPartsArgs& a0, bool rot, bool tab, hipStream_t s) {
  return launch_slices(a0, (int64_t)a0.n * a0.parts, 1, kBlock, [&](const SnrPartsArgs& a, dim3 grid, dim3 block) {
    if (rot && tab) hipLaunchKernelGGL((snr_parts_kernel<true, true>), grid, block, 0, s, a);
    else if (rot) hipLaunchKernelGGL((snr_parts_kernel<true, false>), grid, block, 0, s, a);
    else if (tab) hipLaunchKernelGGL((snr_parts_kernel<false, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((snr_parts_kernel<false, false>), grid, block, 0, s, a);
  });
}

hipError_t launch_snr_combine(const SnrCombineArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(snr_combine_kernel, dim3((unsigned)((a.n + 63) / 64)), dim3(64), 0, s, a);
  return hipGetLastError();
}

int fisher_block() { return kBlock; }

}  // namespace gwf
