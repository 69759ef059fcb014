// gwf_snr_body.hpp -- the per-workgroup SNR accumulation of the
// one-event-per-workgroup kernel (gwf_fisher.hip).
//
// Every lane walks its grid points two at a time as the Fisher kernels do
// (GridWalk) and adds the weighted squared response of each arm to its own
// sums.  The sites' constants are those of site_setup with
// the arms themselves as effective interferometers (kArmsPlain): an L's one
// arm, a triangle's first two, whose third response is minus their sum.
//
// What bounds it: FP64 issue, about 80 instructions per point, 25 per site
// and 15 per arm.  On 3000 neutron-star binaries (2.9e7 points, three sites,
// five interferometers), a workgroup per stretch (gwf_split.hip): 0.237 ms, where
// an exponential per point and site, patterns from frame products and Horner
// series with one workgroup per event took 0.58 ms.
#pragma once

#include "gwf_fisher_body.hpp"

namespace gwf {

constexpr int kSnrSlots = 3 * kMaxSites;     // slot 3 s + k: arm k of site s

// A lane's walk is anchored (grid_values) every kSnrWalk points of the range,
// 16 steps of a workgroup, so its values carry at most 31 u however long the
// grid is.  Walked over the whole of one, the ratios' rounding adds up with one
// sign: 2.7e-12 of SNR^2 on 10^6 points in one workgroup.  The anchors cost 1 to
// 4 % (3000 neutron-star pairs 252 -> 253 us, 20000 black-hole pairs of 5000
// points 350 -> 366 us).
constexpr int kSnrWalk = 16 * kBlock;

// Adds the points of [k0, k1) that lane tid of a workgroup takes to its
// acc[kSnrSlots].  KEPT: the set-up kernel left the walk's ratios.
template <bool ROT, bool EXPL, bool TAB, bool KEPT = false>
__host__ __device__ inline void snr_lane(const EventC& ec, const SiteC* sc, int n_site, int k0, int k1, int tid,
                                         double* acc) {
  constexpr int NQ = 2;
  GridWalk gw;
  if (!EXPL) {
    const int k = point_past(k0, tid, k1) ? k1 - 1 : k0 + tid;
    if (KEPT) gw.start_kept(ec, k);
    else gw.start(ec, k, kBlock);
#pragma unroll
    for (int i = 0; i < 3; ++i) gw.ratio[i] = uniform_d(gw.ratio[i]);
  }
#pragma unroll 1
  for (uint32_t kb = k0; kb < (uint32_t)k1; kb += NQ * kBlock) {
    asm volatile("" ::: "memory");       // constants are re-read rather than held in registers
    const int k = (int)(kb + tid);
    const bool inner = kb > 0 && kb + NQ * kBlock < (uint32_t)k1;
    if (!EXPL && kb > (uint32_t)k0 && (kb - (uint32_t)k0) % kSnrWalk == 0)
      gw.anchor(ec, point_past(k, 0, k1) ? k1 - 1 : k);
    double vv[NQ][3];
    if (!EXPL) walk_points<NQ>(ec, gw, k, kBlock, k1, inner, vv);
    Point q[NQ];
    point_block<NQ, false, ROT, false, EXPL>(ec, k, kBlock, k1, inner, EXPL ? nullptr : vv, q);
    const double cplus = ec.cplus, ccross = ec.ccross;
#pragma unroll
    for (int s = 0; s < kMaxSites; ++s) {
      if (s < n_site) {
        asm volatile("" ::: "memory");
        const SiteC& st = sc[s];
        SiteTrigR sp[NQ];
        double om[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
          double cH, sH;
          hour_angle(q[i], st.cdl, st.sdl, cH, sH);
          trig_basis(cH, sH, 1.0, sp[i]);
          om[i] = psd_weight<TAB>(st, q[i], EXPL ? q[i].w4A2 : q[i].rw * q[i].rw);
        }
        double p0[NQ], x0[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
          p0[i] = cplus * trig_val_r(st.jk[0][0], sp[i]);
          x0[i] = ccross * trig_val_r(st.jk[0][1], sp[i]);
          acc[3 * s] = fma(om[i], fma(p0[i], p0[i], x0[i] * x0[i]), acc[3 * s]);
        }
        if (st.n_arm == 3) {
#pragma unroll
          for (int i = 0; i < NQ; ++i) {
            const double p1 = cplus * trig_val_r(st.jk[1][0], sp[i]), x1 = ccross * trig_val_r(st.jk[1][1], sp[i]);
            const double p2 = p0[i] + p1, x2 = x0[i] + x1;     // minus the third arm
            acc[3 * s + 1] = fma(om[i], fma(p1, p1, x1 * x1), acc[3 * s + 1]);
            acc[3 * s + 2] = fma(om[i], fma(p2, p2, x2 * x2), acc[3 * s + 2]);
          }
        }
      }
    }
  }
}

template <bool ROT, bool EXPL, bool TAB, bool KEPT = false>
__device__ inline void snr_sums(const EventC& ec, const SiteC* sc, int n_site, int k0, int k1, double* acc) {
  snr_lane<ROT, EXPL, TAB, KEPT>(ec, sc, n_site, k0, k1, threadIdx.x, acc);
}

// The workgroup's sums of every interferometer: on return (after a workgroup
// barrier) lane d < n_ifo holds interferometer d's in *tot.  shapes: bit s set
// where site s is a triangle.
__device__ inline void snr_reduce(double* acc, int n_site, int n_ifo, uint32_t shapes,
                                  double (*red)[kMaxIfo], double* tot) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  int idx = 0, cnt = kSnrSlots;
  scatter_sum<kSnrSlots, 32>(acc, lane, idx, cnt);
  const int s = idx / 3, k = idx - 3 * s;
  if (cnt > 0 && s < n_site && (k == 0 || (shapes >> s & 1u)))
    red[wave][s + 2 * __popc(shapes & ((1u << s) - 1u)) + k] = acc[0];
  __syncthreads();
  if (tid < n_ifo) {
    double t = red[0][tid];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) t += red[w][tid];
    *tot = t;
  }
}

__device__ inline uint32_t site_shapes(const NetDesc& net) {
  uint32_t m = 0;
  for (int s = 0; s < net.n_site; ++s) m |= (net.site[s].shape == 1 ? 1u : 0u) << s;
  return m;
}

}  // namespace gwf
