// gwf_waveform.hpp -- helpers shared by the strain kernel (gwf_waveform.hip)
// and the strain-derivative kernel (gwf_waveform_deriv.hip): the event's
// inputs and the phase's reduction in cycles.  The two kernels sit in
// separate sources because they are built with different code-generation
// options (see build.py).
#pragma once

#include "gwf_kernels.hpp"

namespace gwf {

constexpr int kWBlock = 256;

// A workgroup takes one part of an event's grid, whole runs of kWBlock points.
// The first point sits sh = offset mod 8 places past a 128-byte line of the rows
// and runs start on lines (eight complex values): where the row length is a
// multiple of eight, a wavefront's 1 KB store is then whole lines, while a run
// that starts inside one leaves the shared line to be completed by the next
// run.  Strain of 4000 pairs (3.1 GB) 825 -> 697 us, derivatives of 300 (3.0 GB)
// 904 -> 616 us.  Stores past the caches (non-temporal) were slower: 948 and
// 881 us.  Parts are stretches, not runs dealt out in turn, whose shared lines
// two XCDs complete wherever a row is not line-aligned: strain of 10^4 packed
// pairs 1.89 -> 1.75 ms, derivatives of 1000 3.13 -> 2.87 ms.
//
// How many (wave_part): a part pays for a set-up, that of about 1000 points.  A
// grid is cut into `share` parts, which share the idle chip out while the events
// alone do not fill it, and beyond that only into parts of `longest` runs, so
// that no long grid ends the launch alone.  The launchers choose:
//   strain       share 1024 / n (the workgroups that run at once), longest 16
//   derivatives  share 2048 / n below 512 events, else 1; longest 4: they write
//                11 to 14 times as much per point, so a set-up weighs less;
//                above 8192 events one part each
// Measured with one part, two and this: strain of 20000 black-hole pairs of
// 1000 points 374, 424 and 273 us (short grids, one part), of 300 and of 10^4
// neutron-star pairs 148, 95 and 68 us, 1.87, 1.70 and 1.70 ms; derivatives of
// 2000 pairs of 300 points 54, 79 and 50 us, of 64 ragged events 347 (one part)
// and 146 us, of 10^4 pairs of 2000 points 643 and 748 us with one and two.
inline int32_t wave_share(int64_t n, int64_t full) {
  return (int32_t)std::min<int64_t>(64, std::max<int64_t>(full / n, 1));
}

// Part `part` of at most `parts` of a grid of n points whose first sits sh places
// past a line: its points [k0, k1), k0 below 0 where the first run starts before
// the grid; false where it has none.
__host__ __device__ inline bool wave_part(int32_t n, int32_t sh, int32_t part, int32_t parts, int32_t share,
                                          int32_t longest, int32_t& k0, int32_t& k1) {
  const int32_t runs = (int32_t)(((int64_t)n + sh + kWBlock - 1) / kWBlock);
  int32_t m = runs < share ? runs : share;                 // the parts taken, of even length
  if (m * longest < runs) m = (runs - 1) / longest + 1;
  if (m > parts) m = parts;
  if (m <= 1) {
    k0 = -sh;
    k1 = n;
    return part == 0;
  }
  if (part >= m) return false;
  const int32_t each = runs / m, more = runs - each * m;
  const int32_t r0 = part * each + (part < more ? part : more), r1 = r0 + each + (part < more ? 1 : 0);
  k0 = (int32_t)((int64_t)r0 * kWBlock - sh);
  k1 = r1 == runs ? n : (int32_t)((int64_t)r1 * kWBlock - sh);
  return true;
}

// Whether wave_part has nothing for the part, without its divisions.
__host__ __device__ inline bool wave_part_empty(int32_t n, int32_t sh, int32_t part, int32_t share, int32_t longest) {
  return (int64_t)part * (part < share ? 1 : longest) * kWBlock >= (int64_t)n + sh;
}

// Event e's inputs: the 13 parameters (no tidal rows without tides), e0 and
// its reference frequency (with the eccentric flag, else zero).
__device__ inline void load_event(const WaveformArgs& a, int64_t e, bool tidal, double* p) {
  for (int r = 0; r < 13; ++r) p[r] = (r < 11 || tidal) ? a.par[r * a.ld + e] : 0.0;
  p[13] = a.ecc_flag && a.ecc ? a.ecc[e] : 0.0;
  p[14] = a.ecc_flag && a.fref ? a.fref[e] : 0.0;
}

// The event's constants and its sites', by wavefronts side by side: wavefront 0
// the grid, with the check that the event's columns [b, b + npts) lie inside
// a row of the output, and the status; wavefront 1 calls site(s, p) on one lane
// per site; wavefronts 2 and 3 the phase and angle series.  False (for the
// whole workgroup) if there is nothing to write; a workgroup that can have
// no points of the event leaves before any of it.
template <class Site>
__device__ inline bool wave_setup(const WaveformArgs& a, int64_t e, bool tidal, uint32_t flags, EventC& ec,
                                  int32_t& ok, int32_t& k0, int32_t& k1, const Site& site) {
  const int tid = threadIdx.x;
  const int32_t part = (int32_t)blockIdx.y;
  // (the first workgroup stays for the status, and does not wait for the grid's
  // length)
  if (part > 0 && wave_part_empty(a.npts[e], (int32_t)(a.offsets[e] & 7), part, a.share, a.longest)) return false;
  double p[kNparIn];
  load_event(a, e, tidal, p);
  if (tid == 0) {
    event_setup_grid(p, a.fmin, a.fmax, a.npts, a.goff, a.gf, e, flags, ec, kSetupGrid);
    const int64_t b = a.offsets[e];
    const bool range_ok = b >= 0 && b <= a.total - (int64_t)a.npts[e];
    int32_t st = ec.status;
    if (!range_ok) st |= kEvInvalid;
    ok = st == 0;
    if (a.status && blockIdx.y == 0) a.status[e] = st;
  } else if (tid >= 64 && tid < 64 + a.net.n_site) {
    site(tid - 64, p);
  } else if (tid == 128) {
    event_setup_grid(p, a.fmin, a.fmax, a.npts, a.goff, a.gf, e, flags, ec, kSetupPhase);
  } else if (tid == 192) {
    event_setup_grid(p, a.fmin, a.fmax, a.npts, a.goff, a.gf, e, flags, ec, kSetupAngle);
  }
  __syncthreads();
  return ok != 0 &&
         wave_part(ec.n, (int32_t)(a.offsets[e] & 7), part, (int32_t)gridDim.y, a.share, a.longest, k0, k1);
}

// x reduced to [-1/2, 1/2] by subtracting the nearest integer (exact).
__device__ inline double frac_center(double x) { return x - rint(x); }

// sin and cos of 2 pi x for |x| <= 1/2.  FP64: the quarter-turn q = rint(4x)
// and the rest r = x - q/4 are exact in cycles (|r| <= 1/8), so t = 2 pi r
// carries one rounding (|t| <= pi/4) and needs no Cody-Waite reduction; the
// Taylor series of sin to t^17 and cos to t^16 truncate below 1e-18.
// Mixed form: the quarter-turn q = rint(4x) and the rest
// r = x - q/4 (exact, |r| <= 1/8) are taken in FP64, then the Taylor series
// of sin (to the 9th power) and cos (to the 10th) of 2 pi r in FP32, whose
// truncation errors (< 2e-9, < 2e-10 on |2 pi r| <= pi/4) lie below the
// FP32 rounding; the absolute error is a few 1e-8 rad from rounding r and
// about 1e-7 from the FP32 arithmetic.
template <bool MIXED>
__device__ inline void sincos_cycles(double x, double* s, double* c) {
  if (MIXED) {
    const double q = rint(4.0 * x);
    const float t = (float)kTwoPi * (float)fma(-0.25, q, x);
    const float t2 = t * t;
    float ps = fmaf(t2, 1.0f / 362880.0f, -1.0f / 5040.0f);
    ps = fmaf(ps, t2, 1.0f / 120.0f);
    ps = fmaf(ps, t2, -1.0f / 6.0f);
    const float sr = fmaf(t * t2, ps, t);
    float pc = fmaf(t2, -1.0f / 3628800.0f, 1.0f / 40320.0f);
    pc = fmaf(pc, t2, -1.0f / 720.0f);
    pc = fmaf(pc, t2, 1.0f / 24.0f);
    pc = fmaf(pc, t2, -0.5f);
    const float cr = fmaf(t2, pc, 1.0f);
    const int k = (int)q & 3;                  // angle = k quarter turns + t
    const float ss = (k & 1) ? cr : sr, cc = (k & 1) ? sr : cr;
    *s = (double)((k & 2) ? -ss : ss);
    *c = (double)(((k + 1) & 2) ? -cc : cc);
  } else {
    const double q = rint(4.0 * x);
    const double t = kTwoPi * fma(-0.25, q, x);
    const double t2 = t * t;
    double ps = -1.0 / 355687428096000.0;          // -1/17!
    ps = fma(ps, t2, 1.0 / 1307674368000.0);       //  1/15!
    ps = fma(ps, t2, -1.0 / 6227020800.0);         // -1/13!
    ps = fma(ps, t2, 1.0 / 39916800.0);            //  1/11!
    ps = fma(ps, t2, -1.0 / 362880.0);             // -1/9!
    ps = fma(ps, t2, 1.0 / 5040.0);                //  1/7!
    ps = fma(ps, t2, -1.0 / 120.0);                // -1/5!
    ps = fma(ps, t2, 1.0 / 6.0);                   //  1/3!
    const double sr = fma(-t * t2, ps, t);
    double pc = 1.0 / 20922789888000.0;            //  1/16!
    pc = fma(pc, t2, -1.0 / 87178291200.0);        // -1/14!
    pc = fma(pc, t2, 1.0 / 479001600.0);           //  1/12!
    pc = fma(pc, t2, -1.0 / 3628800.0);            // -1/10!
    pc = fma(pc, t2, 1.0 / 40320.0);               //  1/8!
    pc = fma(pc, t2, -1.0 / 720.0);                // -1/6!
    pc = fma(pc, t2, 1.0 / 24.0);                  //  1/4!
    pc = fma(pc, t2, -0.5);                        // -1/2!
    const double cr = fma(t2, pc, 1.0);
    const int k = (int)q & 3;                      // angle = k quarter turns + t
    const double ss = (k & 1) ? cr : sr, cc = (k & 1) ? sr : cr;
    *s = (k & 2) ? -ss : ss;
    *c = ((k + 1) & 2) ? -cc : cc;
  }
}

}  // namespace gwf
