// gwf_fisher_body.hpp -- the per-workgroup Fisher accumulation shared by the
// one-event-per-workgroup kernel and the batched work-item kernel.
//
// A workgroup of kBlock lanes sums the contributions of grid points
// [k0, k1) of one event: each lane takes points k0 + tid + kBlock*it, two at
// a time, sums the products of all interferometers' response vectors at
// each point in registers (NetSums) and adds the point's share of the 8x8
// block of (Mc, eta, dL, theta, phi, iota, psi, tc) to its kGramAcc register
// accumulators (accumulate_sums).  The phase-only blocks Gamma_{b, 8+i} = sum U_b c_i and
// Gamma_{8+i, 8+j} = sum W c_i c_j split in two:
//   * the Phic column (c_0 = -1 at every point) needs only sums of U_b, which
//     are combinations of the lanes' accumulators (gram_phic), and of W c_i;
//   * the rest is a small dense contraction over frequency, X = sum_f a_f c_f^T
//     with a_f = (U_0, U_1, U_3, U_4, U_5, U_6, U_7, W c_1 .. W c_{NPI-1}, W)
//     and c_f = (c_1 .. c_{NPI-1}), its last row the sums of W c_i: every
//     iteration each wavefront stages its points' a_f and c_f in LDS and
//     folds them into 4x4 output tiles of X with the four-block FP64 MFMA
//     4x4x4 (k = frequency).  With tides (NPI = 5) the 12 x 4 block fills
//     three tiles, one MFMA per four points (a fourth tile slot idle); with
//     e0 as well eight tiles, two MFMAs.
// The sums are then reduced in a fixed order (recursive halving over each
// wavefront, then the waves in index order), so results are bitwise
// reproducible.
//
// What bounds it: FP64 issue.  On the BNS catalogue (9.7e7 points, three
// sites, four effective interferometers, P = 13) the work-item kernel takes
// 2.10 ms where the rank-2 update of five derivative rows per interferometer,
// one point per lane, took 2.81 ms.
#pragma once

#include "gwf_kernels.hpp"
#include "gwf_reduce.hpp"

namespace gwf {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int kURow[7] = {0, 1, 3, 4, 5, 6, 7};   // the U rows staged (U_dL = 0)

template <int NPI_>
struct FisherDims {
  static constexpr int NPI = NPI_;                   // phase-only parameters
  static constexpr bool TIDAL = NPI >= 5;
  static constexpr int P = 8 + NPI;
  static constexpr int NG = 36, NX = 8 * NPI, NY = NPI * (NPI + 1) / 2;
  static constexpr int NACC = NG + NX + NY;          // SNR^2 = Gamma_{Phic,Phic}
  // the staged contraction: NA rows of a_f (7 U rows, then W c_i for
  // i = 1..NPI-1, then W), NB columns c_1..c_{NPI-1}; its 4x4 output tiles are
  // those holding a U row, an element of the upper triangle of W c_i c_j or
  // the W row.  Rows and columns beyond NA and NB pad the last tiles: their
  // LDS is never written and their results are not read.
  static constexpr int NA = 7 + NPI, NB = NPI - 1;
  static constexpr int RG = (NA + 3) / 4, CG = (NB + 3) / 4;
  static constexpr int ROWS_A = 4 * RG, ROWS_B = 4 * CG;
  __host__ __device__ static constexpr bool tile_used(int r, int c) {
    return 4 * r < 7 || 4 * r + 3 >= NA - 1 || 4 * c + 3 >= (4 * r > 7 ? 4 * r : 7) - 7;
  }
  __host__ __device__ static constexpr int count_tiles() {
    int n = 0;
    for (int r = 0; r < RG; ++r)
      for (int c = 0; c < CG; ++c) n += tile_used(r, c) ? 1 : 0;
    return n;
  }
  static constexpr int NT = count_tiles();
  static constexpr int NM = (NT + 3) / 4;            // MFMA accumulators (4 tiles each)
  // row group and column group of the t-th used tile (row-major order)
  __host__ __device__ static constexpr int tile_rc(int t, bool col) {
    for (int r = 0; r < RG; ++r)
      for (int c = 0; c < CG; ++c)
        if (tile_used(r, c) && t-- == 0) return col ? c : r;
    return 0;
  }
  __host__ __device__ static constexpr int tile_r(int t) { return tile_rc(t, false); }
  __host__ __device__ static constexpr int tile_c(int t) { return tile_rc(t, true); }
};
static_assert(FisherDims<5>::NM == 1 && FisherDims<3>::NM == 1 && FisherDims<4>::NM == 1 &&
              FisherDims<6>::NM == 2, "tile counts");

// LDS working set of one workgroup whose lanes take NQ points per iteration
// (at most 70 KB, so that two workgroups, two wavefronts per SIMD, share a
// compute unit).
template <int NPI, int NQ>
struct FisherLds {
  using Dm = FisherDims<NPI>;
  // points per lane staged for one MFMA phase: all NQ, unless their rows would
  // leave no room for a second workgroup (e0 and tides)
  static constexpr int NS = NPI == 6 ? 1 : NQ;
  // Row stride of the staged operands, in doubles.  The lanes of an MFMA
  // operand read take rows 4 t + i (up to 16 rows: t the tile slot, i = 0..3)
  // at points 4 s + k, and row r starts on four-byte bank 2 r LD mod 64.  With
  // LD odd, r LD mod 32 differs for all 16 rows (an odd factor permutes the
  // residues), so the rows of a read, and of the paired reads the compiler
  // forms, fall on distinct banks.  Measured with 64 points staged: strides 68
  // and 66 left 3.9e8 and 9.9e7 bank-conflict cycles per launch, 65 and 67
  // none (67 the fastest).
  static constexpr int LD = 64 * NS + 3;
  double red[kWaves][Dm::NACC];
  double stA[kWaves][Dm::ROWS_A][LD];   // staged a_f, [row][point]
  double stB[kWaves][Dm::ROWS_B][LD];   // staged c_f
};

// A double that is the same in every lane, in scalar registers.
__host__ __device__ inline double uniform_d(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  const int64_t b = __double_as_longlong(x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
  return __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo));
#else
  return x;
#endif
}

// Load an event's inputs: the 13 parameters (missing tidal rows read as
// zero), e0 and its reference frequency (zero without eccentricity; a NULL
// f_ref array means the grid's first frequency).
__device__ inline void load_par(const double* __restrict__ par, int64_t ld, int64_t e, bool tidal,
                                const double* ecc, const double* fref, double p[kNparIn]) {
  for (int r = 0; r < 13; ++r) p[r] = (r < 11 || tidal) ? par[r * ld + e] : 0.0;
  p[13] = ecc ? ecc[e] : 0.0;
  p[14] = fref ? fref[e] : 0.0;
}

// Sums of points [k0, k1) of the event whose constants are ec/sc.  On
// return (after a workgroup barrier), lane t < NACC holds accumulator slot t
// (see slot_position) in *tot.
// NQ: the points a lane takes per iteration.  The event's and sites' constants
// are read once for them, and their site terms are independent instruction
// streams.  Measured on the BNS catalogue (10^4 events, 9.7e7 points, P = 13,
// constants in scalar registers): one point 2.37 ms, two 2.23 ms, and 2.14 ms
// with both points' rows staged for one MFMA phase; three wavefronts per SIMD
// at one point, in 168 registers, spill inside the loop (2.73 ms).  With the
// constants in LDS, read into vector registers, two points spill, so that
// kernel takes one.
template <int NPI_, int NQ, bool ROT, bool MIXED = false, bool EXPL = false, bool TAB = true>
__device__ inline void fisher_sums(const EventC& ec, const SiteC* sc, int n_site, int k0, int k1,
                                   FisherLds<NPI_, NQ>& L, double* tot) {
  using Dm = FisherDims<NPI_>;
  using Lds = FisherLds<NPI_, NQ>;
  constexpr int NS = Lds::NS;
  constexpr int NPI = Dm::NPI, NG = Dm::NG, NX = Dm::NX, NACC = Dm::NACC;
  const int tid = threadIdx.x;
  double G[kGramAcc];
#pragma unroll
  for (int i = 0; i < kGramAcc; ++i) G[i] = 0.0;
  // The MFMAs of an iteration alternate between two independent chains
  // per accumulator (summed once at the end), so consecutive MFMAs do not wait
  // for each other's results.  Every instantiation sums in the same order, so
  // a tile holds the same bits whichever tile slot it occupies (e0 = 0 gives
  // the circular matrix exactly).
  constexpr int NC = 2;
  double acc[Dm::NM][NC];
  const int wave = tid >> 6, lane = tid & 63;
  // four-block MFMA 4x4x4 operand layout: lane 16 k + 4 q + i holds A[q][i][k]
  // and B[q][k][i]; the result D[q][i][j] is in lane 16 i + 4 q + j.  Block q
  // of accumulator m is tile 4 m + q; an unused slot repeats the first tile.
  const int kk = lane >> 4, q4 = (lane >> 2) & 3, i4 = lane & 3;
  int arow[Dm::NM], bcol[Dm::NM];
#pragma unroll
  for (int m = 0; m < Dm::NM; ++m) {
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[m][c] = 0.0;
    const int t = 4 * m + q4;
    arow[m] = t < Dm::NT ? 4 * Dm::tile_r(t) + i4 : i4;
    bcol[m] = t < Dm::NT ? 4 * Dm::tile_c(t) + i4 : i4;
  }
  double(*A)[Lds::LD] = L.stA[wave];
  double(*B)[Lds::LD] = L.stB[wave];
  // on a log grid, v, 1/v and v^-12.42 walk from point to point (GridWalk)
  GridWalk gw;
  if (!EXPL) {
    const int k = point_past(k0, tid, k1) ? k1 - 1 : k0 + tid;
    if (NQ == 2) gw.start_kept(ec, k);     // the work-item kernels: the set-up kernel left the ratios
    else gw.start(ec, k, kBlock);
#pragma unroll
    for (int i = 0; i < 3; ++i) gw.ratio[i] = uniform_d(gw.ratio[i]);   // the same step in every lane
  }
  // A point's row into LDS, as the wavefront's staged point 64 i + lane.
  auto stage = [&](int i, const double* U, double W, const double* cph) {
    const int col = 64 * i + lane;
#pragma unroll
    for (int r = 0; r < 7; ++r) A[r][col] = U[kURow[r]];
#pragma unroll
    for (int j = 1; j < NPI; ++j) {
      A[6 + j][col] = W * cph[j];
      B[j - 1][col] = cph[j];
    }
    A[Dm::NA - 1][col] = W;
  };
  // X += A^T B over the wavefront's staged points, four points per step.  The
  // LDS-fed phase runs at raised issue priority, so it drains quickly while
  // the SIMD's other wave keeps the VALU busy.
  auto contract = [&]() {
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int s2 = 0; s2 < 16 * NS; ++s2) {
#pragma unroll
      for (int m = 0; m < Dm::NM; ++m) {
        const double av = A[arow[m]][4 * s2 + kk];
        const double bv = B[bcol[m]][4 * s2 + kk];
        acc[m][s2 % NC] = __builtin_amdgcn_mfma_f64_4x4x4f64(av, bv, acc[m][s2 % NC], 0, 0, 0);
      }
    }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_wave_barrier();
  };
  // A point past the range is evaluated as the range's last point with zero
  // weight; only the iterations that hold an end of the grid or of the range
  // test for it.
  ActiveSites act = active_sites(sc, n_site);
  act.list = (uint32_t)__builtin_amdgcn_readfirstlane((int)act.list);
  act.n = __builtin_amdgcn_readfirstlane(act.n);
#pragma unroll 1
  for (uint32_t kb = k0; kb < (uint32_t)k1; kb += NQ * kBlock) {
    // The per-event constants are re-read every iteration (uniform reads);
    // hoisting them out of the loop would need more registers than a lane has.
    __asm__ volatile("" ::: "memory");
    const int k = (int)(kb + tid);
    const bool inner = kb > 0 && kb + NQ * kBlock < (uint32_t)k1;
    double vv[NQ][3];
    if (!EXPL) walk_points<NQ>(ec, gw, k, kBlock, k1, inner, vv);
    Point q[NQ];
    NetSums net[NQ];
    network_sums<NQ, NPI, ROT, MIXED, EXPL, TAB>(ec, sc, act, k, kBlock, k1, inner, EXPL ? nullptr : vv, q,
                                                       net);
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      double U[8], W, cph[NPI];
      finish_point<NPI, ROT>(ec, q[i], net[i], G, U, W, cph);
      stage(NS == 1 ? 0 : i, U, W, cph);
      if (NS == 1 || i == NQ - 1) contract();
    }
  }

  // ---- deterministic reduction: wavefront butterflies, then the waves in order
  // The 8x8 block (NG values) and the Phic column's part from the lanes'
  // accumulators (8 values: -sum U_b for the rows Mc, eta, theta, phi, iota,
  // psi, tc, then Gamma_{Phic,Phic} = sum W).
  constexpr int NR = NG + 8;
  double rv[NR];
  gram_finish(ec, G, rv);
  {
    double* xc = rv + NG;
    gram_phic(ec, G, xc);
  }
  // Recursive halving over the wavefront: at each step a lane hands half of the
  // values it still holds to its partner and adds the partner's other half,
  // so that each lane ends with one value summed over all lanes: 45 exchanges
  // for 44 values where a butterfly per value takes 264, the same additions
  // in the same order.
  int idx = 0, cnt = NR;
  scatter_sum<NR, 32>(rv, lane, idx, cnt);
  if (cnt > 0) {
    const int x = idx - NG;                          // of the Phic column: rows 0, 1, 3 .. 8
    L.red[wave][idx < NG ? idx : NG + NPI * (x < 2 ? x : x + 1)] = rv[0];
  }
  // the dL row of the phase-only block is exactly zero (U_dL = 0)
  if (lane < NPI) L.red[wave][NG + 2 * NPI + lane] = 0.0;
  // lane 16 i + 4 q + j of accumulator m holds element (i, j) of tile 4 m + q:
  // rows 0..6 of X are U_0, U_1, U_3 .. U_7, rows 7.. the W c_i rows (i >= 1)
  // and the W row, column c is c_{c+1}; the upper triangle of W c_i c_j is kept
#pragma unroll
  for (int m = 0; m < Dm::NM; ++m) {
    const int t = 4 * m + q4;
    if (t >= Dm::NT) continue;
    const int row = 4 * Dm::tile_r(t) + kk, col = 4 * Dm::tile_c(t) + i4;
    int slot = -1;
    if (col < Dm::NB) {
      const int j = col + 1;
      if (row < 7) {
        slot = NG + kURow[row] * NPI + j;
      } else if (row == Dm::NA - 1) {
        slot = NG + NX + j;                          // Gamma_{Phic, 8+j} = -sum W c_j
      } else if (row < Dm::NA) {
        const int i = row - 6;
        if (j >= i) slot = NG + NX + i * NPI - (i * (i - 1)) / 2 + (j - i);
      }
    }
    double x = acc[m][0];
#pragma unroll
    for (int c = 1; c < NC; ++c) x += acc[m][c];
    if (row == Dm::NA - 1) x = -x;
    if (slot >= 0) L.red[wave][slot] = x;
  }
  __syncthreads();
  if (tid < NACC) {
    double t = L.red[0][tid];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) t += L.red[w][tid];
    *tot = t;
  }
}

}  // namespace gwf
