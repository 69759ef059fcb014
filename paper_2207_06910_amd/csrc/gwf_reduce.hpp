// gwf_reduce.hpp -- sums over the 64 lanes of a wavefront.
#pragma once

#include <hip/hip_runtime.h>

namespace gwf {

// The sum of x over the lanes, in every lane.
__device__ inline double wave_sum(double x) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// x of the lane whose number differs in bit BIT, within rows of 16 lanes.
template <int BIT>
__device__ inline double lane_xor(double x) {
  if constexpr (BIT == 4) return __shfl_xor(x, 4, 64);
  constexpr int ctrl = BIT == 8 ? 0x128 : BIT == 2 ? 0x4e : 0xb1;     // rotate by 8; quad (2,3,0,1); quad (1,0,3,2)
  uint32_t a[2];
  __builtin_memcpy(a, &x, 8);
#pragma unroll
  for (int w = 0; w < 2; ++w) a[w] = __builtin_amdgcn_update_dpp(0, a[w], ctrl, 0xf, 0xf, true);
  double y;
  __builtin_memcpy(&y, a, 8);
  return y;
}

// Recursive halving: of the N values v of every lane, the lanes with bit BIT
// keep the upper half and the others the lower, each added to the partner's
// share, and so on with the lower bits down to one value, v[0]; idx is its
// number and cnt <= 0 where the lane ends with none.  Every value is summed
// over the lanes as wave_sum does it.  The halves and rows of the wavefront are
// exchanged by lane swaps, which hand over both shares at once, the lanes of a
// row by rotations; by permutes through LDS, two for each value and four selects,
// 500 pairs' matrices of five interferometers in stretches of 2048 points took
// 534 us in place of 511.
template <int N, int BIT>
__device__ inline void scatter_sum(double* v, int lane, int& idx, int& cnt) {
  constexpr int H = (N + 1) / 2;
  const bool up = (lane & BIT) != 0;
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const double lo = v[i], hi = i + H < N ? v[i + H] : 0.0;
    if constexpr (BIT >= 16) {
      // the lanes with bit BIT clear give their hi for the partner's lo
      uint32_t a[2], b[2];
      __builtin_memcpy(a, &lo, 8);
      __builtin_memcpy(b, &hi, 8);
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const auto r = BIT == 32 ? __builtin_amdgcn_permlane32_swap(a[w], b[w], false, false)
                                 : __builtin_amdgcn_permlane16_swap(a[w], b[w], false, false);
        a[w] = r[0];
        b[w] = r[1];
      }
      double x, y;
      __builtin_memcpy(&x, a, 8);
      __builtin_memcpy(&y, b, 8);
      v[i] = x + y;
    } else {
      v[i] = (up ? hi : lo) + lane_xor<BIT>(up ? lo : hi);
    }
  }
  idx += up ? H : 0;
  cnt = up ? cnt - H : (cnt < H ? cnt : H);
  if constexpr (BIT > 1) scatter_sum<H, BIT / 2>(v, lane, idx, cnt);
}

}  // namespace gwf
