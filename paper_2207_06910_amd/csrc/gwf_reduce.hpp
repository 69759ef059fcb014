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

// Recursive halving: of the N values v of every lane, the lanes with bit BIT
// keep the upper half and the others the lower, each added to the partner's
// share, and so on with the lower bits down to one value, v[0]; idx is its
// number and cnt <= 0 where the lane ends with none.  Every value is summed
// over the lanes as wave_sum does it.
template <int N, int BIT>
__device__ inline void scatter_sum(double* v, int lane, int& idx, int& cnt) {
  constexpr int H = (N + 1) / 2;
  const bool up = (lane & BIT) != 0;
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const double lo = v[i], hi = i + H < N ? v[i + H] : 0.0;
    v[i] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, BIT, 64);
  }
  idx += up ? H : 0;
  cnt = up ? cnt - H : (cnt < H ? cnt : H);
  if constexpr (BIT > 1) scatter_sum<H, BIT / 2>(v, lane, idx, cnt);
}

}  // namespace gwf
