// wave_part_host.hip -- TEST ONLY: how the strain kernels share a grid out over
// workgroups (wave_part of gwf_waveform.hpp), on the host.
#include "../../paper_2207_06910_amd/csrc/gwf_waveform.hpp"

using namespace gwf;

// k[2 p], k[2 p + 1]: the points of part p (0, 0 where it has none); returns the
// number of parts that wave_part_empty gets wrong.
extern "C" int wave_parts_host(int32_t n, int32_t sh, int32_t parts, int32_t share, int32_t longest, int32_t* k) {
  int bad = 0;
  for (int32_t p = 0; p < parts; ++p) {
    int32_t k0 = 0, k1 = 0;
    const bool some = wave_part(n, sh, p, parts, share, longest, k0, k1);
    k[2 * p] = some ? k0 : 0;
    k[2 * p + 1] = some ? k1 : 0;
    // an empty part may not be seen where fewer parts are there than the grid would take
    if (p > 0 && some && wave_part_empty(n, sh, p, share, longest)) ++bad;
  }
  return bad;
}
