// How the depthwise matrix kernel divides a layer's row tiles between wavefronts.  Plain C++, so that a host program can go
// through it.
#pragma once

#include <cstdint>

namespace hago {

struct DwSplit {
  int64_t runs;          // of row tiles, a wavefront each and channel group
  int32_t per, longer;   // tiles of a run; the first `longer` runs have one more
  bool by_xcd;           // an XCD takes its workgroups (gx of a run after gx of the run before) in a row, else every eighth
};

// gx: workgroups of a run, waves: wavefronts of a run, tiles: row tiles of the layer.
//
// Row tiles per wavefront: about as many as leave 2.5 wavefronts per SIMD (a wavefront then has the next tile's loads under
// way while it computes; with half as many, or with one tile each, 32 x 288 planes of 28 x 28 took 7.7 and 8.0 us, so 6.4).
//
// An XCD that takes its workgroups in a row has them from one or two runs, and 32 CUs for them: the layer's time is that of the CU
// with the most tiles, and it has nothing of a short last run, which in launch order fills up every CU.  So the runs are
// equally long but for one tile, and of the length with the least work on the busiest CU, a workgroup's start counted as 0.6 of a tile,
// few workgroups on a CU as what they do not hide of each other's loads, more than four, which it has no room for at once, as
// 8 % (fitted to 258 layers, each with twelve lengths).  Us in launch order with a short last run, by XCD with one, and so: 556 channels
// stride 2 on 21 x 41 x 41 12.2, 14.7, 12.5; 961 stride 2 on 32 x 31 x 31 13.9, 15.4, 13.9; 505 stride 2 on 4 x 112 x 112 10.3, 13.3,
// 10.3; 651 raw on 45 x 32 x 32 40.7, 50.8, 39.8; 222 stride 2 on 7 x 112 x 112 8.9, 10.6, 9.4; 798 on 10 x 20 x 20 6.1, 6.6, 6.1.
//
// Where the busiest CU would still have half as much again as its share (with few tiles, the last a light one), launch order: 136
// channels stride 2 on 2 x 65 x 66, rows 32 + 32 + 2, 3.25, 3.8 by XCD.
inline DwSplit dw_split(int64_t gx, int64_t waves, int64_t tiles) {
  int64_t per = tiles * waves / 2560;
  per = per < 1 ? 1 : (per > 16 ? 16 : per);
  auto busiest = [&](int64_t runs) {
    const int64_t workgroups = ((gx * runs + 7) / 8 + 31) / 32, longest = (tiles + runs - 1) / runs;
    return (double)workgroups * ((double)longest + 0.6) * (workgroups == 1 ? 1.3 : workgroups == 2 ? 1.05 : workgroups <= 4 ? 1.0 : 1.08);
  };
  int64_t runs = (tiles + per - 1) / per;
  const double share = ((double)tiles + 0.6 * (double)runs) * (double)gx / 256;
  double least = busiest(runs);
  if (per > 1)
    for (int64_t longest = per / 2; longest <= 16 && 2 * longest <= 5 * per; ++longest) {
      const int64_t n = (tiles + longest - 1) / longest;
      const double b = n <= 65535 ? busiest(n) : least;  // (a launch's second dimension)
      if (b < least) least = b, runs = n;
    }
  return {runs, (int32_t)(tiles / runs), (int32_t)(tiles % runs), least <= 1.5 * (share < 1.6 ? 1.6 : share)};
}

}  // namespace hago
