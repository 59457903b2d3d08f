// Goes through the work that a depthwise layer's split gives to every CU, for layers of all sizes: the runs hold every row tile
// once, and by XCD no CU has much more than its share.
#include "dw_split.h"

#include <cstdio>
#include <vector>

namespace {

// Work of the busiest CU, in tiles and 0.6 of one for a workgroup's start: workgroup n runs on XCD n % 8, on the CU of it with the least so far.
double busiest_cu(int64_t gx, const std::vector<int64_t>& length, bool by_xcd) {
  std::vector<double> cu(256, 0);
  const int64_t all = gx * (int64_t)length.size();
  double most = 0;
  for (int64_t n = 0; n < all; ++n) {
    const int64_t x = n & 7, each = all >> 3, more = all & 7;
    const int64_t id = by_xcd ? x * each + (x < more ? x : more) + (n >> 3) : n;
    int64_t best = x * 32;
    for (int64_t c = x * 32; c < x * 32 + 32; ++c)
      if (cu[c] < cu[best]) best = c;
    const double work = 0.6 + (double)length[id / gx];
    cu[best] += work;
    most = cu[best] > most ? cu[best] : most;
  }
  return most;
}

}  // namespace

int main() {
  double worst = 0, sum_new = 0, sum_old = 0;
  int layers = 0;
  for (int64_t waves : {1, 5, 64, 130, 245, 288, 408, 490, 556, 798, 832, 888, 961, 1080, 1476, 1922, 2020})
    for (int64_t tiles = 1; tiles <= 130; tiles += tiles < 50 ? 1 : 7) {
      const int64_t gx = (waves + 3) / 4;
      const hago::DwSplit s = hago::dw_split(gx, waves, tiles);
      std::vector<int64_t> length;
      for (int64_t r = 0; r < s.runs; ++r) length.push_back(s.per + (r < s.longer));
      int64_t sum = 0;
      for (int64_t n : length) sum += n;
      if (sum != tiles || s.per < 1 || s.runs < 1 || s.longer < 0 || s.longer >= s.runs)
        return std::printf("%lld waves, %lld tiles: %lld runs of %d, %d longer\n", (long long)waves, (long long)tiles, (long long)s.runs, s.per, s.longer), 1;
      if (tiles * waves < 2 * 2560) continue;   // (one tile a wavefront: nothing to divide)
      // a run length by the number of wavefronts alone, what is left of the tiles as a last short run
      std::vector<int64_t> old;
      const int64_t per = tiles * waves / 2560 > 16 ? 16 : tiles * waves / 2560;
      for (int64_t left = tiles; left > 0; left -= per) old.push_back(left < per ? left : per);
      const double share = (double)gx * ((double)tiles + 0.6 * (double)old.size()) / 256;
      const double ratio = busiest_cu(gx, length, s.by_xcd) / share;
      worst = ratio > worst ? ratio : worst;
      // (what the rule admits before it gives an XCD's rows up)
      if (ratio > 1.5) return std::printf("%lld waves, %lld tiles, %lld runs: the busiest CU has %.2f of its share\n", (long long)waves, (long long)tiles, (long long)s.runs, ratio), 1;
      sum_old += busiest_cu(gx, old, true) / share;
      sum_new += ratio;
      ++layers;
    }
  if (sum_new > 0.95 * sum_old) return std::printf("the busiest CU has %.3f of its share on average, %.3f with short last runs\n", sum_new / layers, sum_old / layers), 1;
  std::printf("depthwise split: ok, the busiest CU has %.3f of its share, %.2f at most; %.3f with short last runs\n", sum_new / layers, worst, sum_old / layers);
  return 0;
}
