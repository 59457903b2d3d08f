// Goes through every load that a dense kernel with 128-byte stages issues for a matrix, by the functions the kernel itself
// computes its offsets with: each fetches 16 bytes of the matrix or nothing, and together they fetch every byte once.
#include "stream_offset.h"

#include <cstdio>
#include <vector>

namespace {

constexpr int kStage = 128;

bool check(int rows, int K) {
  const int64_t size = (int64_t)rows * K;
  std::vector<uint8_t> seen((size_t)size, 0);
  const int stages = (K + kStage - 1) / kStage;
  for (int row = 0; row < rows + 3; ++row)                     // a tile may end beyond the matrix
    for (int chunk = 0; chunk < kStage; chunk += 16) {
      const uint32_t all = hago::stream_row_offset(row, rows, K, chunk);
      for (int stage = 0; stage < stages + 3; ++stage) {       // two more are issued
        const uint32_t lane = hago::stream_lane_offset(all, stage * kStage, chunk, K);
        const uint32_t scalar = hago::stream_scalar_offset(stage * kStage, K);
        const bool wanted = row < rows && stage * kStage + chunk < K;
        if (!wanted) {
          // refused whether or not the scalar offset is counted, however the sum is formed
          if (lane < size || (uint64_t)lane + scalar < (uint64_t)size || (int64_t)lane < size - (int64_t)scalar || scalar > (uint64_t)size)
            return std::printf("rows %d K %d row %d chunk %d stage %d: offset %u + %u is not refused\n", rows, K, row, chunk, stage,
                               lane, scalar), false;
          continue;
        }
        const int64_t at = (int64_t)lane + scalar;
        if (at != (int64_t)row * K + stage * kStage + chunk || at + 16 > size)
          return std::printf("rows %d K %d row %d chunk %d stage %d: byte %lld of %lld\n", rows, K, row, chunk, stage, (long long)at,
                             (long long)size), false;
        for (int e = 0; e < 16; ++e) ++seen[(size_t)at + e];
      }
    }
  for (uint8_t n : seen)
    if (n != 1) return std::printf("rows %d K %d: a byte is fetched %d times\n", rows, K, n), false;
  return true;
}

}  // namespace

int main() {
  for (int K = 16; K <= 1296; K += 16)
    for (int rows : {1, 2, 7, 65})
      if (!check(rows, K)) return 1;
  std::printf("stream offsets: ok\n");
  return 0;
}
