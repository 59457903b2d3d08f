// Goes through every load that the dense kernels issue for a matrix, by the functions the kernels themselves compute their
// offsets with.  Stages: each load fetches 16 bytes of the matrix or nothing, and together they fetch every byte once.  Runs: each
// fetches dwords that hold bytes of the matrix or is refused, and a row's chunk lies in the LDS where it is read from, whole.
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

// Tiles of 32 rows of a matrix that begins `at` bytes into a dword, by runs of loads.
bool check_runs(int rows, int KB, uint32_t at, bool dwords) {
  const int64_t size = hago::run_size(rows, KB, dwords ? at : 0), blocks = (KB + 127) / 128;
  for (int m0 = 0; m0 < rows; m0 += 32)
    for (int b = 0; b < blocks; ++b) {
      const uint32_t base = (uint32_t)(m0 * KB) + (dwords ? at : 0);
      std::vector<int64_t> lds(32 * 128 / 4 + 32, -2);   // dword of the matrix that each of the LDS holds, -1: refused, -2: not written
      auto load = [&](uint32_t lane_offset, uint32_t instruction_offset, int dwords_each, size_t to) {
        for (int d = 0; d < dwords_each; ++d) {
          const uint64_t offset = (uint64_t)lane_offset + instruction_offset + 4u * d;
          if (offset >> 32) return std::printf("offset %llu\n", (unsigned long long)offset), false;
          const bool refused = offset >= (uint64_t)size + hago::kRunBack;
          const int64_t byte = (int64_t)offset - hago::kRunBack;
          if (!refused && (byte < 0 || byte % 4 != 0)) return std::printf("byte %lld\n", (long long)byte), false;
          if (lds[to + d] != -2) return std::printf("two loads to one place\n"), false;
          lds[to + d] = refused ? -1 : byte;
        }
        return true;
      };
      bool ok = true;
      for (uint32_t lane = 0; ok && lane < 64; ++lane)
        for (int i = 0; ok && i < 4; ++i)
          ok = load(hago::run_offset(base, (uint32_t)KB, lane, i, dwords) + 128u * b, 1024u * i, 4, (1024u * i + 16u * lane) / 4);
      for (uint32_t lane = 0; ok && dwords && lane < 32; ++lane)
        ok = load(hago::run_behind_offset(base, (uint32_t)KB, lane) + 128u * b, 0, 1, 32 * 128 / 4 + lane);
      // read back: chunk c of row r at r * 128 + 16 (c ^ (r / 2) % 8), its bytes shifted by those that its row begins into a dword
      for (int r = 0; ok && r < 32; ++r)
        for (int n = 0; ok && n < 128 + (dwords ? 4 : 0); n += 4) {
          const int64_t held = n < 128 ? lds[(r * 128 + 16 * ((n / 16) ^ ((r >> 1) & 7)) + n % 16) / 4] : lds[32 * 128 / 4 + r];
          const int64_t row = (int64_t)(m0 + r) * KB + (dwords ? at : 0), want = (dwords ? row & ~(int64_t)3 : row) + 128 * b + n;
          if (m0 + r < rows && want < row + KB && held != want) ok = (std::printf("row %d byte %d: %lld\n", r, n, (long long)held), false);
          if (m0 + r >= rows && row - (dwords ? 3 : 0) >= size && held != -1) ok = (std::printf("row %d beyond: %lld\n", r, (long long)held), false);
        }
      if (!ok) return std::printf("runs: rows %d KB %d at %u m0 %d block %d\n", rows, KB, at, m0, b), false;
    }
  return true;
}

}  // namespace

int main() {
  for (int K = 16; K <= 1296; K += 16)
    for (int rows : {1, 2, 7, 65})
      if (!check(rows, K)) return 1;
  for (int KB = 1; KB <= 400; ++KB)
    for (int rows : {1, 3, 31, 32, 33, 70}) {
      if (KB % 4 == 0 && !check_runs(rows, KB, 0, false)) return 1;
      for (uint32_t at = 0; at < 4; ++at)
        if (!check_runs(rows, KB, at, true)) return 1;
    }
  // the last rows of a matrix whose offsets are near 2^31
  static_assert(hago::run_offset((1u << 31) - (1u << 16), 128, 63, 0, false) + 1024 * 3 < 0xffffffffu - (1u << 29), "no offset wraps");
  std::printf("stream offsets: ok\n");
  return 0;
}
