// The byte offsets of loads into the LDS.  Plain C++, so that a host program can go through them.
//
// Loads whose k offset travels in the instruction's scalar offset: a raw buffer load's range check looks at the lane's offset
// only, the scalar offset is added behind it.  So a lane that has nothing to fetch, a row beyond the matrix or a k beyond its row, gets
// the lane offset kOob; every other lane's offset is that of 16 bytes inside the matrix.  Stages beyond K have lanes of the first
// kind only and no scalar offset.
#pragma once

#include <cstdint>

namespace hago {

constexpr uint32_t kOob = 0x80000000u;  // offset beyond any tensor (sizes are < 2^31 bytes)

// Of a lane that fetches row `row` (of `rows` rows of K bytes) and byte `chunk` of every stage's piece of it: the part
// that all stages share, ...
constexpr uint32_t stream_row_offset(int row, int rows, int K, int chunk) {
  return row < rows ? (uint32_t)row * (uint32_t)K + (uint32_t)chunk : kOob;
}
// ... the lane's offset in the stage that starts at byte k0 of the rows, ...
constexpr uint32_t stream_lane_offset(uint32_t row_offset, int k0, int chunk, int K) {
  return k0 + chunk < K ? row_offset : kOob;
}
// ... and that stage's scalar offset.
constexpr uint32_t stream_scalar_offset(int k0, int K) { return k0 < K ? (uint32_t)k0 : 0u; }

// Runs: up to four loads of a wavefront fill consecutive KB of LDS from one value of m0, load i with the instruction offset
// i KB.  That offset counts on both sides, so the lane offsets of load i take it back, from a descriptor that starts kRunBack
// bytes before the tensor; it counts in the range check too, which is by the dword.  A block is 128 bytes of 32 rows of KB bytes,
// 16 of which a lane fetches, eight rows a load.
constexpr uint32_t kRunStep = 1024, kRunBack = 3 * kRunStep, kRunBlock = 128;
// The byte of its row's block that the lane fetches from in load i: the chunks of a row are permuted by bits 1 to 3 of the row.
constexpr uint32_t run_chunk(uint32_t lane, int i) { return (((lane & 7u) ^ (lane >> 4)) * 16) ^ (i & 1 ? 64u : 0u); }
// The lane's offset in load i of the first block of the rows that begin `base` bytes into the tensor.  dwords: of the aligned dwords
// that hold them (base: into the dwords that hold the tensor).
constexpr uint32_t run_offset(uint32_t base, uint32_t KB, uint32_t lane, int i, bool dwords) {
  const uint32_t rows = (lane >> 3) * KB, r8 = (uint32_t)(8 * i) * KB, c = run_chunk(lane, i), back = kRunBack - kRunStep * (uint32_t)i;
  return dwords ? ((rows + (base + r8)) & ~3u) + c + back : rows + c + (base + r8 + back);
}
// Of the dword behind the block's of row lane % 32.
constexpr uint32_t run_behind_offset(uint32_t base, uint32_t KB, uint32_t lane) {
  return (((lane & 31u) * KB + base) & ~3u) + (kRunBack + kRunBlock);
}
// Bytes of the dwords that hold a tensor which begins `at` bytes into the first.
constexpr uint32_t run_size(int64_t rows, int64_t KB, uint32_t at) { return (uint32_t)((rows * KB + at + 3) & ~(int64_t)3); }

}  // namespace hago
