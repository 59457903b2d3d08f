// The byte offsets of DMA loads whose k offset travels in the instruction's scalar offset.  Plain C++, so that a host
// program can go through them.
//
// A raw buffer load's range check looks at the lane's offset only, the scalar offset is added behind it.  So a lane that has
// nothing to fetch, a row beyond the matrix or a k beyond its row, gets the lane offset kOob; every other lane's offset is
// that of 16 bytes inside the matrix.  Stages beyond K have lanes of the first kind only and no scalar offset.
#pragma once

#include <cstdint>

namespace hago {

constexpr uint32_t kOob = 0x80002000u;  // offset beyond any tensor (sizes are < 2^31 bytes), and beyond kRunBack more bytes

// Runs of up to four loads of a wavefront fill consecutive KB of LDS from one value of m0, load i with the instruction offset
// i KB.  That offset counts on both sides, so the lane offsets of load i take it back, from a descriptor that starts kRunBack
// bytes before the tensor.
constexpr uint32_t kRunStep = 1024, kRunBack = 3 * kRunStep;
constexpr uint32_t stream_run_offset(uint32_t lane_offset, int i) {
  return lane_offset == kOob ? kOob : lane_offset + (kRunBack - kRunStep * (uint32_t)i);
}

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

}  // namespace hago
