// The byte offsets of DMA loads whose k offset travels in the instruction's scalar offset.  Plain C++, so that a host
// program can go through them.
//
// A raw buffer load's range check looks at the lane's offset only, the scalar offset is added behind it.  So a lane that has
// nothing to fetch, a row beyond the matrix or a k beyond its row, gets the lane offset kOob; every other lane's offset is
// that of 16 bytes inside the matrix.  Stages beyond K have lanes of the first kind only and no scalar offset.
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

}  // namespace hago
