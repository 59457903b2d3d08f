// Pieces shared by the dense kernels for operands of any size and alignment (qgemm_any.hip, qgemm_few.hip).
//
// int16 operands (I16).  gfx950 has no 16-bit integer matrix instruction; a 16-bit value is the sum
// 256 ah + al of a signed high byte and an unsigned low one, and with al' = al - 128 both are signed bytes:
//   a = a' + 128, a' = 256 ah + al',     w likewise,
//   sum a w = 65536 sum ah wh + 256 sum (ah wl' + al' wh) + sum al' wl' + 128 sum a + 128 sum w - 16384 K,
// modulo 2^32 like the sum itself.  Four byte products in three accumulators replace one product (the vector
// ALUs' two-element dot product, which this replaced, runs at 1/32 of the byte rate); the plain sums of a
// row are taken by the lanes that load it.  Elements that pad the reduction are zeros in one operand at least (what the other
// holds there is in its plain sum, and cancels) and are counted in K.
#pragma once

#include "qgemm_common.h"

namespace hago {

// Plain sum of a register's elements, added to s.
template <bool I16>
__device__ __forceinline__ int32_t plain_sum(const v4i& v, int32_t s) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int d = v[e];
    if constexpr (I16)
      s = __builtin_amdgcn_sdot2(__builtin_bit_cast(__attribute__((ext_vector_type(2))) short, d),
                                 __builtin_bit_cast(__attribute__((ext_vector_type(2))) short, 0x00010001), s, false);
    else
      s = __builtin_amdgcn_sdot4(d, 0x01010101, s, false);
  }
  return s;
}

// High and low bytes of four int16 elements (low ones biased to signed).
__device__ __forceinline__ void split16(int d0, int d1, int& hi, int& lo) {
  hi = (int)__builtin_amdgcn_perm((uint32_t)d1, (uint32_t)d0, 0x07050301u);
  lo = (int)(__builtin_amdgcn_perm((uint32_t)d1, (uint32_t)d0, 0x06040200u) ^ 0x80808080u);
}

__device__ __forceinline__ v4i xor4(const v4i& a, uint32_t x) {
  return v4i{(int)((uint32_t)a.x ^ x), (int)((uint32_t)a.y ^ x), (int)((uint32_t)a.z ^ x), (int)((uint32_t)a.w ^ x)};
}

// The accumulators of a 32 x 32 tile and their sum modulo 2^32.
template <bool I16>
struct Tile32 {
  v16i a[I16 ? 3 : 1];
  __device__ void clear() {
#pragma unroll
    for (int i = 0; i < (I16 ? 3 : 1); ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) a[i][r] = 0;
  }
  __device__ int32_t value(int r) const {
    if constexpr (I16)
      return (int32_t)(((uint32_t)a[0][r] << 16) + ((uint32_t)a[1][r] << 8) + (uint32_t)a[2][r]);
    else
      return a[0][r];
  }
};

__device__ __forceinline__ v16i mfma(const v4i& p, const v4i& q, const v16i& a) {
  return __builtin_amdgcn_mfma_i32_32x32x32_i8(p, q, a, 0, 0, 0);
}

// Channel term without the activation's row sum: bias - 16384 K (int16) + coefficient * sum w.
template <bool I16>
__device__ __forceinline__ int32_t channel_term(const QgemmParams& p, int32_t bias, int32_t wsum, int32_t kpad) {
  if constexpr (I16) return bias + (int32_t)((uint32_t)(p.corr_coef + 128) * (uint32_t)wsum) - (int32_t)(16384u * (uint32_t)kpad);
  else return bias + (int32_t)((uint32_t)p.corr_coef * (uint32_t)wsum);
}

// qgemm_few.hip: whether it indexes a layer, whether it is the faster kernel for it, and its launch (4 or 8 wavefronts a
// tile, 0: by the layer's sizes).
bool qgemm_few_ok(const QgemmParams& p, bool i16);
bool qgemm_few_wins(const QgemmParams& p, bool i16);
hipError_t launch_qgemm_few(const QgemmParams& p, bool i16, int waves, hipStream_t st);
hipError_t launch_qgemm_any(const QgemmParams& p, bool i16, int form, hipStream_t st);

}  // namespace hago
