// Device-side helpers shared by the libhago kernels (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hago {

// Requantize epilogue parameters that are uniform over a launch.  The clip
// limits are stored relative to the output zero point:
//   clip(r + z, lo, hi) == clip(r, lo - z, hi - z) + z
// so the sum r + z is only formed once r is already small.
struct RequantScalars {
  int32_t z_out;
  int32_t lo_rel;  // clip_lo - z_out
  int32_t hi_rel;  // clip_hi - z_out
  int32_t half_away;  // tie rule: 0 toward +infinity, 1 away from zero (general code paths only)
};

// r = floor(acc * mult / 2^(31 + sh) + 1/2), exact in 64-bit integers
// (|acc * mult| < 2^62, rounding term <= 2^61).  The result always fits in
// int32 for mult < 2^31.
__device__ __forceinline__ int32_t rounding_mul_shift(int32_t acc, int32_t mult, int32_t sh) {
  const int64_t p = (int64_t)acc * (int64_t)mult + ((int64_t)1 << (30 + sh));
  return (int32_t)(p >> (31 + sh));
}

// Power-of-two scales (Sec. 5.1 of the paper: shifting replaces the multiplication): the
// multiplier array is absent and the requantize is round(acc / 2^s).  That is the general form
// with multiplier 2^30 (one half) and shift s - 1; the 64-bit forms below accept the resulting
// shift of -1 for s == 0 (rounding term 2^29, shift distance 30), the folded fast paths of the
// kernels exclude it like they exclude shift 0.
__device__ __forceinline__ int32_t rq_mult(const int32_t* mult, int64_t i) {
  return mult ? mult[i] : (1 << 30);
}
__device__ __forceinline__ int32_t rq_shift(const int32_t* mult, const int32_t* shift, int64_t i) {
  return shift[i] - (mult ? 0 : 1);
}
// The shift-only form itself, without a multiplication: floor(acc / 2^s + 1/2) is the floored
// quotient plus the first bit shifted out (no rounding term is added, so nothing can wrap).
__device__ __forceinline__ int32_t shift_round(int32_t acc, int32_t s) {
  return s > 0 ? (acc >> s) + ((acc >> (s - 1)) & 1) : acc;
}

// Accumulators narrower than 32 bits (int16 accumulation; 24-bit accumulators): the 32-bit sum
// reduced modulo 2^bits and sign-extended, which equals accumulating in that width all along
// (the reduction is a ring homomorphism).  wrap_shift = 32 - bits, 0 for a full int32.
__device__ __forceinline__ int32_t wrap_acc_bits(int32_t acc, int32_t wrap_shift) {
  return (int32_t)((uint32_t)acc << wrap_shift) >> wrap_shift;
}

// A 64-bit shift whose amount is in the last register a wavefront was allocated takes another amount, some of the time:
// where the wavefront's registers are the last of the register file, by what the errors look like (int16 requantize over
// rows of any length, 32 registers with an amount in v31: 5.8% of the wavefronts, of 16 places in the file; per-lane
// amounts; never elsewhere).  The compiler does not avoid it, so build.py looks through every kernel's assembly and refuses
// this form, and the kernels it names make their allocation one block larger: VGPR is a register of that block.
#define HAGO_SPARE_REGISTER(VGPR) asm volatile("" ::: VGPR)

// Workgroups go to the eight XCDs round-robin, each with an L2 of its own.  Numbered like this instead, an XCD works on a
// run of consecutive ones: number `id` of `count` in launch order -> its place.  Every kernel whose places follow the
// activations (images first, then pixels) so keeps an eighth of them on one XCD from layer to layer: what a layer wrote is
// in the L2 that the next one reads it through, and no L2 holds lines that another one writes.
__device__ __forceinline__ uint32_t xcd_run(uint32_t id, uint32_t count) {
  const uint32_t x = id & 7, each = count >> 3, more = count & 7;
  return x * each + (x < more ? x : more) + (id >> 3);
}

// Brings the first BYTES bytes of the kernel's arguments into the scalar cache, in one go.  A launch's arguments are in no cache
// when it starts, a line takes 500 to 600 cycles, and the compiler fetches fields where they are first used, one line behind
// the other.
template <int BYTES>
__device__ __forceinline__ void fetch_arguments() {
  static_assert(BYTES <= 384, "six lines");
  const auto args = __builtin_amdgcn_kernarg_segment_ptr();
  constexpr int kLast = (BYTES - 4) & ~3;
  constexpr auto line = [](int i) { return 64 * i < kLast ? 64 * i : kLast; };
  uint32_t d0, d1, d2, d3, d4, d5;
  asm volatile(
      "s_load_dword %0, %6, %7\n\ts_load_dword %1, %6, %8\n\ts_load_dword %2, %6, %9\n\t"
      "s_load_dword %3, %6, %10\n\ts_load_dword %4, %6, %11\n\ts_load_dword %5, %6, %12\n\ts_waitcnt lgkmcnt(0)"
      : "=&s"(d0), "=&s"(d1), "=&s"(d2), "=&s"(d3), "=&s"(d4), "=&s"(d5)
      : "s"(args), "n"(line(0)), "n"(line(1)), "n"(line(2)), "n"(line(3)), "n"(line(4)), "n"(line(5)));
}

// A store that goes through the L2 to memory at once (sc1).  An ordinary one, nontemporal or not, leaves a line that the end of the
// kernel has to write back, since other XCDs may read it next, and the launch behind waits for that: 4.2 MB from 256 workgroups take
// 1.87 us so and 2.31 with ordinary stores, 16.8 MB 3.43 and 4.64 (nontemporal 3.75), 231 MB 35.4 and 37.3; what the same XCD reads
// next is in its L2 either way.  Pieces of a line do not meet in the L2 first, so this is for wavefronts that write at least 64
// aligned consecutive bytes at a time, or 128 at any address (64 bytes per quad of lanes 2.18 us, ordinary 2.34; 32 bytes 4.30,
// 2.99; 128 bytes off four 2.35, 2.46, nontemporal 2.83).  Those are buffers that the last-level cache holds: beyond it pieces go to memory one by one, and large
// results are better left to the L2 or the nontemporal hint (the rules stand where it is called).  The asm says nothing of memory: no kernel reads what it writes so.
template <typename T>
__device__ __forceinline__ void store_through(void* dst, T v) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8 || sizeof(T) == 16, "one store");
  if constexpr (sizeof(T) == 4) asm volatile("global_store_dword %0, %1, off sc1" ::"v"(dst), "v"(v));
  else if constexpr (sizeof(T) == 8) asm volatile("global_store_dwordx2 %0, %1, off sc1" ::"v"(dst), "v"(v));
  else asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(dst), "v"(v));  // (two wait states before its data registers are written again)
}

// 16 bytes at any address, through the L2 or (pieces of a line meet there first) not; `through` is uniform.
__device__ __forceinline__ void store16(bool through, void* dst, uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  typedef uint32_t v4u __attribute__((ext_vector_type(4)));
  typedef v4u v4u_any __attribute__((aligned(1)));
  const v4u v = {a, b, c, d};
  if (through) store_through(dst, v);
  else *static_cast<v4u_any*>(dst) = v;
}

// median of three = clamp when lo <= hi; one instruction instead of two compare/select pairs
__device__ __forceinline__ int32_t med3(int32_t x, int32_t lo, int32_t hi) {
  int32_t r;
  asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(lo), "v"(hi));
  return r;
}

__device__ __forceinline__ int32_t requant_one(int32_t acc, int32_t mult, int32_t sh,
                                               const RequantScalars& rs) {
  const int32_t r = rounding_mul_shift(acc, mult, sh);
  return med3(r, rs.lo_rel, rs.hi_rel) + rs.z_out;
}

// Nearest with halves away from zero: round the magnitude half up and give the sign back,
// which for a negative product is floor((product + rounding term - 1) / 2^(31 + sh)).  The
// product has the sign of acc (mult >= 0; a zero product rounds to 0 either way), so the
// correction is acc's sign bit added to the 64-bit sum.  It differs from ties toward +infinity
// exactly on negative ties, and there by one.
__device__ __forceinline__ int32_t requant_half_away(int32_t acc, int32_t mult, int32_t sh,
                                                     const RequantScalars& rs) {
  const int64_t p = (int64_t)acc * (int64_t)mult + ((int64_t)1 << (30 + sh)) + (int64_t)(acc >> 31);
  return med3((int32_t)(p >> (31 + sh)), rs.lo_rel, rs.hi_rel) + rs.z_out;
}

// The general form, with the launch's tie rule.
__device__ __forceinline__ int32_t requant_general(int32_t acc, int32_t mult, int32_t sh,
                                                   const RequantScalars& rs) {
  return rs.half_away ? requant_half_away(acc, mult, sh, rs) : requant_one(acc, mult, sh, rs);
}

// Byte B of dst <- low byte of (src >> sh) (arithmetic); B == 0 clears the other bytes, the
// later ones keep them: four of these in a row shift and pack four results with no separate
// pack instructions (the destination-byte select of the sub-dword addressing forms).
template <int B>
__device__ __forceinline__ void ashr_into_byte(uint32_t& dst, int32_t src, int32_t sh) {
  static_assert(B >= 0 && B < 4, "byte index");
  if constexpr (B == 0)
    asm("v_ashrrev_i32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:DWORD"
        : "=v"(dst) : "v"(sh), "v"(src));
  else if constexpr (B == 1)
    asm("v_ashrrev_i32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD"
        : "+v"(dst) : "v"(sh), "v"(src));
  else if constexpr (B == 2)
    asm("v_ashrrev_i32_sdwa %0, %1, %2 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD"
        : "+v"(dst) : "v"(sh), "v"(src));
  else
    asm("v_ashrrev_i32_sdwa %0, %1, %2 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD"
        : "+v"(dst) : "v"(sh), "v"(src));
}

// Bytes 2 HALF and 2 HALF + 1 of dst <- a >> sh and b >> sh, saturated to int8; the other two bytes stay.  Shift, clip to the
// whole range and pack of two results in one instruction of 8.5 cycles on a SIMD, against 2.7 + 4.3 for the shift and the
// clip of one and 4.5 for each byte permute that packs them (measured with four wavefronts on every SIMD).
template <int HALF>
__device__ __forceinline__ void ashr_sat_pair(uint32_t& dst, int32_t a, int32_t b, int32_t sh) {
  if constexpr (HALF == 0)
    asm("v_ashr_pk_i8_i32 %0, %1, %2, %3" : "=v"(dst) : "v"(a), "v"(b), "v"(sh));
  else
    asm("v_ashr_pk_i8_i32 %0, %1, %2, %3 op_sel:[0,0,0,1]" : "+v"(dst) : "v"(a), "v"(b), "v"(sh));
}

// v, unknown to the optimizer.  Where several forms of an epilogue follow one another, it widens the factors of their
// products to 64 bits once, in front of all, and the products then take a full 64 x 64 multiply instead of v_mad_i64_i32.
__device__ __forceinline__ int32_t opaque(int32_t v) {
  asm("" : "+v"(v));
  return v;
}

// d[t] of lane r of a quad <-> d[r] of its lane t (every lane of the quad takes part).  Where a lane holds 16 bytes of each of
// four pieces of a row, the quad's stores then write 64 consecutive bytes: 64 cycles of the memory pipe for a wavefront's 16
// bytes per lane, against 168 where every lane writes to a line of its own and 256 off four bytes.
template <int D>
__device__ __forceinline__ void quad_transpose(uint32_t (&d)[4][D], int lane) {
  auto exchange = [&]<int CTRL>(uint32_t& lower, uint32_t& upper, bool high) {
    const uint32_t from_upper = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)upper, CTRL, 0xf, 0xf, true);
    const uint32_t from_lower = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lower, CTRL, 0xf, 0xf, true);
    lower = high ? from_upper : lower;
    upper = high ? upper : from_lower;
  };
#pragma unroll
  for (int k = 0; k < D; ++k) {
    exchange.template operator()<0xB1>(d[0][k], d[1][k], lane & 1);  // quad_perm 1,0,3,2
    exchange.template operator()<0xB1>(d[2][k], d[3][k], lane & 1);
    exchange.template operator()<0x4E>(d[0][k], d[2][k], lane & 2);  // quad_perm 2,3,0,1
    exchange.template operator()<0x4E>(d[1][k], d[3][k], lane & 2);
  }
}

// v; what follows from it is computed where it is used, not in front of the loop around
__device__ __forceinline__ int stay_here(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// The upper sixteen lanes of each half of the wavefront give their a to, and take b from, the lower ones: sixteen lanes then hold, of
// their channel in a and of the one sixteen further on in b, what is a in the lower sixteen and b in the upper ones.  Lanes i, i + 16,
// i + 32 and i + 48 write 64 consecutive bytes of a channel so.
__device__ __forceinline__ void swap_sixteens(uint32_t (&a)[4], uint32_t (&b)[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const auto s = __builtin_amdgcn_permlane16_swap(a[k], b[k], false, false);
    a[k] = s[0], b[k] = s[1];
  }
}

// Whether the output's clip limits are its container's whole range, so that this saturation is the clip.  sat_bias is added
// to the output zero point (inside the 64-bit constant of the folded forms) to centre the range on int8's, and sat_flip
// undoes it in the packed dword: 0 and 0 for int8, -128 and 0x80 per byte for uint8.
__host__ __device__ __forceinline__ bool sat_range(const RequantScalars& rs) { return rs.hi_rel - rs.lo_rel == 255; }
__device__ __forceinline__ int32_t sat_bias(const RequantScalars& rs) { return -128 - (rs.lo_rel + rs.z_out); }
__device__ __forceinline__ uint32_t sat_flip(const RequantScalars& rs) { return rs.lo_rel + rs.z_out == 0 ? 0x80808080u : 0u; }

// Clip limits moved in front of a right shift by s: clip(y >> s, lo, hi) == clip(y, lo * 2^s,
// (hi + 1) * 2^s - 1) >> s for the flooring shift; a limit that leaves int32 saturates there
// (no y lies beyond it, so it is inactive, as it should be).
__device__ __forceinline__ int32_t clip_lo_before_shift(int32_t lo, int32_t s) {
  const int64_t v = (int64_t)lo * ((int64_t)1 << s);
  return v < INT32_MIN ? INT32_MIN : (v > INT32_MAX ? INT32_MAX : (int32_t)v);
}
__device__ __forceinline__ int32_t clip_hi_before_shift(int32_t hi, int32_t s) {
  const int64_t v = ((int64_t)hi + 1) * ((int64_t)1 << s) - 1;
  return v > INT32_MAX ? INT32_MAX : (v < INT32_MIN ? INT32_MIN : (int32_t)v);
}

// Four results -> one little-endian dword of their low bytes.
__device__ __forceinline__ uint32_t pack4_perm(int32_t b0, int32_t b1, int32_t b2, int32_t b3) {
  const uint32_t lo = __builtin_amdgcn_perm((uint32_t)b1, (uint32_t)b0, 0x0c0c0400u);
  const uint32_t hi = __builtin_amdgcn_perm((uint32_t)b3, (uint32_t)b2, 0x04000c0cu);
  return lo | hi;
}

__device__ __forceinline__ uint32_t pack4(int32_t b0, int32_t b1, int32_t b2, int32_t b3) {
  return (uint32_t)(b0 & 0xff) | ((uint32_t)(b1 & 0xff) << 8) | ((uint32_t)(b2 & 0xff) << 16) |
         ((uint32_t)b3 << 24);
}

}  // namespace hago
