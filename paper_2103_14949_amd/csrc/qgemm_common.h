// Pieces shared by the two int8-MFMA GEMM kernels (register-staged generic
// kernel and the LDS-DMA dense kernel): launch parameters, the per-tile
// channel terms and the requantize/store epilogue.
#pragma once

#include "hago_device.h"
#include "launch.h"

#include <cstdlib>

namespace hago {

#ifdef HAGO_PHASE_TIMING
#ifdef HAGO_STAMP_CYCLES
#define HAGO_STAMP_CLOCK clock64       // shader clock cycles
#else
#define HAGO_STAMP_CLOCK wall_clock64  // 100 MHz
#endif
#define HAGO_STAMP(p, i) do { if (threadIdx.x == 0 && (p).dbg) (p).dbg[blockIdx.x * 8 + (i)] = HAGO_STAMP_CLOCK(); } while (0)
#else
#define HAGO_STAMP(p, i) do { } while (0)
#endif

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v4i_any __attribute__((ext_vector_type(4), aligned(1)));
typedef int v16i __attribute__((ext_vector_type(16)));

#ifdef HAGO_PHASE_TIMING
// development builds only: where the kernels write their phase timestamps (set by the timing driver)
inline long long* g_stamp_buffer = nullptr;
inline int g_stamp_skip = 0;
#endif

struct QgemmParams {
  const uint8_t* act;
  const int8_t* wgt;
  const int32_t* bias;
  void* out;
  const int32_t* mult;
  const int32_t* shift;
  int32_t M, N, K;
  int32_t per_channel, has_rq, acc16;
  int32_t acc_wrap_shift;  // 32 - accumulator bits (0, 16 or 8)
  int32_t out_mode;    // 0: requantized 8-bit, 1: raw int32, 2: raw int16
  uint32_t act_xor4;   // 0x80808080 for uint8 activations, else 0
  int32_t corr_coef;   // off - z_a
  uint32_t pad_byte;   // staged value of a padded tap: (z_a XOR act_xor) & 0xff
  int32_t vec_k;       // rows of both operands can be read as aligned 16-byte chunks
  int32_t vec_out;     // NCHW: four consecutive pixels lie in one image and form one aligned store
  int32_t line_out;    // dense: every 64th result of a row begins a line of 64 bytes
  RequantScalars rs;
  ConvGeom g;
  int32_t tile0;       // first tile of this launch (a problem of many tiles takes several)
  // implicit GEMM over a prepacked copy: its byte size and ceil(2^32 / C), ceil(2^32 / KW)
  uint32_t act_bytes, inv_c, inv_kw;
  // implicit GEMM over the caller's tensor: ceil(2^32 / (OH OW)) and of OW where that divides exactly, else 0
  uint32_t inv_ohw, inv_ow;
#ifdef HAGO_PHASE_TIMING
  long long* dbg;  // per-workgroup phase timestamps (development builds only)
  int dbg_skip;    // bit mask of main-loop parts to leave out in timing experiments
#endif
};

inline QgemmParams make_qgemm_params(const GemmArgs& a, const ConvGeom* cg) {
  QgemmParams p{};
  p.act = static_cast<const uint8_t*>(a.act);
  p.wgt = a.wgt;
  p.bias = a.bias;
  p.out = a.out;
  p.mult = a.rq.multiplier;
  p.shift = a.rq.shift;
  p.M = a.M; p.N = a.N; p.K = a.K;
  p.per_channel = a.rq.per_channel;
  p.has_rq = a.has_rq;
  p.acc16 = a.acc16;
  p.acc_wrap_shift = a.acc_wrap_shift;
  p.out_mode = a.has_rq ? 0 : (a.acc16 ? 2 : 1);
  p.act_xor4 = a.act_unsigned ? 0x80808080u : 0u;
  p.corr_coef = (a.act_unsigned ? 128 : 0) - a.act_zero_point;
  p.pad_byte = ((uint32_t)a.act_zero_point ^ (a.act_unsigned ? 0x80u : 0u)) & 0xffu;
  p.rs = RequantScalars{a.rq.z_out, a.rq.clip_lo - a.rq.z_out, a.rq.clip_hi - a.rq.z_out, a.rq.half_away};
  if (cg) p.g = *cg;
#ifdef HAGO_PHASE_TIMING
  p.dbg = g_stamp_buffer;
  p.dbg_skip = g_stamp_skip;
#endif
  return p;
}

inline size_t qgemm_out_elem_size(const GemmArgs& a) { return a.has_rq ? 1 : (a.acc16 ? 2 : 4); }

// Turn the weight row sums that sit in s_corr[0..CH) into the per-channel
// terms of the tile: corr = bias + (off - z_a) * sum_k w, multiplier, shift.
// Channels beyond N get zeros.  Ends with a barrier.
template <int NT, int CH>
__device__ __forceinline__ void stage_channel_terms(const QgemmParams& p, int w0, int32_t* s_corr,
                                                    int32_t* s_mult, int32_t* s_shift) {
  const int t = threadIdx.x;
  for (int ci = t; ci < CH; ci += NT) {
    const int n = w0 + ci;
    int32_t corr = 0, mu = 0, sh = 0;
    if (n < p.N) {
      corr = (p.bias ? p.bias[n] : 0) + p.corr_coef * s_corr[ci];
      if (p.has_rq) {
        mu = rq_mult(p.mult, p.per_channel ? n : 0);
        sh = rq_shift(p.mult, p.shift, p.per_channel ? n : 0);
      }
    }
    s_corr[ci] = corr;
    s_mult[ci] = mu;
    s_shift[ci] = sh;
  }
  __syncthreads();
}

// Per-channel epilogue inputs fetched at kernel start (so that their latency hides
// behind the main loop); one slot per channel this lane is responsible for.
template <int NT, int CH>
struct ChannelRegs {
  static constexpr int kSlots = (CH + NT - 1) / NT;
  int32_t bias[kSlots], mult[kSlots], shift[kSlots];
};

template <int NT, int CH>
__device__ __forceinline__ void load_channel_regs(const QgemmParams& p, int w0, ChannelRegs<NT, CH>& r) {
#pragma unroll
  for (int s = 0; s < ChannelRegs<NT, CH>::kSlots; ++s) {
    const int ci = (int)threadIdx.x + NT * s;
    const int n = w0 + ci;
    r.bias[s] = 0; r.mult[s] = 0; r.shift[s] = 1;
    if (ci < CH && n < p.N) {
      if (p.bias) r.bias[s] = p.bias[n];
      if (p.has_rq) {
        r.mult[s] = rq_mult(p.mult, p.per_channel ? n : 0);
        r.shift[s] = rq_shift(p.mult, p.shift, p.per_channel ? n : 0);
      }
    }
  }
}

// Forms of a staged tile's requantize arithmetic.
//   kRqGeneral: any shift, any correction.
//   kRqFolded: (acc + corr) * mult + rounding term is one 64-bit multiply-add with the channel's constant, and the result is
//     its high dword shifted right.
//   kRqSat: the same with the output zero point in the constant, for outputs clipped to their container's whole range:
//     shift, clip and pack of two results are one instruction (ashr_sat_pair).
enum { kRqGeneral, kRqFolded, kRqSat };

// Results of a kernel, which has the forms for them alone: what other forms need is code that the compiler puts in front of all of them
// and that a launch of one tile per CU waits for (us in one kernel and so: the four layers of 4096 x 768 51.3, 50.9; 3000 x 128 -> 1001 5.19, 5.07; 8192 x 64 -> 1024 6.42,
// 6.27; the channel-last bottleneck of 16 x 28 x 28 x 256 12.8, 12.6).
//   kOutFull: one byte, clipped to its whole range, of a 32-bit accumulator, rounding half up, an output zero point that kRqSat takes; kRqFolded
//     beside it for tiles with a shift above 21 (us in the general form and so: 4096 x 768 -> 2304 13.1, 12.4; 8192 x 64 -> 1024 7.15, 6.75; tiles
//     without the same);
//   kOutClipped: the same but for the clip or the zero point; both leave the tile in LDS first.
//   kOutOther: what the straight-line epilogue writes.
enum { kOutFull, kOutClipped, kOutOther };
inline bool qgemm_full_codes(const QgemmParams& p) {
  return p.out_mode == 0 && !p.rs.half_away && sat_range(p.rs) && p.rs.z_out >= -128 && p.rs.z_out <= 255;
}
inline int qgemm_out(const QgemmParams& p) {
  if (p.out_mode != 0 || p.acc_wrap_shift || p.rs.half_away) return kOutOther;
  return qgemm_full_codes(p) ? kOutFull : kOutClipped;
}

// s_corr holds the weight row sums on entry (s_sum2, if given, a second part to add; it may be
// s_mult); on exit s_corr/s_mult/s_shift hold the
// per-channel terms and s_c64 the folded addend corr * mult + 2^(30+shift), with which
// (acc + corr) * mult + rounding term is one 64-bit multiply-add per element.
// Returns (block-uniform) the arithmetic the tile takes.  It needs the general one if some channel has
// shift 0 (the result is then not the high dword shifted right), or a correction so large
// that acc + corr could leave int32 (whose wrap-around the folded form would not reproduce;
// |acc| <= K * 2^14 < 2^30 for K <= 2^16).  kRqSat: shifts up to 21 too (products and correction are below 2^61, the zero
// point's 9 bits shifted by 31 + 21 below 2^61 as well).
// s_vote: zero on entry.  The workgroup's vote is one word of LDS and one barrier (by __syncthreads_or, which has three, small
// calls took 0.1 us longer: 170 x 64 -> 128 3.20, 3.09 so).
template <int NT, int CH, int OUT>
__device__ __forceinline__ int finish_channel_terms(const QgemmParams& p, const ChannelRegs<NT, CH>& r,
                                                    int32_t* s_corr, int32_t* s_mult,
                                                    int32_t* s_shift, int64_t* s_c64, int32_t* s_vote,
                                                    const int32_t* s_sum2 = nullptr,
                                                    int32_t* s_shm1 = nullptr) {
  if constexpr (OUT == kOutOther) {  // (raw 6132 x 640 -> 192 6.0 us through the vote below, 5.4 so)
#pragma unroll
    for (int s = 0; s < ChannelRegs<NT, CH>::kSlots; ++s) {
      const int ci = (int)threadIdx.x + NT * s;
      if (ci < CH) {
        s_corr[ci] = r.bias[s] + p.corr_coef * (s_corr[ci] + (s_sum2 ? s_sum2[ci] : 0));
        if (p.out_mode == 0) s_mult[ci] = r.mult[s], s_shift[ci] = r.shift[s];
      }
    }
    __syncthreads();
    return kRqGeneral;
  }
  const int32_t z = p.rs.z_out;
  constexpr bool sat = OUT == kOutFull;
  const int32_t zc = sat ? z + sat_bias(p.rs) : 0;
  int general = p.K > 65536, high = 0;
#pragma unroll
  for (int s = 0; s < ChannelRegs<NT, CH>::kSlots; ++s) {
    const int ci = (int)threadIdx.x + NT * s;
    if (ci < CH) {
      const int32_t wsum = s_corr[ci] + (s_sum2 ? s_sum2[ci] : 0);
      const int32_t corr = r.bias[s] + p.corr_coef * wsum;
      s_corr[ci] = corr;
      s_mult[ci] = r.mult[s];
      s_shift[ci] = r.shift[s];
      if (s_shm1) s_shm1[ci] = r.shift[s] - 1;  // the folded forms shift the high dword by this
      s_c64[ci] = (int64_t)corr * (int64_t)r.mult[s] + ((int64_t)1 << (30 + (r.shift[s] & 31))) +
                  (sat ? (int64_t)zc << (31 + (r.shift[s] & 31)) : 0);
      general |= (r.shift[s] <= 0) | (corr >= (1 << 30)) | (corr <= -(1 << 30));
      high |= r.shift[s] > 21;
    }
  }
  const uint64_t any_general = __builtin_amdgcn_ballot_w64(general != 0), any_high = __builtin_amdgcn_ballot_w64(high != 0);
  if ((any_general | any_high) != 0 && (threadIdx.x & 63) == 0) atomicOr(s_vote, (any_general ? 1 : 0) | (any_high ? 2 : 0));
  __syncthreads();
  const int vote = __builtin_amdgcn_readfirstlane(*s_vote);
  if (sat) {
    if (vote == 0) return kRqSat;
#pragma unroll
    for (int s = 0; s < ChannelRegs<NT, CH>::kSlots; ++s) {
      const int ci = (int)threadIdx.x + NT * s;
      if (ci < CH) s_c64[ci] = (int64_t)s_corr[ci] * (int64_t)r.mult[s] + ((int64_t)1 << (30 + (r.shift[s] & 31)));
    }
    __syncthreads();
  }
  return vote & 1 ? kRqGeneral : kRqFolded;
}

// r = floor((a * m + 2^(30+sh)) / 2^(31+sh)).  With SH_GE1 (sh >= 1) the shift
// distance is at least 32, so the result is the high dword shifted by sh - 1:
// one 32-bit shift instead of a 64-bit one.
template <bool SH_GE1>
__device__ __forceinline__ int32_t mul_shift_fast(int32_t a, int32_t m, int64_t rnd, int32_t sh) {
  const int64_t pr = (int64_t)a * (int64_t)m + rnd;
  if constexpr (SH_GE1) return (int32_t)(pr >> 32) >> (sh - 1);
  return (int32_t)(pr >> (31 + sh));
}

// Dense epilogue of a tile (interior or ragged) through LDS: requantize, pack four channels
// per dword, write the tile to LDS in output order [row m][channel n], then copy
// it out with 16-byte stores that cover whole output rows, at whatever byte those start (rows of 1001 results stored one by
// one from the registers: 64 x 256 -> 129 6.1 us, 3.6 so; 4096 x 768 -> 3070 49, 17).  LDS rows are BP + 16 bytes
// apart, so the 32 rows a wavefront writes at once spread over the banks.
// s_out: BQ * (BP + 16) bytes.  FORM: see finish_channel_terms.
// Bound by vector-ALU issue.  kRqSat: 4.7 cycles of a SIMD for an output's multiply-add, 4.3 for its half of a saturating
// shift of two rows of a channel, 1.1 for the permutes that sort the pairs into rows (10.1; 11.6 where a wavefront has one
// row block, and shifts before it packs), against 14.6 for multiply-add, shift, clip and pack one by one.
template <int WP, int WQ, int TP, int TQ, int FORM>
__device__ __forceinline__ void qgemm_epilogue_dense_staged(const QgemmParams& p,
                                                            v16i (&acc)[TP][TQ], int p0, int q0,
                                                            const int32_t* s_corr,
                                                            const int32_t* s_mult,
                                                            const int32_t* s_shift,
                                                            const int64_t* s_c64,
                                                            const int32_t* s_shm1,
                                                            uint8_t* s_out) {
  constexpr int NT = 64 * WP * WQ;
  constexpr int BP = WP * TP * 32, BQ = WQ * TQ * 32;
  constexpr int CPR = BP / 16;   // 16-byte chunks per tile row
  constexpr int RS = BP + 16;    // LDS row stride
  constexpr bool FOLDED = FORM != kRqGeneral;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wp = wave % WP, wq = wave / WP;
  const int frow = lane & 31, fhalf = lane >> 5;
  const uint32_t sflip = sat_flip(p.rs);
  int32_t lo = p.rs.lo_rel, hi = p.rs.hi_rel;
  const int32_t z = p.rs.z_out;
  // v_med3 takes one scalar operand at most: keep the bounds in vector registers once
  asm volatile("" : "+v"(lo), "+v"(hi));
  uint8_t* my_row = s_out + ((wq * TQ) * 32 + frow) * RS + wp * TP * 32 + fhalf * 4;
  // Per-channel terms of group g = (ti, g4): four consecutive channels.  The terms of the next
  // group are fetched while the current one is computed, and no further ahead (fetching all
  // groups up front would cost more registers than the accumulators leave).
  struct Terms { int4 m4, s4, c4; longlong2 ca, cb; };
  auto load_terms = [&](int g) {
    const int i_loc = (wp * TP + g / 4) * 32 + (g % 4) * 8 + fhalf * 4;
    Terms t;
    t.m4 = *reinterpret_cast<const int4*>(s_mult + i_loc);
    t.s4 = *reinterpret_cast<const int4*>((FOLDED ? s_shm1 : s_shift) + i_loc);
    if constexpr (FOLDED) {
      t.ca = *reinterpret_cast<const longlong2*>(s_c64 + i_loc);
      t.cb = *reinterpret_cast<const longlong2*>(s_c64 + i_loc + 2);
    } else {
      t.c4 = *reinterpret_cast<const int4*>(s_corr + i_loc);
    }
    return t;
  };
  Terms cur = load_terms(0);
#pragma unroll
  for (int g = 0; g < TP * 4; ++g) {
    const int ti = g / 4, g4 = g % 4;
    Terms nxt = cur;
    if (g + 1 < TP * 4) nxt = load_terms(g + 1);
    __builtin_amdgcn_sched_barrier(0);
    const int32_t mm[4] = {cur.m4.x, cur.m4.y, cur.m4.z, cur.m4.w};
    const int32_t ss[4] = {cur.s4.x, cur.s4.y, cur.s4.z, cur.s4.w};
    int32_t r[TQ][4];
    if constexpr (FOLDED) {
      const int64_t c64[4] = {cur.ca.x, cur.ca.y, cur.cb.x, cur.cb.y};
#pragma unroll
      for (int tj = 0; tj < TQ; ++tj)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t pr = (int64_t)acc[ti][tj][g4 * 4 + e] * (int64_t)mm[e] + c64[e];
          r[tj][e] = (int32_t)(pr >> 32);
          // (ss = shift - 1 here; kRqSat shifts row blocks two at a time below)
          if (FORM != kRqSat || (tj == TQ - 1 && TQ % 2 == 1)) r[tj][e] >>= ss[e];
        }
    } else {
      const int32_t cc[4] = {cur.c4.x, cur.c4.y, cur.c4.z, cur.c4.w};
#pragma unroll
      for (int tj = 0; tj < TQ; ++tj)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          r[tj][e] = mul_shift_fast<false>(acc[ti][tj][g4 * 4 + e] + cc[e], mm[e],
                                           (int64_t)1 << (30 + ss[e]), ss[e]);
    }
    if constexpr (FORM == kRqSat) {
      auto put = [&](int tj, uint32_t dw) { *reinterpret_cast<uint32_t*>(my_row + tj * 32 * RS + ti * 32 + g4 * 8) = dw ^ sflip; };
#pragma unroll
      for (int tj = 0; tj + 1 < TQ; tj += 2) {
        uint32_t d01, d23;  // channels 0, 1 and 2, 3: rows tj and tj + 1 of each
        ashr_sat_pair<0>(d01, r[tj][0], r[tj + 1][0], ss[0]);
        ashr_sat_pair<0>(d23, r[tj][2], r[tj + 1][2], ss[2]);
        ashr_sat_pair<1>(d01, r[tj][1], r[tj + 1][1], ss[1]);
        ashr_sat_pair<1>(d23, r[tj][3], r[tj + 1][3], ss[3]);
        put(tj, __builtin_amdgcn_perm(d23, d01, 0x06040200u));
        put(tj + 1, __builtin_amdgcn_perm(d23, d01, 0x07050301u));
      }
      if constexpr (TQ % 2 == 1) {
        uint32_t dw;
        ashr_sat_pair<0>(dw, r[TQ - 1][0], r[TQ - 1][1], 0);
        ashr_sat_pair<1>(dw, r[TQ - 1][2], r[TQ - 1][3], 0);
        put(TQ - 1, dw);
      }
      __builtin_amdgcn_sched_barrier(0);
      cur = nxt;
      continue;
    }
#pragma unroll
    for (int tj = 0; tj < TQ; ++tj) {
      int32_t r0 = med3(r[tj][0], lo, hi), r1 = med3(r[tj][1], lo, hi);
      int32_t r2 = med3(r[tj][2], lo, hi), r3 = med3(r[tj][3], lo, hi);
      if (z != 0) { r0 += z; r1 += z; r2 += z; r3 += z; }
      *reinterpret_cast<uint32_t*>(my_row + tj * 32 * RS + ti * 32 + g4 * 8) =
          pack4_perm(r0, r1, r2, r3);
    }
    __builtin_amdgcn_sched_barrier(0);
    cur = nxt;
  }
  __syncthreads();
  HAGO_STAMP(p, 5);
  uint8_t* out8 = static_cast<uint8_t*>(p.out);
  const bool ragged = q0 + BQ > p.M || p0 + BP > p.N;  // block-uniform
  // Up to 4 MB of results of rows of whole lines go through the L2, more and others carry the nontemporal hint, unless they are narrow and do not begin with
  // a line.  Us through the L2 and with the hint, from the last-level cache and on buffers beyond it: 12544 x 64 -> 256 4.40, 4.60 and 4.67, 4.97; 6000 x
  // 64 -> 512 4.00, 4.33 and 4.44, 4.74; 4096 x 768 -> 768 6.67, 6.86 and 8.06, 7.96; but 2048 x 768 -> 2304 8.86, 9.03 and 11.4, 9.7; 4096 x 768 -> 2304
  // 11.9, 11.9 and 13.7, 12.0; 8192 x 512 -> 1536 10.9, 11.0 and 15.6, 11.5; 3000 x 768 -> 2001 10.5, 10.6 and 14.1, 11.2.  (Left in the L2 4096 x 768 -> 2304
  // 12.7 and 14.9.)
  const bool through = p.line_out && (uint64_t)(uint32_t)p.M * (uint32_t)p.N <= 4000000u;
  const bool stream = BP >= 128 || p.line_out;
#pragma unroll
  for (int s = 0; s < (BQ * CPR) / NT; ++s) {
    const int q = (int)threadIdx.x + NT * s;
    const int row = q / CPR, c = q % CPR;
    const v4i v = *reinterpret_cast<const v4i*>(s_out + row * RS + c * 16);
    // ragged tiles: rows beyond M and channels beyond N stay in LDS
    if (ragged && (q0 + row >= p.M || p0 + c * 16 >= p.N)) continue;
    uint8_t* dst = out8 + (size_t)(q0 + row) * p.N + p0 + c * 16;
    if (p0 + c * 16 + 16 <= p.N) {
      if (through) store_through(dst, v);
      else if (stream) __builtin_nontemporal_store(v, reinterpret_cast<v4i_any*>(dst));
      else *reinterpret_cast<v4i_any*>(dst) = v;  // (pieces of a line meet in L2)
    } else {  // the row's last channels
      const int left = p.N - p0 - c * 16;
      uint32_t w[4] = {(uint32_t)v.x, (uint32_t)v.y, (uint32_t)v.z, (uint32_t)v.w};
#pragma unroll
      for (int e = 0; e < 15; ++e)
        if (e < left) dst[e] = (uint8_t)(w[e >> 2] >> (8 * (e & 3)));
    }
  }
  HAGO_STAMP(p, 6);
}

// Four results of one output row, channels n .. n + 3, where they exist.  Raw int32 ones go through the L2 where they are
// aligned: eight lanes write 128 bytes of a row.
template <bool RQ>
__device__ __forceinline__ void store_four(const QgemmParams& p, int m, int n, const int32_t (&v)[4]) {
  const int out_mode = RQ ? 0 : (p.out_mode == 1 ? 1 : 2);
  const int64_t o = (int64_t)m * p.N + n;
  if (n + 4 <= p.N) {
    if (out_mode == 0) {
      typedef uint32_t u32_any __attribute__((aligned(1)));
      *reinterpret_cast<u32_any*>(static_cast<uint8_t*>(p.out) + o) = pack4_perm(v[0], v[1], v[2], v[3]);
    } else if (out_mode == 1) {
      const bool through = (p.N & 3) == 0 && (reinterpret_cast<uintptr_t>(p.out) & 15u) == 0;
      store16(through, static_cast<int32_t*>(p.out) + o, (uint32_t)v[0], (uint32_t)v[1], (uint32_t)v[2], (uint32_t)v[3]);
    } else {
      typedef int v2i_any __attribute__((ext_vector_type(2), aligned(1)));
      *reinterpret_cast<v2i_any*>(static_cast<int16_t*>(p.out) + o) =
          v2i_any{(int)(((uint32_t)v[0] & 0xffffu) | ((uint32_t)v[1] << 16)), (int)(((uint32_t)v[2] & 0xffffu) | ((uint32_t)v[3] << 16))};
    }
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (n + e >= p.N) break;
    if (out_mode == 0) static_cast<uint8_t*>(p.out)[o + e] = (uint8_t)v[e];
    else if (out_mode == 1) static_cast<int32_t*>(p.out)[o + e] = v[e];
    else static_cast<int16_t*>(p.out)[o + e] = (int16_t)v[e];
  }
}

// Straight-line epilogue of a tile (interior or ragged): groups of four along the packed axis are one store, in a dense
// tile at any address and cut where the row ends, else aligned and inside the tensor or outside.
// OM: 0 requantized 8-bit, 1 raw int32, 2 raw int16.
template <int OM>
__device__ __forceinline__ void store_group(void* out, size_t off, int32_t v0, int32_t v1,
                                            int32_t v2, int32_t v3) {
  typedef uint32_t u32_any __attribute__((aligned(1)));
  typedef short v4s_any __attribute__((ext_vector_type(4), aligned(1)));
  if constexpr (OM == 0)
    *reinterpret_cast<u32_any*>(static_cast<uint8_t*>(out) + off) = pack4(v0, v1, v2, v3);
  else if constexpr (OM == 1)
    *reinterpret_cast<v4i_any*>(static_cast<int32_t*>(out) + off) = v4i{v0, v1, v2, v3};
  else
    *reinterpret_cast<v4s_any*>(static_cast<int16_t*>(out) + off) = v4s_any{(short)v0, (short)v1, (short)v2, (short)v3};
}
// The first n results of a group.
template <int OM>
__device__ __forceinline__ void store_some(void* out, size_t off, const int32_t (&v)[4], int n) {
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    if (e >= n) break;
    if constexpr (OM == 0) static_cast<uint8_t*>(out)[off + e] = (uint8_t)v[e];
    else if constexpr (OM == 1) static_cast<int32_t*>(out)[off + e] = v[e];
    else static_cast<int16_t*>(out)[off + e] = (int16_t)v[e];
  }
}

template <int OM, bool AWAY>
__device__ __forceinline__ int32_t finish_one(int32_t a, int32_t m, int32_t sh, int32_t acc16,
                                              const RequantScalars& rs) {
  if (acc16) a = wrap_acc_bits(a, acc16);  // (the wrap shift of a narrow accumulator, 0 for int32)
  if constexpr (OM == 0) a = AWAY ? requant_half_away(a, m, sh, rs) : requant_one(a, m, sh, rs);
  return a;
}

// Row r of a 32-row block holds pixel pix_perm(r) of the block when the loader placed the pixels
// that way (PIXPERM): registers 4g + e of lane half h are then the 16 consecutive pixels
// 16h + 4g + e, which go out as one 16-byte store per channel instead of four scattered dwords.
__device__ __forceinline__ constexpr int pix_perm(int r) {
  return 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3);
}

// Tiles inside the matrix store without a check, tiles that end with it check every group of four, and only where the packed
// extent is no multiple of four is a group cut (checking for that everywhere: raw results of 2 x 16 -> 16 3.1 us, 2.8 so;
// 6132 x 640 -> 192 6.1, 5.6).
enum { kInside, kWholeGroups, kCutGroups };

template <int WP, int WQ, int TP, int TQ, bool ACT_ON_P, int OM, bool PIXPERM, int EDGE, bool AWAY>
__device__ __forceinline__ void qgemm_epilogue_fast(const QgemmParams& p, v16i (&acc)[TP][TQ],
                                                    int p0, int q0, const int32_t* s_corr,
                                                    const int32_t* s_mult,
                                                    const int32_t* s_shift) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wp = wave % WP, wq = wave / WP;
  const int frow = lane & 31, fhalf = lane >> 5;
  const RequantScalars rs = p.rs;
  const int32_t acc16 = p.acc_wrap_shift;
  const int P_ext = ACT_ON_P ? p.M : p.N;
  const int Q_ext = ACT_ON_P ? p.N : p.M;
  if constexpr (OM == 1 && (!ACT_ON_P || PIXPERM)) {
    // Raw int32, bound by its stores: the quads of lanes transpose pieces of 16 bytes and write 64 consecutive ones of a row (of a channel),
    // through the L2 if the pieces are aligned.  Us, a lane's 16 bytes to 32 rows by themselves and so: 4096 x 768 -> 768 9.5, 7.8; -> 2304 19.0, 15.3;
    // 8192 x 64 -> 1024 11.6, 8.55; 3000 x 128 -> 1001 7.6, 6.45; 3x3 through a workspace, 128 -> 128 on 8 x 56 x 56, 11.1, 9.6, channel-last 14.6, 12.4.
    const int at = stay_here(lane), q4 = 4 * (at & 3) + 16 * (at >> 5), jq = at & 28;
    const bool through = ((ACT_ON_P ? 0 : p.N) & 3) == 0 && (reinterpret_cast<uintptr_t>(p.out) & 15u) == 0;
#pragma unroll
    for (int ti = 0; ti < TP; ++ti) {
      const int i = p0 + (wp * TP + ti) * 32 + q4;
      const int b = ACT_ON_P ? i / (p.g.OH * p.g.OW) : 0;
#pragma unroll
      for (int tj = 0; tj < TQ; ++tj) {
        uint32_t v[4][4];
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const int4 c4 = ACT_ON_P ? make_int4(s_corr[(wq * TQ + tj) * 32 + frow], 0, 0, 0)
                                   : *reinterpret_cast<const int4*>(s_corr + (wp * TP + ti) * 32 + g4 * 8 + fhalf * 4);
          const int32_t cc[4] = {c4.x, ACT_ON_P ? c4.x : c4.y, ACT_ON_P ? c4.x : c4.z, ACT_ON_P ? c4.x : c4.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) v[g4][e] = (uint32_t)finish_one<OM, AWAY>(acc[ti][tj][g4 * 4 + e] + cc[e], 0, 0, acc16, rs);
        }
        if constexpr (!ACT_ON_P) {
          // a lane has channels 8 g + 4 half ..; the halves swap groups and then have 16 consecutive ones each
#pragma unroll
          for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int g4 = 0; g4 < 2; ++g4) {
              const auto sw = __builtin_amdgcn_permlane32_swap(v[g4][e], v[g4 + 2][e], false, false);
              v[g4][e] = sw[0], v[g4 + 2][e] = sw[1];
            }
            const uint32_t x = v[1][e];
            v[1][e] = v[2][e], v[2][e] = x;
          }
        }
        quad_transpose(v, lane);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int j = q0 + (wq * TQ + tj) * 32 + jq + t;
          const size_t o = ACT_ON_P ? ((size_t)b * p.N + j) * (size_t)(p.g.OH * p.g.OW) + (size_t)(i - b * (p.g.OH * p.g.OW)) : (size_t)j * p.N + i;
          if (EDGE == kInside || (j < Q_ext && i + (EDGE == kCutGroups ? 4 : 1) <= P_ext))
            store16(through, static_cast<int32_t*>(p.out) + o, v[t][0], v[t][1], v[t][2], v[t][3]);
          else if (EDGE == kCutGroups && j < Q_ext)
            store_some<OM>(p.out, o, {(int32_t)v[t][0], (int32_t)v[t][1], (int32_t)v[t][2], (int32_t)v[t][3]}, P_ext - i);
        }
      }
    }
    return;
  }
  // Raw int16: of 32 bytes per lane the sixteens of lanes swap pieces of 16, and four lanes write 64 consecutive bytes.
  // (3x3 through a workspace, 128 -> 128 on 8 x 56 x 56: 9.7 us before, 9.0 so; channel-last 10.7, 9.3.)
  const bool pieces = OM == 2 && ((ACT_ON_P ? p.g.OH * p.g.OW : p.N) & 7) == 0 && (reinterpret_cast<uintptr_t>(p.out) & 15u) == 0;
  if constexpr (OM == 2 && (!ACT_ON_P || PIXPERM)) {
    if (pieces) {
      const int at = stay_here(lane), q8 = 16 * (at >> 5) + 8 * ((at >> 4) & 1), jq = at & 15;
#pragma unroll
      for (int ti = 0; ti < TP; ++ti) {
        const int i = p0 + (wp * TP + ti) * 32 + q8;
        const int b = ACT_ON_P ? i / (p.g.OH * p.g.OW) : 0;
#pragma unroll
        for (int tj = 0; tj < TQ; ++tj) {
          uint32_t d[4][2];  // (the low sixteen bits are the wrapped sum's for any accumulator of at least that width)
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4) {
            const int4 c4 = ACT_ON_P ? make_int4(s_corr[(wq * TQ + tj) * 32 + frow], 0, 0, 0)
                                     : *reinterpret_cast<const int4*>(s_corr + (wp * TP + ti) * 32 + g4 * 8 + fhalf * 4);
            const int32_t cc[4] = {c4.x, ACT_ON_P ? c4.x : c4.y, ACT_ON_P ? c4.x : c4.z, ACT_ON_P ? c4.x : c4.w};
#pragma unroll
            for (int e = 0; e < 2; ++e)
              d[g4][e] = ((uint32_t)(acc[ti][tj][g4 * 4 + 2 * e] + cc[2 * e]) & 0xffffu) | ((uint32_t)(acc[ti][tj][g4 * 4 + 2 * e + 1] + cc[2 * e + 1]) << 16);
          }
          if constexpr (!ACT_ON_P) {  // as above
#pragma unroll
            for (int e = 0; e < 2; ++e) {
#pragma unroll
              for (int g4 = 0; g4 < 2; ++g4) {
                const auto sw = __builtin_amdgcn_permlane32_swap(d[g4][e], d[g4 + 2][e], false, false);
                d[g4][e] = sw[0], d[g4 + 2][e] = sw[1];
              }
              const uint32_t x = d[1][e];
              d[1][e] = d[2][e], d[2][e] = x;
            }
          }
          uint32_t dq[2][4] = {{d[0][0], d[0][1], d[1][0], d[1][1]}, {d[2][0], d[2][1], d[3][0], d[3][1]}};
          swap_sixteens(dq[0], dq[1]);
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            const int j = q0 + (wq * TQ + tj) * 32 + 16 * g + jq;
            const size_t o = ACT_ON_P ? ((size_t)b * p.N + j) * (size_t)(p.g.OH * p.g.OW) + (size_t)(i - b * (p.g.OH * p.g.OW)) : (size_t)j * p.N + i;
            if (EDGE == kInside || (j < Q_ext && i < P_ext)) store_through(static_cast<int16_t*>(p.out) + o, v4i{(int)dq[g][0], (int)dq[g][1], (int)dq[g][2], (int)dq[g][3]});
          }
        }
      }
      return;
    }
  }
  if constexpr (!ACT_ON_P) {
#pragma unroll
    for (int ti = 0; ti < TP; ++ti) {
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int i_loc = (wp * TP + ti) * 32 + g4 * 8 + fhalf * 4;
        const int4 c4 = *reinterpret_cast<const int4*>(s_corr + i_loc);
        const int4 m4 = *reinterpret_cast<const int4*>(s_mult + i_loc);
        const int4 s4 = *reinterpret_cast<const int4*>(s_shift + i_loc);
#pragma unroll
        for (int tj = 0; tj < TQ; ++tj) {
          const int j = q0 + (wq * TQ + tj) * 32 + frow;
          const int32_t r0 = finish_one<OM, AWAY>(acc[ti][tj][g4 * 4 + 0] + c4.x, m4.x, s4.x, acc16, rs);
          const int32_t r1 = finish_one<OM, AWAY>(acc[ti][tj][g4 * 4 + 1] + c4.y, m4.y, s4.y, acc16, rs);
          const int32_t r2 = finish_one<OM, AWAY>(acc[ti][tj][g4 * 4 + 2] + c4.z, m4.z, s4.z, acc16, rs);
          const int32_t r3 = finish_one<OM, AWAY>(acc[ti][tj][g4 * 4 + 3] + c4.w, m4.w, s4.w, acc16, rs);
          const size_t o = (size_t)j * p.N + (p0 + i_loc);
          if (EDGE == kInside || (j < Q_ext && p0 + i_loc + (EDGE == kCutGroups ? 4 : 1) <= P_ext))
            store_group<OM>(p.out, o, r0, r1, r2, r3);
          else if (EDGE == kCutGroups && j < Q_ext)
            store_some<OM>(p.out, o, {r0, r1, r2, r3}, P_ext - p0 - i_loc);
        }
      }
    }
  } else {
    const int ohw = p.g.OH * p.g.OW;
    // 16 consecutive pixels of a lane lie in one image and form one aligned store
    const bool vec16 = PIXPERM && OM == 0 && (ohw & 15) == 0 && (reinterpret_cast<uintptr_t>(p.out) & 15u) == 0;
#pragma unroll
    for (int tj = 0; tj < TQ; ++tj) {
      const int j_loc = (wq * TQ + tj) * 32 + frow;
      const int j = q0 + j_loc;
      const int32_t c = s_corr[j_loc], m = s_mult[j_loc], sh = s_shift[j_loc];
      if constexpr (PIXPERM && OM == 0 && TP % 2 == 0) {
        if (vec16) {  // pixels of two row blocks: four lanes write 64 consecutive bytes of a channel
#pragma unroll
          for (int ti = 0; ti < TP; ti += 2) {
            uint32_t dw[2][4];
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
              for (int g4 = 0; g4 < 4; ++g4)
                dw[f][g4] = pack4(finish_one<OM, AWAY>(acc[ti + f][tj][g4 * 4 + 0] + c, m, sh, acc16, rs),
                                  finish_one<OM, AWAY>(acc[ti + f][tj][g4 * 4 + 1] + c, m, sh, acc16, rs),
                                  finish_one<OM, AWAY>(acc[ti + f][tj][g4 * 4 + 2] + c, m, sh, acc16, rs),
                                  finish_one<OM, AWAY>(acc[ti + f][tj][g4 * 4 + 3] + c, m, sh, acc16, rs));
            swap_sixteens(dw[0], dw[1]);
            const int at = stay_here(lane);
            const int i = p0 + (wp * TP + ti + ((at >> 4) & 1)) * 32 + 16 * (at >> 5);
            const int b = i / ohw;
#pragma unroll
            for (int f = 0; f < 2; ++f) {
              const int jj = q0 + (wq * TQ + tj) * 32 + 16 * f + (at & 15);
              if (EDGE == kInside || (jj < Q_ext && i < P_ext))
                store_through(static_cast<uint8_t*>(p.out) + ((size_t)b * p.N + jj) * ohw + (i - b * ohw),
                              v4i{(int)dw[f][0], (int)dw[f][1], (int)dw[f][2], (int)dw[f][3]});
            }
          }
          continue;
        }
      }
#pragma unroll
      for (int ti = 0; ti < TP; ++ti) {
        if constexpr (PIXPERM && OM == 0) {
          if (vec16) {
            const int i = p0 + (wp * TP + ti) * 32 + fhalf * 16;
            const int b = i / ohw;
            const int pix = i - b * ohw;
            uint32_t dw[4];
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
              dw[g4] = pack4(finish_one<OM, AWAY>(acc[ti][tj][g4 * 4 + 0] + c, m, sh, acc16, rs),
                             finish_one<OM, AWAY>(acc[ti][tj][g4 * 4 + 1] + c, m, sh, acc16, rs),
                             finish_one<OM, AWAY>(acc[ti][tj][g4 * 4 + 2] + c, m, sh, acc16, rs),
                             finish_one<OM, AWAY>(acc[ti][tj][g4 * 4 + 3] + c, m, sh, acc16, rs));
            if (EDGE == kInside || (j < Q_ext && i < P_ext))
              *reinterpret_cast<uint4*>(static_cast<uint8_t*>(p.out) + ((size_t)b * p.N + j) * ohw + pix) =
                  make_uint4(dw[0], dw[1], dw[2], dw[3]);
            continue;
          }
        }
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const int i = p0 + (wp * TP + ti) * 32 + (PIXPERM ? fhalf * 16 + g4 * 4 : g4 * 8 + fhalf * 4);
          const int b = i / ohw;
          const int pix = i - b * ohw;
          const int32_t r0 = finish_one<OM, AWAY>(acc[ti][tj][g4 * 4 + 0] + c, m, sh, acc16, rs);
          const int32_t r1 = finish_one<OM, AWAY>(acc[ti][tj][g4 * 4 + 1] + c, m, sh, acc16, rs);
          const int32_t r2 = finish_one<OM, AWAY>(acc[ti][tj][g4 * 4 + 2] + c, m, sh, acc16, rs);
          const int32_t r3 = finish_one<OM, AWAY>(acc[ti][tj][g4 * 4 + 3] + c, m, sh, acc16, rs);
          if (EDGE == kInside || (j < Q_ext && i < P_ext))
            store_group<OM>(p.out, ((size_t)b * p.N + j) * ohw + pix, r0, r1, r2, r3);
        }
      }
    }
  }
}

// Epilogue of one workgroup tile.  acc[ti][tj] is the 32x32 MFMA result of
// sub-tile (ti, tj) of this wavefront: lane l owns column j = l % 32 and, in
// registers 4g .. 4g+3, rows 8g + 4*(l / 32) + 0..3.
//   ACT_ON_P == false (dense, NHWC): i = output channel n, j = row m, out[m*N + n]
//   ACT_ON_P == true  (NCHW)       : i = pixel m, j = channel n, out[(b*N + n)*OHW + pix]
// Dense tiles, and others whose groups of four results along the packed axis are aligned stores,
// take a straight-line path; NCHW images off a multiple of four are stored one by one.
template <int WP, int WQ, int TP, int TQ, bool ACT_ON_P, bool PIXPERM = false>
__device__ __forceinline__ void qgemm_epilogue(const QgemmParams& p, v16i (&acc)[TP][TQ], int p0,
                                               int q0, const int32_t* s_corr,
                                               const int32_t* s_mult, const int32_t* s_shift) {
  constexpr int BP = WP * TP * 32, BQ = WQ * TQ * 32;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wp = wave % WP, wq = wave / WP;
  const int frow = lane & 31, fhalf = lane >> 5;
  const int P_ext = ACT_ON_P ? p.M : p.N;
  const int Q_ext = ACT_ON_P ? p.N : p.M;
  const int ohw = p.g.OH * p.g.OW;
  const bool fast = !ACT_ON_P || p.vec_out;

  if (fast) {
    // interior tiles (block-uniform) run without the per-store bounds checks
    const bool ragged = p0 + BP > P_ext || q0 + BQ > Q_ext;
#define HAGO_FAST_EPILOGUE_E(OM, EDGE, AWAY) \
  qgemm_epilogue_fast<WP, WQ, TP, TQ, ACT_ON_P, OM, PIXPERM, EDGE, AWAY>(p, acc, p0, q0, s_corr, s_mult, s_shift)
#define HAGO_FAST_EPILOGUE_R(OM, AWAY)                                                        \
  (!ragged ? HAGO_FAST_EPILOGUE_E(OM, kInside, AWAY)                                          \
           : ACT_ON_P || P_ext % 4 == 0 ? HAGO_FAST_EPILOGUE_E(OM, kWholeGroups, AWAY)        \
                                        : HAGO_FAST_EPILOGUE_E(OM, (ACT_ON_P ? kWholeGroups : kCutGroups), AWAY))
    // (the tie rule only matters for requantized output)
#define HAGO_FAST_EPILOGUE(OM) HAGO_FAST_EPILOGUE_R(OM, false)
    if (p.out_mode == 0) {
      if (p.rs.half_away)
        HAGO_FAST_EPILOGUE_R(0, true);
      else
        HAGO_FAST_EPILOGUE(0);
    } else if (p.out_mode == 1) {
      HAGO_FAST_EPILOGUE(1);
    } else {
      HAGO_FAST_EPILOGUE(2);
    }
#undef HAGO_FAST_EPILOGUE_R
#undef HAGO_FAST_EPILOGUE_E
#undef HAGO_FAST_EPILOGUE
    return;
  }

  // ---- NCHW output whose image size is not a multiple of 4 (7 x 7 feature maps): a lane's 16
  // consecutive pixels are stored one by one, walking (image, pixel) without a division per element
  if constexpr (ACT_ON_P && PIXPERM) {
    const int32_t acc16 = p.acc_wrap_shift;
#pragma unroll 1
    for (int tj = 0; tj < TQ; ++tj) {
      const int j_loc = (wq * TQ + tj) * 32 + frow;
      const int j = q0 + j_loc;
      const int32_t c = s_corr[j_loc], m = s_mult[j_loc], sh = s_shift[j_loc];
#pragma unroll
      for (int ti = 0; ti < TP; ++ti) {
        const int i0 = p0 + (wp * TP + ti) * 32 + fhalf * 16;
        int b = i0 / ohw;
        int pix = i0 - b * ohw;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          // acc[..][tj] with a runtime tj would need dynamic register indexing; select instead
          int32_t raw = 0;
#pragma unroll
          for (int x = 0; x < TQ; ++x) raw = (x == tj) ? acc[ti][x][r] : raw;
          int32_t a = raw + c;
          if (acc16) a = wrap_acc_bits(a, acc16);
          if (p.has_rq) a = requant_general(a, m, sh, p.rs);
          if (j < Q_ext && i0 + r < P_ext) {
            const int64_t o = ((int64_t)b * p.N + j) * ohw + pix;
            if (p.out_mode == 0)
              static_cast<uint8_t*>(p.out)[o] = (uint8_t)a;
            else if (p.out_mode == 1)
              static_cast<int32_t*>(p.out)[o] = a;
            else
              static_cast<int16_t*>(p.out)[o] = (int16_t)a;
          }
          if (++pix == ohw) { pix = 0; ++b; }
        }
      }
    }
    return;
  }

  // ---- NCHW pixels in the order of the rows (the general kernel), images off a multiple of four: one by one
  if constexpr (ACT_ON_P && !PIXPERM) {
#pragma unroll 1
    for (int tj = 0; tj < TQ; ++tj) {
      const int j_loc = (wq * TQ + tj) * 32 + frow;
      const int j = q0 + j_loc;
#pragma unroll
      for (int ti = 0; ti < TP; ++ti) {
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const int i = p0 + (wp * TP + ti) * 32 + g4 * 8 + fhalf * 4;
          int b = i / ohw;
          int pix = i - b * ohw;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            // acc[..][tj] with a runtime tj would need dynamic register indexing; select instead
            int32_t raw = 0;
#pragma unroll
            for (int x = 0; x < TQ; ++x) raw = (x == tj) ? acc[ti][x][g4 * 4 + r] : raw;
            int32_t a = raw + s_corr[j_loc];
            if (p.acc_wrap_shift) a = wrap_acc_bits(a, p.acc_wrap_shift);
            if (p.has_rq) a = requant_general(a, s_mult[j_loc], s_shift[j_loc], p.rs);
            if (j < Q_ext && i + r < P_ext) {
              const int64_t o = ((int64_t)b * p.N + j) * ohw + pix;
              if (p.out_mode == 0) static_cast<uint8_t*>(p.out)[o] = (uint8_t)a;
              else if (p.out_mode == 1) static_cast<int32_t*>(p.out)[o] = a;
              else static_cast<int16_t*>(p.out)[o] = (int16_t)a;
            }
            if (++pix == ohw) { pix = 0; ++b; }
          }
        }
      }
    }
  }
}

}  // namespace hago
