// Dense GEMM for operands of any size and alignment, on the int8 matrix cores, where there are more output tiles than
// qgemm_few.hip is for: tiles of 64 or 128 rows, operands through registers into a double-buffered LDS stage of 128 source
// bytes per row, two stages of loads in flight.
//
// Rows may start at any byte and the reduction may have any length.  A 16-byte load needs no alignment (off a multiple of
// four bytes it costs four times as much: 64 cycles of a CU's memory pipe for 64 lanes in a row instead of 16).  The last,
// incomplete chunk of a row is read from the 16 elements that END the row and shifted into place.
#include "qgemm_any.h"

namespace hago {

namespace {


// 16 NV bytes of a row in registers.
template <int NV>
struct Run {
  v4i v[NV];
  __device__ void load(const uint8_t* ptr) {
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = *reinterpret_cast<const v4i_any*>(ptr + 16 * i);
  }
};

// Elements k, k + 1, ... of the row at `row` (K elements), as many as a run has room for; zeros beyond the row's end.  In two
// halves, so that other work can lie between the loads and their use: request_tail reads the row's last elements (or the
// run, if the row has all of it), finish_tail moves them into place.
template <int NV, int kEsz>
__device__ __forceinline__ const uint8_t* tail_start(const uint8_t* row, int k, int K) {
  constexpr int E = 16 * NV / kEsz;
  return row + (size_t)(K - k >= E ? k : K - E) * kEsz;
}
template <int NV, int kEsz>
__device__ __forceinline__ void request_tail(Run<NV>& c, const uint8_t* row, int k, int K) {
  if (K >= 16 * NV / kEsz) c.load(tail_start<NV, kEsz>(row, k, K));  // (uniform)
}
template <int NV, int kEsz>
__device__ __forceinline__ void finish_tail(Run<NV>& c, const uint8_t* row, int k, int K) {
  constexpr int ND = 4 * NV, E = 16 * NV / kEsz;
  const int left = K - k;
  uint32_t w[ND];
  if (K < E) {  // the row is shorter than a run: element by element
#pragma unroll
    for (int i = 0; i < ND; ++i) w[i] = 0;
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e < left) {
        const uint32_t x = kEsz == 2 ? *reinterpret_cast<const uint16_t*>(row + (size_t)(k + e) * 2) : row[k + e];
        w[e * kEsz / 4] |= x << (8 * (e * kEsz % 4));
      }
  } else {
#pragma unroll
    for (int i = 0; i < ND; ++i) w[i] = (uint32_t)c.v[i / 4][i % 4];
    if (__builtin_amdgcn_ballot_w64(left > 0 && left < E) == 0) {  // whole runs and none
#pragma unroll
      for (int i = 0; i < ND; ++i) c.v[i / 4][i % 4] = left > 0 ? c.v[i / 4][i % 4] : 0;
      return;
    }
    const int bytes = left >= E ? 0 : left <= 0 ? 16 * NV : (E - left) * kEsz;  // shift towards byte 0 by this many
#pragma unroll
    for (int b = 0; (1 << b) <= ND; ++b)
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        const uint32_t from = i + (1 << b) < ND ? w[i + (1 << b)] : 0u;
        w[i] = ((bytes >> (2 + b)) & 1) ? from : w[i];
      }
#pragma unroll
    for (int i = 0; i < ND; ++i) w[i] = __builtin_amdgcn_alignbyte(i + 1 < ND ? w[i + 1] : 0u, w[i], bytes & 3);
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) c.v[i] = v4i{(int)w[4 * i], (int)w[4 * i + 1], (int)w[4 * i + 2], (int)w[4 * i + 3]};
}

constexpr int kRow = 128;  // bytes of an LDS row = source bytes of a row per stage (256: 9.7 us for 1021 x 1283 -> 1001, 8.6 so)

__device__ __forceinline__ int lds_off(int row, int chunk) { return row * kRow + ((chunk ^ row ^ (row >> 3)) & 7) * 16; }

// KS sets of WP x WQ wavefronts take the stage's 32-k groups in turn and meet in LDS at the end: with one tile per
// CU a second set halves what every wavefront loads, converts and multiplies per stage.
// OUT: codes as kOutFull (qgemm_common.h), the same of a narrow accumulator, any other codes, or sums (us in one kernel and so: 2000 x 700 -> 1003 8.1,
// 7.7, raw 8.0, 7.3; raw 3000 x 101 -> 1984 8.9, 8.1; 1021 x 1283 -> 1001 9.0, 8.8; int16 1024 x 768 -> 768 8.3, 8.0).  Narrow accumulators have a
// kernel for the large tiles only (16 bits, us as any other codes and so: 3000 x 101 -> 1984 9.8, 8.8; 2000 x 2001 -> 2003 21.6, 20.8; as a second form of
// the kernel for other codes: clipped 3000 x 101 -> 1984 9.4, 9.8, and 64 x 64 tiles no faster).
enum { kAnyCodes = kOutFull + 1, kSums, kNarrowFull };
template <bool I16, int WP, int WQ, int TP, int TQ, int KS, int OUT>
__global__ __launch_bounds__(64 * WP * WQ * KS) void qgemm_staged_kernel(QgemmParams p) {
  constexpr int kEsz = I16 ? 2 : 1;
  constexpr int NT = 64 * WP * WQ * KS, BP = 32 * WP * TP, BQ = 32 * WQ * TQ;
  constexpr int UPR = kRow / 16 / kEsz;    // 16-element units per row and stage
  constexpr int BK = 16 * UPR;            // elements per stage
  constexpr int RPU = NT / UPR;           // rows that the threads cover at a time, weights first, then activations
  constexpr int NU = (BP + BQ) / RPU;     // units per thread
  static_assert(NU * RPU == BP + BQ && (RPU <= BP ? BP % RPU : RPU % BP) == 0, "whole units per thread, of one operand in a wavefront");
  constexpr int STAGE = (BP + BQ) * kRow;
  constexpr int RS = BP * 4 + 16;         // output rows in LDS (the widest element)
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];  // 2 stages | output tile
  __shared__ __attribute__((aligned(16))) int32_t s_corr[BP], s_mult[BP], s_shift[BP], s_asum[I16 ? BQ : 1];
  __shared__ __attribute__((aligned(16))) int64_t s_c64[BP];

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wp = wave % WP, wq = wave / WP % WQ, kset = wave / (WP * WQ);
  const int frow = lane & 31, fhalf = lane >> 5;
  const int tiles_p = (p.N + BP - 1) / BP;
  const int tile = p.tile0 + (int)xcd_run(blockIdx.x, gridDim.x);
  const int tile_q = tile / tiles_p;
  const int p0 = (tile - tile_q * tiles_p) * BP, q0 = tile_q * BQ;

  const int unit = t % UPR, row_t = t / UPR;  // unit n of a thread: row row_t + n RPU of both operands' rows, same unit
  auto is_weight = [&](int n) { return RPU <= BP ? n * RPU < BP : wave * 64 / UPR < BP; };  // (uniform)
  const uint8_t* row[NU];
#pragma unroll
  for (int n = 0; n < NU; ++n) {
    const int r = row_t + n * RPU;
    if (is_weight(n)) row[n] = reinterpret_cast<const uint8_t*>(p.wgt) + (size_t)(p0 + r < p.N ? p0 + r : p.N - 1) * p.K * kEsz;
    else row[n] = p.act + (size_t)(q0 + r - BP < p.M ? q0 + r - BP : p.M - 1) * p.K * kEsz;
  }
  constexpr int kVec = I16 ? 2 : 1;
  struct Regs {
    Run<kVec> c[NU];  // (shifting rows off a multiple of four bytes costs more here than its loads: 9.0 us, 8.6)
  };
  int32_t sum[NU];
#pragma unroll
  for (int n = 0; n < NU; ++n) sum[n] = 0;
  auto load = [&]<bool TAIL>(int kt, Regs& r) {
    const int k = kt * BK + unit * 16;
#pragma unroll
    for (int n = 0; n < NU; ++n) {
      if constexpr (TAIL) request_tail<kVec, kEsz>(r.c[n], row[n], k, p.K);
      else r.c[n].load(row[n] + (size_t)k * kEsz);
    }
  };
  auto stash = [&](int buf, const Regs& r) {
    uint8_t* base = smem + buf * STAGE;
#pragma unroll
    for (int n = 0; n < NU; ++n) {
      const int at = row_t + n * RPU;
      const Run<kVec>& c = r.c[n];
      if (I16 || is_weight(n))
#pragma unroll
        for (int i = 0; i < kVec; ++i) sum[n] = plain_sum<I16>(c.v[i], sum[n]);
      if constexpr (I16) {
        v4i hi, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          int h, l;
          split16(c.v[e / 2 % kVec][2 * (e % 2)], c.v[e / 2 % kVec][2 * (e % 2) + 1], h, l);
          hi[e] = h;
          lo[e] = l;
        }
        *reinterpret_cast<v4i*>(base + lds_off(at, unit)) = hi;
        *reinterpret_cast<v4i*>(base + lds_off(at, unit + UPR)) = lo;
      } else {
        *reinterpret_cast<v4i*>(base + lds_off(at, unit)) = is_weight(n) ? c.v[0] : xor4(c.v[0], p.act_xor4);
      }
    }
  };

  Tile32<I16> acc[TP][TQ];
#pragma unroll
  for (int i = 0; i < TP; ++i)
#pragma unroll
    for (int j = 0; j < TQ; ++j) acc[i][j].clear();
  auto multiply = [&](int buf) {
    const uint8_t* base = smem + buf * STAGE;
#pragma unroll
    for (int kk = 0; kk < BK / 32 / KS; ++kk) {
      const int ks = kk * KS + kset;
      v4i ph[TP], pl[TP], qh[TQ], ql[TQ];
#pragma unroll
      for (int i = 0; i < TP; ++i) {
        const int r = (wp * TP + i) * 32 + frow;
        ph[i] = *reinterpret_cast<const v4i*>(base + lds_off(r, ks * 2 + fhalf));
        if constexpr (I16) pl[i] = *reinterpret_cast<const v4i*>(base + lds_off(r, ks * 2 + fhalf + UPR));
      }
#pragma unroll
      for (int j = 0; j < TQ; ++j) {
        const int r = BP + (wq * TQ + j) * 32 + frow;
        qh[j] = *reinterpret_cast<const v4i*>(base + lds_off(r, ks * 2 + fhalf));
        if constexpr (I16) ql[j] = *reinterpret_cast<const v4i*>(base + lds_off(r, ks * 2 + fhalf + UPR));
      }
#pragma unroll
      for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TQ; ++j) {
          acc[i][j].a[0] = mfma(ph[i], qh[j], acc[i][j].a[0]);
          if constexpr (I16) {
            acc[i][j].a[1] = mfma(ph[i], ql[j], acc[i][j].a[1]);
            acc[i][j].a[2] = mfma(pl[i], ql[j], acc[i][j].a[2]);
            acc[i][j].a[1] = mfma(pl[i], qh[j], acc[i][j].a[1]);
          }
        }
    }
  };

  // Stage s + 2 is requested before stage s is multiplied; stage s + 1 goes to LDS after it.  (Four stages ahead were no
  // faster.)  The order of the stages is free: the one that K ends inside comes first, the loop has complete ones only.
  const int KT = (p.K + BK - 1) / BK, tail = KT - p.K / BK;  // stages; 1: one is incomplete
  Regs r0, r1;
  auto request = [&](int s, Regs& r) { load.template operator()<false>(s - tail, r); };
  if (tail) load.template operator()<true>(KT - 1, r0);
  else if (KT > 0) request(0, r0);
  if (KT > 1) request(1, r1);
  // (the constants of the thread that will form a channel's terms, under way during the reduction)
  constexpr int NC = (BP + RPU - 1) / RPU;
  int32_t bias[NC], mult[NC], shift[NC];
#pragma unroll
  for (int n = 0; n < NC; ++n) {
    const int r = row_t + n * RPU;
    bias[n] = 0; mult[n] = 0; shift[n] = 1;
    if (unit == 0 && r < BP && p0 + r < p.N) {
      if (p.bias) bias[n] = p.bias[p0 + r];
      if (OUT != kSums) {
        mult[n] = rq_mult(p.mult, p.per_channel ? p0 + r : 0);
        shift[n] = rq_shift(p.mult, p.shift, p.per_channel ? p0 + r : 0);
      }
    }
  }
  if (tail)
#pragma unroll
    for (int n = 0; n < NU; ++n) finish_tail<kVec, kEsz>(r0.c[n], row[n], (KT - 1) * BK + unit * 16, p.K);
  if (KT > 0) stash(0, r0);
  __syncthreads();
  int s = 0;
  for (; s + 3 < KT; s += 2) {  // every request of the two steps exists
    request(s + 2, r0);
    multiply(0);
    stash(1, r1);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);  // (else sums of the next stage move up and wait for its loads)
    request(s + 3, r1);
    multiply(1);
    stash(0, r0);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
  }
  if (s < KT) {  // one to three stages are left
    if (s + 2 < KT) request(s + 2, r0);
    multiply(0);
    if (s + 1 < KT) {
      stash(1, r1);
      __syncthreads();
      multiply(1);
      if (s + 2 < KT) {
        stash(0, r0);
        __syncthreads();
        multiply(0);
      }
    }
  }

  // ---- channel terms: the UPR threads of a row hold its sum.  SAT: the output is clipped to its container's whole range
  // and every shift is 1 to 21: the rounding term and the zero point are one constant, and the packing saturates (products
  // are at most 2^62, the constant below 2^61 + 2^51).
  constexpr bool sat_ok = OUT == kOutFull || OUT == kNarrowFull;
  const int out_mode = OUT != kSums ? 0 : (p.out_mode == 1 ? 1 : 2);
  int no_sat = !sat_ok;
#pragma unroll
  for (int n = 0; n < NU; ++n) {
    int32_t v = sum[n];
#pragma unroll
    for (int d = 1; d < UPR; d <<= 1) v += __shfl_xor(v, d);
    const int at = row_t + n * RPU;
    if (unit == 0) {
      if (is_weight(n)) {
        const int32_t sh = shift[n < NC ? n : 0];
        s_corr[at] = p0 + at < p.N ? channel_term<I16>(p, bias[n < NC ? n : 0], v, KT * BK) : 0;
        s_mult[at] = mult[n < NC ? n : 0];
        s_shift[at] = sh;
        s_c64[at] = ((int64_t)1 << (30 + (sh & 31))) + ((int64_t)(p.rs.z_out + sat_bias(p.rs)) << (31 + (sh & 31)));
        no_sat |= sh < 1 || sh > 21;
      } else if constexpr (I16) {
        s_asum[at - BP] = 128 * v;
      }
    }
  }
  bool sat = false;
  if constexpr (sat_ok) sat = __syncthreads_or(no_sat) == 0;  // (also: the stages have been consumed)
  else __syncthreads();

  // ---- the sets' sums meet in LDS: of two, each finishes half of the register groups
  static_assert(KS <= 2, "each set finishes half");
  constexpr int NG = 4 / KS;        // register groups that a wavefront finishes, from g_mine on
  const int g_mine = kset * NG;
  int32_t val[TP][TQ][NG][4];
  if constexpr (KS == 2) {
    int32_t* s_sum = reinterpret_cast<int32_t*>(smem);
    auto at = [&](int set, int i, int j, int g) { return ((((set * WP * WQ + wave % (WP * WQ)) * TP + i) * TQ + j) * NG + g) * 256 + lane * 4; };
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TQ; ++j)
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          int32_t give[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int32_t lo = acc[i][j].value(4 * g + e), hi = acc[i][j].value(4 * (NG + g) + e);
            val[i][j][g][e] = kset ? hi : lo;
            give[e] = kset ? lo : hi;
          }
          *reinterpret_cast<v4i*>(s_sum + at(kset ^ 1, i, j, g)) = v4i{give[0], give[1], give[2], give[3]};
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TQ; ++j)
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const v4i o = *reinterpret_cast<const v4i*>(s_sum + at(kset, i, j, g));
#pragma unroll
          for (int e = 0; e < 4; ++e) val[i][j][g][e] += o[e];
        }
    __syncthreads();
  } else {
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TQ; ++j)
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
          for (int e = 0; e < 4; ++e) val[i][j][g][e] = acc[i][j].value(4 * g + e);
  }

  // ---- requantize into an LDS tile in output order, then rows of 16-byte pieces at any alignment
  const int esz = out_mode == 0 ? 1 : (out_mode == 1 ? 4 : 2);
  const uint32_t sflip = sat_flip(p.rs);
#pragma unroll
  for (int i = 0; i < TP; ++i)
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int ch = (wp * TP + i) * 32 + 8 * (g_mine + g) + 4 * fhalf;
      const int4 c4 = *reinterpret_cast<const int4*>(s_corr + ch);
      const int4 m4 = *reinterpret_cast<const int4*>(s_mult + ch);
      const int4 h4 = *reinterpret_cast<const int4*>(s_shift + ch);
      const longlong2 ka = *reinterpret_cast<const longlong2*>(s_c64 + ch), kb = *reinterpret_cast<const longlong2*>(s_c64 + ch + 2);
      const int32_t cc[4] = {c4.x, c4.y, c4.z, c4.w}, mm[4] = {m4.x, m4.y, m4.z, m4.w}, hh[4] = {h4.x, h4.y, h4.z, h4.w};
      const int64_t k64[4] = {ka.x, ka.y, kb.x, kb.y};
#pragma unroll
      for (int j = 0; j < TQ; ++j) {
        const int r = (wq * TQ + j) * 32 + frow;
        int32_t v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = val[i][j][g][e] + cc[e];
          if constexpr (I16) v[e] += s_asum[r];
          if (OUT != kOutFull && p.acc_wrap_shift) v[e] = wrap_acc_bits(v[e], p.acc_wrap_shift);
        }
        uint8_t* dst = smem + r * RS + ch * esz;
        if (sat) {
          uint32_t dw;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = (int32_t)(((int64_t)v[e] * (int64_t)mm[e] + k64[e]) >> 32) >> (hh[e] - 1);
          ashr_sat_pair<0>(dw, v[0], v[1], 0);
          ashr_sat_pair<1>(dw, v[2], v[3], 0);
          *reinterpret_cast<uint32_t*>(dst) = dw ^ sflip;
        } else if (out_mode == 0) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = requant_general(v[e], mm[e], hh[e], p.rs);
          *reinterpret_cast<uint32_t*>(dst) = pack4_perm(v[0], v[1], v[2], v[3]);
        } else if (out_mode == 1) {
          *reinterpret_cast<int4*>(dst) = make_int4(v[0], v[1], v[2], v[3]);
        } else {
          *reinterpret_cast<uint2*>(dst) =
              make_uint2(((uint32_t)v[0] & 0xffffu) | ((uint32_t)v[1] << 16), ((uint32_t)v[2] & 0xffffu) | ((uint32_t)v[3] << 16));
        }
      }
    }
  __syncthreads();
  const int ppr = BP * esz / 16, epp = 16 / esz;  // pieces per row, elements per piece (powers of two)
  // Rows of 128 bytes and more go through the L2, of 64 where they begin with a line, else pieces of a line meet there (us, left in the L2 and so:
  // raw 3000 x 101 -> 1984 11.1, 8.9, 3000 x 100 -> 1999 12.75, 11.4, 2000 x 701 -> 1002 10.0, 9.2; 8 bits 3000 x 101 -> 1984 9.4, 8.8).
  const bool through = ppr >= 8 || p.line_out;
  const int lppr = 31 - __builtin_clz((unsigned)ppr);
  for (int q = t; q < BQ * ppr; q += NT) {
    const int r = q >> lppr, c = q & (ppr - 1);
    const int m = q0 + r, n = p0 + c * epp;
    if (m >= p.M || n >= p.N) continue;
    const uint8_t* src = smem + r * RS + c * 16;
    uint8_t* dst = static_cast<uint8_t*>(p.out) + ((size_t)m * p.N + n) * esz;
    if (n + epp <= p.N) {
      const v4i v = *reinterpret_cast<const v4i*>(src);
      if (through) store_through(dst, v);
      else *reinterpret_cast<v4i_any*>(dst) = v;
    } else {
      for (int b = 0; b < (p.N - n) * esz; ++b) dst[b] = src[b];
    }
  }
}

// A launch holds fewer than 2^32 threads, which 128 x 128 tiles of 512 threads reach at 2^30 rows: in as many launches
// as that takes.
hipError_t launch_tiles(void (*kern)(QgemmParams), QgemmParams p, int64_t tiles, int threads, int lds, hipStream_t st) {
  if (tiles >= (1ll << 31)) return hipErrorInvalidValue;
  const int64_t most = (1ll << 32) / threads - 8;  // (a multiple of the eight XCDs)
  for (int64_t first = 0; first < tiles; first += most) {
    p.tile0 = (int32_t)first;
    const hipError_t e = launch_kernel(kern, dim3((unsigned)(tiles - first < most ? tiles - first : most)), dim3(threads), lds, st, p);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <bool I16, int WP, int WQ, int TP, int TQ, int KS>
hipError_t launch_staged(QgemmParams p, hipStream_t st) {
  constexpr int BP = 32 * WP * TP, BQ = 32 * WQ * TQ;
  constexpr int stages = 2 * (BP + BQ) * kRow, out = BQ * (BP * 4 + 16), sums = (KS - 1) * BP * BQ * 4;
  constexpr int most = stages > out ? stages : out, lds = most > sums ? most : sums;
  const int64_t tiles = (int64_t)((p.N + BP - 1) / BP) * ((p.M + BQ - 1) / BQ);
  p.line_out = p.N % 64 == 0 && ptr_aligned(p.out, 64);
  const bool full = qgemm_full_codes(p);
  int form = p.out_mode != 0 ? kSums : full && !p.acc_wrap_shift ? kOutFull : kAnyCodes;
  auto kern = form == kSums      ? qgemm_staged_kernel<I16, WP, WQ, TP, TQ, KS, kSums>
              : form == kOutFull ? qgemm_staged_kernel<I16, WP, WQ, TP, TQ, KS, kOutFull> : qgemm_staged_kernel<I16, WP, WQ, TP, TQ, KS, kAnyCodes>;
  if constexpr (!I16 && KS == 1) {
    if (full && p.acc_wrap_shift) form = kNarrowFull, kern = qgemm_staged_kernel<I16, WP, WQ, TP, TQ, KS, kNarrowFull>;
  }
  static std::atomic<uint64_t> attr_set[4];
  hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), lds, attr_set[form]);
  if (e != hipSuccess) return e;
  return launch_tiles(kern, p, tiles, 64 * WP * WQ * KS, lds, st);
}

}  // namespace

// Any M, N >= 1, K >= 0 and alignment.  form < 0: by size (us on one MI355X beside each rule); 0 and 1 few tiles with 8 and 4
// wavefronts (where qgemm_few.hip indexes the layer), 3 staged 128 x 128, 4 and others staged 64 x 64 with two sets of
// wavefronts.
hipError_t launch_qgemm_any(const QgemmParams& p, bool i16, int form, hipStream_t st) {
  const int64_t t64 = (int64_t)((p.M + 63) / 64) * ((p.N + 63) / 64);
  if (form < 0 && qgemm_few_wins(p, i16)) return launch_qgemm_few(p, i16, 0, st);
  if ((form == 0 || form == 1) && qgemm_few_ok(p, i16)) return launch_qgemm_few(p, i16, form == 0 ? 8 : 4, st);
  // 128 x 128 tiles once four rounds of 64 x 64 ones would run (2000 x 2001 -> 2003 24 against 34); else 64 x 64 with two sets
  // of wavefronts (1021 x 1283 -> 1001 8.6, 9.9 with one; int16 1024 x 768 -> 768 8.1, 9.3)
  const bool large = form < 0 ? t64 >= 1024 : form == 3;
  if (i16) return large ? launch_staged<true, 2, 4, 2, 1, 1>(p, st) : launch_staged<true, 2, 2, 1, 1, 2>(p, st);
  return large ? launch_staged<false, 2, 4, 2, 1, 1>(p, st) : launch_staged<false, 2, 2, 1, 1, 2>(p, st);
}

}  // namespace hago
