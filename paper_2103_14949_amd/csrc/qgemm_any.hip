// Dense GEMM for operands of any size and alignment, on the int8 matrix cores, in two forms:
//
//   direct : few output tiles.  A workgroup owns ONE 32 x 32 tile and its wavefronts split the reduction;
//            fragments go from global memory straight into registers (no LDS, no barrier in the loop),
//            the partial sums meet in LDS once.  What bounds such a problem is the chain
//            launch - first load - reduction - store, so the chain is what this form shortens.
//   staged : many output tiles.  Tiles of 64 or 128 rows, operands through registers into a
//            double-buffered LDS stage of 128 source bytes per row, two stages of loads in flight.
//
// Rows may start at any byte and the reduction may have any length.  A 16-byte load needs no alignment, but off a multiple
// of four bytes it costs four times as much: 64 cycles of a CU's memory pipe for 64 lanes in a row instead of 16, 256 for
// 64 lanes in rows of their own instead of 64 (measured).  So rows off it (MIS) are loaded from the aligned dwords that hold
// them, one dword more per run, and shifted into place in registers; the first and last of these dwords hold bytes of the
// row, so no page is touched that the row has no part in.  The last, incomplete chunk of a row is read from the 16 elements
// that END the row and shifted into place.
//
// int16 operands (I16).  gfx950 has no 16-bit integer matrix instruction; a 16-bit value is the sum
// 256 ah + al of a signed high byte and an unsigned low one, and with al' = al - 128 both are signed bytes:
//   a = a' + 128, a' = 256 ah + al',     w likewise,
//   sum a w = 65536 sum ah wh + 256 sum (ah wl' + al' wh) + sum al' wl' + 128 sum a + 128 sum w - 16384 K,
// modulo 2^32 like the sum itself.  Four byte products in three accumulators replace one product (the vector
// ALUs' two-element dot product, which this replaced, runs at 1/32 of the byte rate); the plain sums of a
// row are taken by the lanes that load it.  Elements that pad the reduction are zeros in both operands and are
// counted in K.
#include "qgemm_common.h"

namespace hago {

namespace {


// 16 NV bytes of a row in registers.  MIS: as the aligned dwords that hold them, `at` the first byte's place in the first.
template <int NV, bool MIS>
struct Run {
  v4i v[NV];
  uint32_t more;
  __device__ void load(const uint8_t* ptr) {
    if constexpr (MIS) {
      typedef int v4i_dword __attribute__((ext_vector_type(4), aligned(4)));
      const uintptr_t a = reinterpret_cast<uintptr_t>(ptr);
      const uint8_t* base = reinterpret_cast<const uint8_t*>(a & ~(uintptr_t)3);
#pragma unroll
      for (int i = 0; i < NV; ++i) v[i] = *reinterpret_cast<const v4i_dword*>(base + 16 * i);
      more = *reinterpret_cast<const uint32_t*>(base + 16 * NV - ((a & 3) ? 0 : 4));
    } else {
#pragma unroll
      for (int i = 0; i < NV; ++i) v[i] = *reinterpret_cast<const v4i_any*>(ptr + 16 * i);
    }
  }
  // the bytes themselves; at = address of the first modulo 4
  __device__ void settle(uint32_t at) {
    if constexpr (MIS) {
#pragma unroll
      for (int i = 0; i < 4 * NV; ++i) {
        const uint32_t next = i + 1 < 4 * NV ? (uint32_t)v[(i + 1) / 4][(i + 1) % 4] : more;
        v[i / 4][i % 4] = (int)__builtin_amdgcn_alignbyte(next, (uint32_t)v[i / 4][i % 4], at);
      }
    }
  }
};

// Elements k, k + 1, ... of the row at `row` (K elements), as many as a run has room for; zeros beyond the row's end.  In two
// halves, so that other work can lie between the loads and their use: request_tail reads the row's last elements (or the
// run, if the row has all of it), finish_tail moves them into place.
template <int NV, bool MIS, int kEsz>
__device__ __forceinline__ const uint8_t* tail_start(const uint8_t* row, int k, int K) {
  constexpr int E = 16 * NV / kEsz;
  return row + (size_t)(K - k >= E ? k : K - E) * kEsz;
}
template <int NV, bool MIS, int kEsz>
__device__ __forceinline__ void request_tail(Run<NV, MIS>& c, const uint8_t* row, int k, int K) {
  if (K >= 16 * NV / kEsz) c.load(tail_start<NV, MIS, kEsz>(row, k, K));  // (uniform)
}
template <int NV, bool MIS, int kEsz>
__device__ __forceinline__ void finish_tail(Run<NV, MIS>& c, const uint8_t* row, int k, int K) {
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
    c.settle((uint32_t)reinterpret_cast<uintptr_t>(tail_start<NV, MIS, kEsz>(row, k, K)) & 3u);
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

// Four results of one output row, channels n .. n + 3, where they exist.
__device__ __forceinline__ void store_four(const QgemmParams& p, int m, int n, const int32_t (&v)[4]) {
  const int64_t o = (int64_t)m * p.N + n;
  if (n + 4 <= p.N) {
    if (p.out_mode == 0) {
      typedef uint32_t u32_any __attribute__((aligned(1)));
      *reinterpret_cast<u32_any*>(static_cast<uint8_t*>(p.out) + o) = pack4_perm(v[0], v[1], v[2], v[3]);
    } else if (p.out_mode == 1) {
      *reinterpret_cast<v4i_any*>(static_cast<int32_t*>(p.out) + o) = v4i{v[0], v[1], v[2], v[3]};
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
    if (p.out_mode == 0) static_cast<uint8_t*>(p.out)[o + e] = (uint8_t)v[e];
    else if (p.out_mode == 1) static_cast<int32_t*>(p.out)[o + e] = v[e];
    else static_cast<int16_t*>(p.out)[o + e] = (int16_t)v[e];
  }
}

// ---- direct form.  NW wavefronts share one tile; U: 32-k groups per wavefront and batch of loads, two
// batches in flight.  256 threads (four results each) finish the tile.
template <bool I16, bool MIS, int NW, int U>
__global__ __launch_bounds__(64 * NW) void qgemm_direct_kernel(QgemmParams p) {
  constexpr int kEsz = I16 ? 2 : 1;
  __shared__ __attribute__((aligned(16))) int32_t s_part[NW][4][64][4];  // [wavefront][register group][lane][4]
  __shared__ __attribute__((aligned(16))) int32_t s_wsum[NW][32], s_asum[I16 ? NW : 1][32], s_constant[3][32];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int frow = lane & 31, fhalf = lane >> 5;
  const int tiles_m = (p.M + 31) / 32;
  const int tile = p.tile0 + xcd_remap(blockIdx.x, gridDim.x);  // consecutive tiles share weight rows, on one XCD
  const int tile_n = tile / tiles_m;
  const int n0 = tile_n * 32, m0 = (tile - tile_n * tiles_m) * 32;

  // rows beyond the matrix read its last row (their results are dropped)
  const uint8_t* wrow = reinterpret_cast<const uint8_t*>(p.wgt) + (size_t)(n0 + frow < p.N ? n0 + frow : p.N - 1) * p.K * kEsz;
  const uint8_t* arow = p.act + (size_t)(m0 + frow < p.M ? m0 + frow : p.M - 1) * p.K * kEsz;
  const int groups = (p.K + 31) >> 5;
  const int g0 = groups * wave / NW, g1 = groups * (wave + 1) / NW;
  const int gf = g1 < (p.K >> 5) ? g1 : (p.K >> 5);  // complete groups end here

  // the tile's per-channel constants: wavefronts 0, 1 and 2 load the bias, the multipliers and the shifts, one dword per lane,
  // in front of the operands; they meet the finishing threads in LDS.  (Loaded by those themselves, three times 16 bytes per
  // lane in each of four wavefronts, they kept the memory pipe from the operands: us, so and then, 1280 x 1776 -> 192 6.3, 6.7;
  // 1128 x 1552 -> 112 5.2, 5.45; 3 x 1680 -> 32 4.1, 4.45; int16 128 x 256 -> 512 4.3, 4.45, 100 x 400 -> 300 4.3, 4.5.)
  int32_t constant = 0;
  if (wave < 3) {
    const int32_t* src = wave == 0 ? p.bias : !p.has_rq ? nullptr : wave == 1 ? p.mult : p.shift;
    const bool each = wave == 0 || p.per_channel;
    const int left = p.N - n0 < 32 ? p.N - n0 : 32;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(src + (src && each ? n0 : 0)), 0,
                                                                       src ? (each ? 4 * left : 4) : 0, 0x00020000);
    constant = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(r, each ? 4 * frow : 0, 0, 0);
  }
  Tile32<I16> acc;
  acc.clear();
  int32_t wsum = 0, asum = 0;
  const bool need_wsum = I16 || p.corr_coef != 0;
  constexpr int kVec = I16 ? 2 : 1;  // a lane's 16 elements
  using Chunk = Run<kVec, MIS>;
  const uint32_t wat = (uint32_t)reinterpret_cast<uintptr_t>(wrow) & 3u, aat = (uint32_t)reinterpret_cast<uintptr_t>(arow) & 3u;
  auto multiply = [&](const Chunk& w, const Chunk& a) {
    if (need_wsum)
#pragma unroll
      for (int i = 0; i < kVec; ++i) wsum = plain_sum<I16>(w.v[i], wsum);
    if constexpr (I16) {
      v4i wh, wl, ah, al;
#pragma unroll
      for (int i = 0; i < kVec; ++i) asum = plain_sum<I16>(a.v[i], asum);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int h, l;
        split16(w.v[e / 2 % kVec][2 * (e % 2)], w.v[e / 2 % kVec][2 * (e % 2) + 1], h, l);
        wh[e] = h;
        wl[e] = l;
        split16(a.v[e / 2 % kVec][2 * (e % 2)], a.v[e / 2 % kVec][2 * (e % 2) + 1], h, l);
        ah[e] = h;
        al[e] = l;
      }
      acc.a[0] = mfma(wh, ah, acc.a[0]);
      acc.a[1] = mfma(wh, al, acc.a[1]);
      acc.a[2] = mfma(wl, al, acc.a[2]);
      acc.a[1] = mfma(wl, ah, acc.a[1]);
    } else {
      acc.a[0] = mfma(w.v[0], xor4(a.v[0], p.act_xor4), acc.a[0]);
    }
  };
  Chunk wt, at;  // the reduction's last, incomplete group (where its loads are many, they are under way from the start)
  auto request_last = [&]() {
    request_tail<kVec, MIS, kEsz>(wt, wrow, gf * 32 + 16 * fhalf, p.K);
    request_tail<kVec, MIS, kEsz>(at, arow, gf * 32 + 16 * fhalf, p.K);
  };
  if ((MIS || I16) && gf < g1) request_last();  // uniform
  if (g0 < gf) {
    struct Batch {
      Chunk w[U], a[U];
    };
    // (a batch beyond the last group reads that group again: the loads stay unconditional)
    auto load = [&](int g, Batch& b) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int gg = g + u < gf ? g + u : gf - 1;
        const size_t off = (size_t)(gg * 32 + 16 * fhalf) * kEsz;
        b.w[u].load(wrow + off);
        b.a[u].load(arow + off);
      }
    };
    auto use = [&](int g, Batch& b) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (g + u < gf) {
          b.w[u].settle(wat);
          b.a[u].settle(aat);
          multiply(b.w[u], b.a[u]);
        }
    };
    Batch b0, b1;
    load(g0, b0);
    for (int g = g0; g < gf; g += 2 * U) {
      if (g + U < gf) load(g + U, b1);
      use(g, b0);
      if (g + 2 * U < gf) load(g + 2 * U, b0);
      if (g + U < gf) use(g + U, b1);
    }
  }
  if (gf < g1) {
    const int k = gf * 32 + 16 * fhalf;
    if (!MIS && !I16) request_last();
    finish_tail<kVec, MIS, kEsz>(wt, wrow, k, p.K);
    finish_tail<kVec, MIS, kEsz>(at, arow, k, p.K);
    multiply(wt, at);
  }

  wsum += __shfl_xor(wsum, 32);
  if constexpr (I16) asum += __shfl_xor(asum, 32);
  if (fhalf == 0) {
    s_wsum[wave][frow] = wsum;
    if constexpr (I16) s_asum[wave][frow] = asum;
    if (wave < 3) s_constant[wave][frow] = constant;
  }
#pragma unroll
  for (int g = 0; g < 4; ++g)
    *reinterpret_cast<v4i*>(s_part[wave][g][lane]) = v4i{acc.value(4 * g), acc.value(4 * g + 1), acc.value(4 * g + 2), acc.value(4 * g + 3)};
  __syncthreads();
  if (t >= 256) return;

  // thread (g4 = t / 64, lane): channels fin_n .. fin_n + 3 of row m0 + lane % 32
  const int g4 = t >> 6, m = m0 + frow, fin = 8 * g4 + 4 * fhalf, fin_n = n0 + fin;
  v4i s = {0, 0, 0, 0};
  int32_t ws[4] = {0, 0, 0, 0}, as = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const v4i q = *reinterpret_cast<const v4i*>(s_part[w][g4][lane]);
    const v4i qs = *reinterpret_cast<const v4i*>(&s_wsum[w][fin]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s[e] += q[e];
      ws[e] += qs[e];
    }
    if constexpr (I16) as += s_asum[w][frow];
  }
  if (m >= p.M || fin_n >= p.N) return;
  const v4i bias = *reinterpret_cast<const v4i*>(&s_constant[0][fin]), mu = *reinterpret_cast<const v4i*>(&s_constant[1][fin]),
            sh = *reinterpret_cast<const v4i*>(&s_constant[2][fin]);
  int32_t v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = s[e] + channel_term<I16>(p, bias[e], ws[e], groups * 32) + 128 * as;
    if (p.acc_wrap_shift) v[e] = wrap_acc_bits(v[e], p.acc_wrap_shift);
    if (p.has_rq) v[e] = requant_general(v[e], p.mult ? mu[e] : 1 << 30, sh[e] - (p.mult ? 0 : 1), p.rs);  // (as rq_mult, rq_shift)
  }
  store_four(p, m, fin_n, v);
}

// ---- staged form
constexpr int kRow = 128;  // bytes of an LDS row = source bytes of a row per stage (256: 9.7 us for 1021 x 1283 -> 1001, 8.6 so)

__device__ __forceinline__ int lds_off(int row, int chunk) { return row * kRow + ((chunk ^ row ^ (row >> 3)) & 7) * 16; }

// KS sets of WP x WQ wavefronts take the stage's 32-k groups in turn and meet in LDS at the end: with one tile per
// CU a second set halves what every wavefront loads, converts and multiplies per stage.
template <bool I16, int WP, int WQ, int TP, int TQ, int KS>
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
  const int tile = p.tile0 + xcd_remap(blockIdx.x, gridDim.x);
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
    Run<kVec, false> c[NU];  // (shifting rows off a multiple of four bytes costs more here than its loads: 9.0 us, 8.6)
  };
  int32_t sum[NU];
#pragma unroll
  for (int n = 0; n < NU; ++n) sum[n] = 0;
  auto load = [&]<bool TAIL>(int kt, Regs& r) {
    const int k = kt * BK + unit * 16;
#pragma unroll
    for (int n = 0; n < NU; ++n) {
      if constexpr (TAIL) request_tail<kVec, false, kEsz>(r.c[n], row[n], k, p.K);
      else r.c[n].load(row[n] + (size_t)k * kEsz);
    }
  };
  auto stash = [&](int buf, const Regs& r) {
    uint8_t* base = smem + buf * STAGE;
#pragma unroll
    for (int n = 0; n < NU; ++n) {
      const int at = row_t + n * RPU;
      const Run<kVec, false>& c = r.c[n];
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
      if (p.has_rq) {
        mult[n] = rq_mult(p.mult, p.per_channel ? p0 + r : 0);
        shift[n] = rq_shift(p.mult, p.shift, p.per_channel ? p0 + r : 0);
      }
    }
  }
  if (tail)
#pragma unroll
    for (int n = 0; n < NU; ++n) finish_tail<kVec, false, kEsz>(r0.c[n], row[n], (KT - 1) * BK + unit * 16, p.K);
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
  const bool sat_ok = p.out_mode == 0 && sat_range(p.rs) && !p.rs.half_away && p.rs.z_out >= -128 && p.rs.z_out <= 255;
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
  const bool sat = __syncthreads_or(no_sat) == 0;  // (also: the stages have been consumed)

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
  const int esz = p.out_mode == 0 ? 1 : (p.out_mode == 1 ? 4 : 2);
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
          if (p.acc_wrap_shift) v[e] = wrap_acc_bits(v[e], p.acc_wrap_shift);
        }
        uint8_t* dst = smem + r * RS + ch * esz;
        if (sat) {
          uint32_t dw;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = (int32_t)(((int64_t)v[e] * (int64_t)mm[e] + k64[e]) >> 32) >> (hh[e] - 1);
          ashr_sat_pair<0>(dw, v[0], v[1], 0);
          ashr_sat_pair<1>(dw, v[2], v[3], 0);
          *reinterpret_cast<uint32_t*>(dst) = dw ^ sflip;
        } else if (p.out_mode == 0) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = requant_general(v[e], mm[e], hh[e], p.rs);
          *reinterpret_cast<uint32_t*>(dst) = pack4_perm(v[0], v[1], v[2], v[3]);
        } else if (p.out_mode == 1) {
          *reinterpret_cast<int4*>(dst) = make_int4(v[0], v[1], v[2], v[3]);
        } else {
          *reinterpret_cast<uint2*>(dst) =
              make_uint2(((uint32_t)v[0] & 0xffffu) | ((uint32_t)v[1] << 16), ((uint32_t)v[2] & 0xffffu) | ((uint32_t)v[3] << 16));
        }
      }
    }
  __syncthreads();
  const int ppr = BP * esz / 16, epp = 16 / esz;  // pieces per row, elements per piece (powers of two)
  const int lppr = 31 - __builtin_clz((unsigned)ppr);
  for (int q = t; q < BQ * ppr; q += NT) {
    const int r = q >> lppr, c = q & (ppr - 1);
    const int m = q0 + r, n = p0 + c * epp;
    if (m >= p.M || n >= p.N) continue;
    const uint8_t* src = smem + r * RS + c * 16;
    uint8_t* dst = static_cast<uint8_t*>(p.out) + ((size_t)m * p.N + n) * esz;
    if (n + epp <= p.N) {
      *reinterpret_cast<v4i_any*>(dst) = *reinterpret_cast<const v4i*>(src);
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
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles - first < most ? tiles - first : most)), dim3(threads), lds, st, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <bool I16, bool MIS, int NW, int U>
hipError_t launch_direct(const QgemmParams& p, hipStream_t st) {
  const int64_t tiles = (int64_t)((p.M + 31) / 32) * ((p.N + 31) / 32);
  return launch_tiles(qgemm_direct_kernel<I16, MIS, NW, U>, p, tiles, 64 * NW, 0, st);
}

template <bool I16, int WP, int WQ, int TP, int TQ, int KS>
hipError_t launch_staged(const QgemmParams& p, hipStream_t st) {
  constexpr int BP = 32 * WP * TP, BQ = 32 * WQ * TQ;
  constexpr int stages = 2 * (BP + BQ) * kRow, out = BQ * (BP * 4 + 16), sums = (KS - 1) * BP * BQ * 4;
  constexpr int most = stages > out ? stages : out, lds = most > sums ? most : sums;
  const int64_t tiles = (int64_t)((p.N + BP - 1) / BP) * ((p.M + BQ - 1) / BQ);
  auto kern = qgemm_staged_kernel<I16, WP, WQ, TP, TQ, KS>;
  static std::atomic<uint64_t> attr_set{0};
  hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), lds, attr_set);
  if (e != hipSuccess) return e;
  return launch_tiles(kern, p, tiles, 64 * WP * WQ * KS, lds, st);
}

}  // namespace

// Any M, N >= 1, K >= 0 and alignment.  form < 0: by size (us on one MI355X beside each rule); 0 direct with 8
// wavefronts, 1 direct with 4 (int16: with 8 too), 3 staged 128 x 128, 4 and others staged 64 x 64 with two sets of wavefronts.
hipError_t launch_qgemm_any(const QgemmParams& p, bool i16, int form, hipStream_t st) {
  const int64_t t32 = (int64_t)((p.M + 31) / 32) * ((p.N + 31) / 32), t64 = (int64_t)((p.M + 63) / 64) * ((p.N + 63) / 64);
  const int64_t groups = (p.K + 31) / 32;
  if (form < 0) {
    // The direct form reads 64 row segments per load, a workgroup per 32 x 32 tile: it wins while those are one round over
    // the chip (us, direct and staged: 333 x 1251 -> 221 7.5, 8.0; 7 x 3001 -> 1001 9.1, 12.7; 412 x 1111 -> 285 6.1, 7.8;
    // 141 x 2145 -> 1327 9.5, 10.6; but 305 tiles of 1937 x 3015 -> 154 24, 13; int16 332 x 131 -> 721 4.5, 5.9; 512 x 768 ->
    // 768 9.2, 8.0), or their reductions are one or two groups (int8 2572 x 25 -> 132 4.1, 5.0; int16 1024 x 64 -> 768 5.0, 4.3).
    if (t32 <= 256) form = 0;
    else if (!i16 && t32 * groups <= 1024) form = 1;
    // 128 x 128 tiles once four rounds of 64 x 64 ones would run (2000 x 2001 -> 2003 24 against 34)
    else if (t64 >= 1024) form = 3;
    // two sets of wavefronts (1021 x 1283 -> 1001 8.6, 9.9 with one; int16 1024 x 768 -> 768 8.1, 9.3)
    else form = 4;
  }
  const size_t esz = i16 ? 2 : 1;
  // (up to two groups are over before the shifts pay: 4 x 43 -> 34 3.2 us, 3.5 with them; 32 x 257 -> 32 9.2, 5.5 with them)
  const bool mis = groups > 2 && ((size_t)p.K * esz % 4 != 0 || !ptr_aligned(p.act, 4) || !ptr_aligned(p.wgt, 4));
  auto run = [&]<bool MIS>() {
    if (i16) {
      switch (form) {
        case 0:
        case 1: return launch_direct<true, MIS, 8, 2>(p, st);
        case 3: return launch_staged<true, 2, 4, 2, 1, 1>(p, st);
        default: return launch_staged<true, 2, 2, 1, 1, 2>(p, st);
      }
    }
    switch (form) {
      case 0: return launch_direct<false, MIS, 8, 4>(p, st);
      case 1: return launch_direct<false, MIS, 4, 4>(p, st);
      case 3: return launch_staged<false, 2, 4, 2, 1, 1>(p, st);
      default: return launch_staged<false, 2, 2, 1, 1, 2>(p, st);
    }
  };
  return mis ? run.template operator()<true>() : run.template operator()<false>();
}

}  // namespace hago
