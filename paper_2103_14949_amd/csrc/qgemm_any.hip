// Dense GEMM for operands of any size and alignment, on the int8 matrix cores, in two forms:
//
//   direct : few output tiles.  A workgroup owns ONE 32 x 32 tile and its wavefronts split the reduction;
//            fragments go from global memory straight into registers (no LDS, no barrier in the loop),
//            the partial sums meet in LDS once.  What bounds such a problem is the chain
//            launch - first load - reduction - store, so the chain is what this form shortens.
//   staged : many output tiles.  Tiles of 64 or 128 rows, operands through registers into a
//            double-buffered LDS stage of 128 source bytes per row, two stages of loads in flight.
//
// Rows may start at any byte and the reduction may have any length: 16-byte loads of gfx950 need no alignment,
// and the last, incomplete chunk of a row is read from the 16 elements that END the row and shifted into place, so
// nothing outside the row is touched.  (Byte-by-byte assembly of such rows took 162 us for
// 1021 x 1283 -> 1001.)
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

typedef int v4i_any __attribute__((ext_vector_type(4), aligned(1)));

// The 16 elements of a row that one lane feeds to a 32-k matrix instruction.
template <bool I16>
struct Chunk {
  static constexpr int kVec = I16 ? 2 : 1;
  v4i v[kVec];
};

template <bool I16>
__device__ __forceinline__ Chunk<I16> load_chunk(const uint8_t* ptr) {
  Chunk<I16> c;
#pragma unroll
  for (int i = 0; i < Chunk<I16>::kVec; ++i) c.v[i] = *reinterpret_cast<const v4i_any*>(ptr + 16 * i);
  return c;
}

// Elements k .. k + 15 of the row at `row` (K elements), zeros beyond its end.
template <bool I16>
__device__ __forceinline__ Chunk<I16> load_chunk_tail(const uint8_t* row, int k, int K) {
  constexpr int kEsz = I16 ? 2 : 1, ND = 4 * Chunk<I16>::kVec;
  Chunk<I16> c;
#pragma unroll
  for (int i = 0; i < Chunk<I16>::kVec; ++i) c.v[i] = v4i{0, 0, 0, 0};
  const int left = K - k;
  if (left >= 16) return load_chunk<I16>(row + (size_t)k * kEsz);
  if (left <= 0) return c;
  uint32_t w[ND];
  if (K < 16) {  // the row is shorter than a chunk: element by element
#pragma unroll
    for (int i = 0; i < ND; ++i) w[i] = 0;
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if (e < left) {
        const uint32_t x = I16 ? *reinterpret_cast<const uint16_t*>(row + (size_t)(k + e) * 2) : row[k + e];
        w[e * kEsz / 4] |= x << (8 * (e * kEsz % 4));
      }
  } else {
    c = load_chunk<I16>(row + (size_t)(K - 16) * kEsz);
#pragma unroll
    for (int i = 0; i < ND; ++i) w[i] = (uint32_t)c.v[i / 4][i % 4];
    const int bytes = (16 - left) * kEsz;  // shift towards byte 0 by this many
#pragma unroll
    for (int b = 0; (1 << b) < ND; ++b)
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        const uint32_t from = i + (1 << b) < ND ? w[i + (1 << b)] : 0u;
        w[i] = ((bytes >> (2 + b)) & 1) ? from : w[i];
      }
#pragma unroll
    for (int i = 0; i < ND; ++i) w[i] = __builtin_amdgcn_alignbyte(i + 1 < ND ? w[i + 1] : 0u, w[i], bytes & 3);
  }
#pragma unroll
  for (int i = 0; i < Chunk<I16>::kVec; ++i)
    c.v[i] = v4i{(int)w[4 * i], (int)w[4 * i + 1], (int)w[4 * i + 2], (int)w[4 * i + 3]};
  return c;
}

// Plain sum of the chunk's elements, added to s.
template <bool I16>
__device__ __forceinline__ int32_t chunk_sum(const Chunk<I16>& c, int32_t s) {
#pragma unroll
  for (int i = 0; i < Chunk<I16>::kVec; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int d = c.v[i][e];
      if constexpr (I16)
        s = __builtin_amdgcn_sdot2(__builtin_bit_cast(__attribute__((ext_vector_type(2))) short, d),
                                   __builtin_bit_cast(__attribute__((ext_vector_type(2))) short, 0x00010001), s, false);
      else
        s = __builtin_amdgcn_sdot4(d, 0x01010101, s, false);
    }
  return s;
}

// High and low bytes of 16 int16 elements (low ones biased to signed).
__device__ __forceinline__ void split16(const Chunk<true>& c, v4i& hi, v4i& lo) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t d0 = (uint32_t)c.v[e / 2][2 * (e % 2)], d1 = (uint32_t)c.v[e / 2][2 * (e % 2) + 1];
    hi[e] = (int)__builtin_amdgcn_perm(d1, d0, 0x07050301u);
    lo[e] = (int)(__builtin_amdgcn_perm(d1, d0, 0x06040200u) ^ 0x80808080u);
  }
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
template <bool I16, int NW, int U>
__global__ __launch_bounds__(64 * NW) void qgemm_direct_kernel(QgemmParams p) {
  constexpr int kEsz = I16 ? 2 : 1;
  __shared__ __attribute__((aligned(16))) int32_t s_part[NW][4][64][4];  // [wavefront][register group][lane][4]
  __shared__ __attribute__((aligned(16))) int32_t s_wsum[NW][32], s_asum[I16 ? NW : 1][32];
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

  // per-channel constants of the finishing threads: thread (g4, lane) of the first 256
  const int fin_n = n0 + 8 * (t >> 6) + 4 * fhalf;  // first of its four channels (t < 256)
  int32_t bias[4], mu[4], sh[4];
  if (t < 256) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = fin_n + e < p.N ? fin_n + e : p.N - 1;
      bias[e] = p.bias ? p.bias[n] : 0;
      mu[e] = p.has_rq ? rq_mult(p.mult, p.per_channel ? n : 0) : 0;
      sh[e] = p.has_rq ? rq_shift(p.mult, p.shift, p.per_channel ? n : 0) : 0;
    }
  }

  Tile32<I16> acc;
  acc.clear();
  int32_t wsum = 0, asum = 0;
  const bool need_wsum = I16 || p.corr_coef != 0;
  auto multiply = [&](const Chunk<I16>& w, const Chunk<I16>& a) {
    if (need_wsum) wsum = chunk_sum<I16>(w, wsum);
    if constexpr (I16) {
      asum = chunk_sum<I16>(a, asum);
      v4i wh, wl, ah, al;
      split16(w, wh, wl);
      split16(a, ah, al);
      acc.a[0] = mfma(wh, ah, acc.a[0]);
      acc.a[1] = mfma(wh, al, acc.a[1]);
      acc.a[2] = mfma(wl, al, acc.a[2]);
      acc.a[1] = mfma(wl, ah, acc.a[1]);
    } else {
      acc.a[0] = mfma(w.v[0], xor4(a.v[0], p.act_xor4), acc.a[0]);
    }
  };
  if (g0 < gf) {
    struct Batch {
      Chunk<I16> w[U], a[U];
    };
    // (a batch beyond the last group reads that group again: the loads stay unconditional)
    auto load = [&](int g, Batch& b) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int gg = g + u < gf ? g + u : gf - 1;
        const size_t off = (size_t)(gg * 32 + 16 * fhalf) * kEsz;
        b.w[u] = load_chunk<I16>(wrow + off);
        b.a[u] = load_chunk<I16>(arow + off);
      }
    };
    auto use = [&](int g, const Batch& b) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (g + u < gf) multiply(b.w[u], b.a[u]);
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
  if (gf < g1) {  // the reduction's last, incomplete group
    const int k = gf * 32 + 16 * fhalf;
    multiply(load_chunk_tail<I16>(wrow, k, p.K), load_chunk_tail<I16>(arow, k, p.K));
  }

  wsum += __shfl_xor(wsum, 32);
  if constexpr (I16) asum += __shfl_xor(asum, 32);
  if (fhalf == 0) {
    s_wsum[wave][frow] = wsum;
    if constexpr (I16) s_asum[wave][frow] = asum;
  }
#pragma unroll
  for (int g = 0; g < 4; ++g)
    *reinterpret_cast<v4i*>(s_part[wave][g][lane]) = v4i{acc.value(4 * g), acc.value(4 * g + 1), acc.value(4 * g + 2), acc.value(4 * g + 3)};
  __syncthreads();
  if (t >= 256) return;

  // thread (g4 = t / 64, lane): channels fin_n .. fin_n + 3 of row m0 + lane % 32
  const int g4 = t >> 6, m = m0 + frow;
  v4i s = {0, 0, 0, 0};
  int32_t ws[4] = {0, 0, 0, 0}, as = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const v4i q = *reinterpret_cast<const v4i*>(s_part[w][g4][lane]);
    const v4i qs = *reinterpret_cast<const v4i*>(&s_wsum[w][8 * g4 + 4 * fhalf]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s[e] += q[e];
      ws[e] += qs[e];
    }
    if constexpr (I16) as += s_asum[w][frow];
  }
  if (m >= p.M || fin_n >= p.N) return;
  int32_t v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = s[e] + channel_term<I16>(p, bias[e], ws[e], groups * 32) + 128 * as;
    if (p.acc_wrap_shift) v[e] = wrap_acc_bits(v[e], p.acc_wrap_shift);
    if (p.has_rq) v[e] = requant_general(v[e], mu[e], sh[e], p.rs);
  }
  store_four(p, m, fin_n, v);
}

// ---- staged form
constexpr int kRow = 128;  // bytes of an LDS row = source bytes of a row per stage

__device__ __forceinline__ int lds_off(int row, int chunk) { return row * kRow + ((chunk ^ row ^ (row >> 3)) & 7) * 16; }

// KS sets of WP x WQ wavefronts take the stage's 32-k groups in turn and meet in LDS at the end: with one tile per
// CU a second set halves what every wavefront loads, converts and multiplies per stage.
template <bool I16, int WP, int WQ, int TP, int TQ, int KS>
__global__ __launch_bounds__(64 * WP * WQ * KS) void qgemm_staged_kernel(QgemmParams p) {
  constexpr int kEsz = I16 ? 2 : 1;
  constexpr int NT = 64 * WP * WQ * KS, BP = 32 * WP * TP, BQ = 32 * WQ * TQ;
  constexpr int UPR = I16 ? 4 : 8;        // 16-element units per row and stage
  constexpr int BK = 16 * UPR;            // elements per stage
  constexpr int NP = BP * UPR / NT, NQ = BQ * UPR / NT;  // units per thread
  static_assert(NP * NT == BP * UPR && NQ * NT == BQ * UPR, "whole units per thread");
  constexpr int STAGE = (BP + BQ) * kRow;
  constexpr int RS = BP * 4 + 16;         // output rows in LDS (the widest element)
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];  // 2 stages | output tile
  __shared__ __attribute__((aligned(16))) int32_t s_corr[BP], s_mult[BP], s_shift[BP], s_asum[I16 ? BQ : 1];

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wp = wave % WP, wq = wave / WP % WQ, kset = wave / (WP * WQ);
  const int frow = lane & 31, fhalf = lane >> 5;
  const int tiles_p = (p.N + BP - 1) / BP;
  const int tile = p.tile0 + xcd_remap(blockIdx.x, gridDim.x);
  const int tile_q = tile / tiles_p;
  const int p0 = (tile - tile_q * tiles_p) * BP, q0 = tile_q * BQ;

  const int unit = t % UPR, row_t = t / UPR;  // unit s of a thread: row row_t + s * NT / UPR, same unit
  const uint8_t *wrow[NP], *arow[NQ];
#pragma unroll
  for (int s = 0; s < NP; ++s) {
    const int r = p0 + row_t + s * (NT / UPR);
    wrow[s] = reinterpret_cast<const uint8_t*>(p.wgt) + (size_t)(r < p.N ? r : p.N - 1) * p.K * kEsz;
  }
#pragma unroll
  for (int s = 0; s < NQ; ++s) {
    const int r = q0 + row_t + s * (NT / UPR);
    arow[s] = p.act + (size_t)(r < p.M ? r : p.M - 1) * p.K * kEsz;
  }
  struct Regs {
    Chunk<I16> w[NP], a[NQ];
  };
  int32_t wsum[NP], asum[NQ];
#pragma unroll
  for (int s = 0; s < NP; ++s) wsum[s] = 0;
#pragma unroll
  for (int s = 0; s < NQ; ++s) asum[s] = 0;
  auto load = [&]<bool TAIL>(int kt, Regs& r) {
    const int k = kt * BK + unit * 16;
#pragma unroll
    for (int s = 0; s < NP; ++s)
      r.w[s] = TAIL ? load_chunk_tail<I16>(wrow[s], k, p.K) : load_chunk<I16>(wrow[s] + (size_t)k * kEsz);
#pragma unroll
    for (int s = 0; s < NQ; ++s)
      r.a[s] = TAIL ? load_chunk_tail<I16>(arow[s], k, p.K) : load_chunk<I16>(arow[s] + (size_t)k * kEsz);
  };
  auto put = [&](uint8_t* base, int row, const Chunk<I16>& c, uint32_t flip) {
    if constexpr (I16) {
      v4i hi, lo;
      split16(c, hi, lo);
      *reinterpret_cast<v4i*>(base + lds_off(row, unit)) = hi;
      *reinterpret_cast<v4i*>(base + lds_off(row, unit + 4)) = lo;
    } else {
      *reinterpret_cast<v4i*>(base + lds_off(row, unit)) = xor4(c.v[0], flip);
    }
  };
  auto stash = [&](int buf, const Regs& r) {
    uint8_t* base = smem + buf * STAGE;
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      wsum[s] = chunk_sum<I16>(r.w[s], wsum[s]);
      put(base, row_t + s * (NT / UPR), r.w[s], 0u);
    }
#pragma unroll
    for (int s = 0; s < NQ; ++s) {
      if constexpr (I16) asum[s] = chunk_sum<I16>(r.a[s], asum[s]);
      put(base + BP * kRow, row_t + s * (NT / UPR), r.a[s], p.act_xor4);
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
        const int row = (wp * TP + i) * 32 + frow;
        ph[i] = *reinterpret_cast<const v4i*>(base + lds_off(row, ks * 2 + fhalf));
        if constexpr (I16) pl[i] = *reinterpret_cast<const v4i*>(base + lds_off(row, ks * 2 + fhalf + 4));
      }
#pragma unroll
      for (int j = 0; j < TQ; ++j) {
        const int row = (wq * TQ + j) * 32 + frow;
        qh[j] = *reinterpret_cast<const v4i*>(base + BP * kRow + lds_off(row, ks * 2 + fhalf));
        if constexpr (I16) ql[j] = *reinterpret_cast<const v4i*>(base + BP * kRow + lds_off(row, ks * 2 + fhalf + 4));
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

  // Stage kt + 2 is requested before stage kt is multiplied; stage kt + 1 goes to LDS after it.
  const int KT = (p.K + BK - 1) / BK, KF = p.K / BK;  // stages, complete stages
  Regs r0, r1;
  auto request = [&](int kt, Regs& r) {
    if (kt < KF) load.template operator()<false>(kt, r);
    else if (kt < KT) load.template operator()<true>(kt, r);
  };
  request(0, r0);
  request(1, r1);
  if (KT > 0) stash(0, r0);
  __syncthreads();
  int kt = 0;
  for (; kt + 3 < KF; kt += 2) {  // every request of the two steps is a complete stage
    load.template operator()<false>(kt + 2, r0);
    multiply(0);
    stash(1, r1);
    __syncthreads();
    load.template operator()<false>(kt + 3, r1);
    multiply(1);
    stash(0, r0);
    __syncthreads();
  }
  for (; kt < KT; kt += 2) {
    request(kt + 2, r0);
    multiply(0);
    if (kt + 1 >= KT) break;
    stash(1, r1);
    __syncthreads();
    request(kt + 3, r1);
    multiply(1);
    if (kt + 2 >= KT) break;
    stash(0, r0);
    __syncthreads();
  }

  // ---- channel terms: the UPR threads of a row hold its sum
#pragma unroll
  for (int s = 0; s < NP; ++s) {
    int32_t v = wsum[s];
#pragma unroll
    for (int d = 1; d < UPR; d <<= 1) v += __shfl_xor(v, d);
    const int row = row_t + s * (NT / UPR), n = p0 + row;
    if (unit == 0) {
      const bool in = n < p.N;
      s_corr[row] = in ? channel_term<I16>(p, p.bias ? p.bias[n] : 0, v, KT * BK) : 0;
      s_mult[row] = in && p.has_rq ? rq_mult(p.mult, p.per_channel ? n : 0) : 0;
      s_shift[row] = in && p.has_rq ? rq_shift(p.mult, p.shift, p.per_channel ? n : 0) : 0;
    }
  }
  if constexpr (I16) {
#pragma unroll
    for (int s = 0; s < NQ; ++s) {
      int32_t v = asum[s];
#pragma unroll
      for (int d = 1; d < UPR; d <<= 1) v += __shfl_xor(v, d);
      if (unit == 0) s_asum[row_t + s * (NT / UPR)] = 128 * v;
    }
  }
  __syncthreads();  // (also: the stages have been consumed)

  if constexpr (KS > 1) {  // the other sets' sums, through LDS
    int32_t* s_sum = reinterpret_cast<int32_t*>(smem);
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TQ; ++j) {
        const int at = (((kset - 1) * WP * WQ + wave % (WP * WQ)) * TP + i) * TQ + j;
        if (kset > 0)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            *reinterpret_cast<v4i*>(s_sum + ((at * 4 + g) * 64 + lane) * 4) =
                v4i{acc[i][j].value(4 * g), acc[i][j].value(4 * g + 1), acc[i][j].value(4 * g + 2), acc[i][j].value(4 * g + 3)};
      }
    __syncthreads();
    if (kset == 0) {
#pragma unroll
      for (int z = 1; z < KS; ++z)
#pragma unroll
        for (int i = 0; i < TP; ++i)
#pragma unroll
          for (int j = 0; j < TQ; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              const int at = (((z - 1) * WP * WQ + wave) * TP + i) * TQ + j;
              const v4i o = *reinterpret_cast<const v4i*>(s_sum + ((at * 4 + g) * 64 + lane) * 4);
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[i][j].a[I16 ? 2 : 0][4 * g + e] += o[e];
            }
    }
    __syncthreads();
  }

  // ---- requantize into an LDS tile in output order, then rows of 16-byte pieces at any alignment
  const int esz = p.out_mode == 0 ? 1 : (p.out_mode == 1 ? 4 : 2);
  if (kset == 0)
#pragma unroll
  for (int i = 0; i < TP; ++i)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int ch = (wp * TP + i) * 32 + 8 * g + 4 * fhalf;
      const int4 c4 = *reinterpret_cast<const int4*>(s_corr + ch);
      const int4 m4 = *reinterpret_cast<const int4*>(s_mult + ch);
      const int4 h4 = *reinterpret_cast<const int4*>(s_shift + ch);
      const int32_t cc[4] = {c4.x, c4.y, c4.z, c4.w}, mm[4] = {m4.x, m4.y, m4.z, m4.w}, hh[4] = {h4.x, h4.y, h4.z, h4.w};
#pragma unroll
      for (int j = 0; j < TQ; ++j) {
        const int row = (wq * TQ + j) * 32 + frow;
        int32_t v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = acc[i][j].value(4 * g + e) + cc[e];
          if constexpr (I16) v[e] += s_asum[row];
          if (p.acc_wrap_shift) v[e] = wrap_acc_bits(v[e], p.acc_wrap_shift);
        }
        uint8_t* dst = smem + row * RS + ch * esz;
        if (p.out_mode == 0) {
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
    const int row = q >> lppr, c = q & (ppr - 1);
    const int m = q0 + row, n = p0 + c * epp;
    if (m >= p.M || n >= p.N) continue;
    const uint8_t* src = smem + row * RS + c * 16;
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

template <bool I16, int NW, int U>
hipError_t launch_direct(const QgemmParams& p, hipStream_t st) {
  const int64_t tiles = (int64_t)((p.M + 31) / 32) * ((p.N + 31) / 32);
  return launch_tiles(qgemm_direct_kernel<I16, NW, U>, p, tiles, 64 * NW, 0, st);
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
// wavefronts, 1 direct with 4, 2 staged 64 x 64, 3 staged 128 x 128, 4 staged 64 x 64 with two sets (int8).
hipError_t launch_qgemm_any(const QgemmParams& p, bool i16, int form, hipStream_t st) {
  const int64_t t32 = (int64_t)((p.M + 31) / 32) * ((p.N + 31) / 32), t64 = (int64_t)((p.M + 63) / 64) * ((p.N + 63) / 64);
  const int64_t groups = (p.K + 31) / 32;
  if (form < 0) {
    // The direct form pays 64 row segments per 16 loads: it wins while the whole problem is short (int8, rows
    // at odd bytes: 333 x 251 -> 221 5.7 against 5.8; 942 x 2521 -> 127 15 against 12.8).  int16 rows carry twice
    // the bytes per segment and four times the products (773 x 305 -> 173 6.3 against 8.1, 512 x 768 -> 768
    // 9.3 against 9.1).
    if (t32 * groups <= (i16 ? 8192 : 1024)) form = t32 <= 64 ? 0 : 1;
    // 128 x 128 tiles once four rounds of 64 x 64 ones would run (2000 x 2001 -> 2003 24 against 34)
    else if (t64 >= 1024) form = 3;
    // two sets while a CU holds about one workgroup (1021 x 1283 -> 1001 10.0 against 11.0)
    else form = i16 ? 2 : 4;
  }
  if (i16) {
    switch (form) {
      case 0: return launch_direct<true, 8, 2>(p, st);
      case 1: return launch_direct<true, 4, 2>(p, st);
      case 3: return launch_staged<true, 2, 4, 2, 1, 1>(p, st);
      default: return launch_staged<true, 2, 2, 1, 1, 1>(p, st);
    }
  }
  switch (form) {
    case 0: return launch_direct<false, 8, 4>(p, st);
    case 1: return launch_direct<false, 4, 4>(p, st);
    case 2: return launch_staged<false, 2, 2, 1, 1, 1>(p, st);
    case 3: return launch_staged<false, 2, 4, 2, 1, 1>(p, st);
    default: return launch_staged<false, 2, 2, 1, 1, 2>(p, st);
  }
}

}  // namespace hago
