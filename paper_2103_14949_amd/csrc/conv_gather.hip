// Channel-last convolution of 16 or more channels in one launch, without LDS staging: out[b][oy][ox][n] =
// sum_{ky,kx,c} (a[b][oy sh + ky - ph][ox sw + kx - pw][c] - z_a) * w[n][ky][kx][c] + bias[n].
//
// In channel-last tensors the 16 reduction bytes that a lane gives to a matrix instruction lie together in memory, for the
// pixels as for the weights, so both operands are loaded straight into registers: lane (n, h) loads chunk h of a pair of
// 16-byte chunks of its pixel's tap, and of its output channel's weights.  A workgroup owns 32 TP pixels x 32 TC output
// channels; KS wavefronts share it, each takes a run of the chunk pairs ("steps"), and they add up through LDS.  That suits
// layers that are short of tiles: every load of a wavefront's run is under way at once, there is nothing to rewrite, to
// stage or to wait for in between.  A lane's 16 bytes are a memory-pipe pass of their own, which bounds it at about an
// eighth of the matrix rate, so large layers go elsewhere (see the launch rule).
//   Taps outside the image are loads out of the descriptor's range: they read 0 and become the zero point under the flip
//   mask.  C % 16 != 0: the last chunk of a tap is moved back to end with it, and the weights of the channels it repeats
//   are zeroed.  The rows of the weight operand are permuted so that a lane's 16 results of a 32-channel tile are 16
//   consecutive channels.
#include "hago_device.h"
#include "launch.h"

namespace hago {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef v4i v4i_u __attribute__((aligned(1)));
typedef uint32_t u32_u __attribute__((aligned(1)));
typedef int v2i_u __attribute__((ext_vector_type(2), aligned(1)));

constexpr uint32_t kOob = 0x80000000u;

struct CgParams {
  const uint8_t* act;
  const int8_t* wgt;
  const int32_t* bias;
  void* out;
  const int32_t* mult;
  const int32_t* shift;
  int32_t M, N, C, H, W, OH, OW, KH, KW, sh, sw, ph, pw;
  int32_t cpt, chunks, steps;   // 16-byte chunks of a tap, of a reduction; pairs of them
  int32_t tiles_n;
  uint32_t inv_ohw, inv_ow, inv_cpt, inv_kw, inv_tn;  // ceil(2^32 / d), 0: d = 1 or not exact over the range
  uint32_t act_bytes, wgt_bytes;
  uint32_t x4, pad4;            // sign flip of uint8 bytes; the flipped zero point
  int32_t corr_coef, per_channel, acc_wrap_shift;
  RequantScalars rs;
};

__device__ __forceinline__ uint32_t div_by(uint32_t n, uint32_t d, uint32_t inv) { return d == 1 ? n : (inv ? __umulhi(n, inv) : n / d); }

// row of the weight operand <-> output channel of a 32-channel tile: registers 4 g + e of lane half h are rows
// 8 g + 4 h + e and channels 16 h + 4 g + e
__device__ __forceinline__ int channel_of_row(int r) { return 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3); }

// MODE 0: requantized 8-bit, 1: raw int32, 2: raw int16.
template <int MODE, int TP, int TC, int KS>
__global__ __launch_bounds__(64 * KS) void conv_gather_kernel(CgParams p) {
  constexpr int NTILE = TP * TC;
  constexpr int UPW = 4 * NTILE / KS;   // groups of four registers that a wavefront finishes (1, 2 or 4 of one tile)
  constexpr int U = 5 * 4 / (TP + TC);  // steps whose loads are in flight together
  static_assert(UPW >= 1 && UPW <= 4, "a wavefront finishes at most one tile");
  __shared__ v4i s_part[KS * NTILE * 4 * 64];
  __shared__ int32_t s_wsum[KS][32 * TC];
  __shared__ __align__(16) int32_t s_corr[32 * TC], s_m[32 * TC], s_sh[32 * TC];
  __shared__ __align__(16) int64_t s_k64[32 * TC];
  __shared__ int32_t s_general;
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // consecutive tiles share pixels (and their neighbours' rows): an XCD gets a run of them
  uint32_t id;
  {
    const uint32_t nt = gridDim.x, x = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const uint32_t qn = nt >> 3, rn = nt & 7;
    id = x * qn + (x < rn ? x : rn) + slot;
  }
  const uint32_t tile_m = div_by(id, (uint32_t)p.tiles_n, p.inv_tn);
  const int m0 = (int)tile_m * 32 * TP, n0 = (int)(id - tile_m * (uint32_t)p.tiles_n) * 32 * TC;

  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.act), 0, (int)p.act_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(p.wgt), 0, (int)p.wgt_bytes, 0x00020000);
  // the lane's pixels: byte offset of the window's first tap (it may lie before the tensor), and the filter rows and
  // columns that are inside the image
  uint32_t poff[TP], rows_in[TP], cols_in[TP];
#pragma unroll
  for (int t = 0; t < TP; ++t) {
    const int m = m0 + 32 * t + n;
    const uint32_t ohw = (uint32_t)(p.OH * p.OW);
    const uint32_t b = div_by((uint32_t)m, ohw, p.inv_ohw), r = (uint32_t)m - b * ohw;
    const uint32_t oy = div_by(r, (uint32_t)p.OW, p.inv_ow);
    const int iy = (int)oy * p.sh - p.ph, ix = (int)(r - oy * (uint32_t)p.OW) * p.sw - p.pw;
    poff[t] = (uint32_t)((((int)b * p.H + iy) * p.W + ix) * p.C);
    auto inside = [](int first, int taps, int size) {  // bit k: 0 <= first + k < size
      const int lo = first < 0 ? -first : 0, hi = size - first < taps ? size - first : taps;
      return lo < hi ? (0xffffffffu >> (32 - hi)) & (0xffffffffu << lo) : 0u;
    };
    rows_in[t] = m < p.M ? inside(iy, p.KH, p.H) : 0u;
    cols_in[t] = inside(ix, p.KW, p.W);
  }
  uint32_t woff[TC];
  const uint32_t kbytes = (uint32_t)(p.KH * p.KW * p.C);
#pragma unroll
  for (int t = 0; t < TC; ++t) {
    const int ch = n0 + 32 * t + channel_of_row(n);
    woff[t] = ch < p.N ? (uint32_t)ch * kbytes : kOob;
  }

  v16i acc[TP][TC];
  int32_t wsum[TC];
#pragma unroll
  for (int j = 0; j < TC; ++j) {
    wsum[j] = 0;
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
  }
  const int s_first = p.steps * wave / KS, s_last = p.steps * (wave + 1) / KS;
  for (int s0 = s_first; s0 < s_last; s0 += U) {
    v4i pa[U][TP], wa[U][TC];
    uint32_t flip[U][TP], dup[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < s_last) {  // uniform
        const uint32_t q = 2u * (uint32_t)(s0 + u) + (uint32_t)h;
        const uint32_t tap = div_by(q, (uint32_t)p.cpt, p.inv_cpt), j = q - tap * (uint32_t)p.cpt;
        const uint32_t ky = div_by(tap, (uint32_t)p.KW, p.inv_kw), kx = tap - ky * (uint32_t)p.KW;
        const uint32_t c0 = 16 * j < (uint32_t)p.C - 16 ? 16 * j : (uint32_t)p.C - 16;
        dup[u] = 16 * j - c0;  // channels of the chunk before it, repeated
        const uint32_t toff = (ky * (uint32_t)p.W + kx) * (uint32_t)p.C + c0;
        const bool real = q < (uint32_t)p.chunks;
#pragma unroll
        for (int t = 0; t < TP; ++t) {
          const bool ok = real && ((rows_in[t] >> ky) & (cols_in[t] >> kx) & 1u);
          flip[u][t] = ok ? p.x4 : p.pad4;
          pa[u][t] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(ra, ok ? poff[t] + toff : kOob, 0, 0));
        }
#pragma unroll
        for (int t = 0; t < TC; ++t)
          wa[u][t] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(
              rw, real && woff[t] != kOob ? woff[t] + tap * (uint32_t)p.C + c0 : kOob, 0, 0));
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < s_last) {  // uniform
#pragma unroll
        for (int t = 0; t < TC; ++t) {
          if (p.C & 15) {  // uniform
#pragma unroll
            for (int d = 0; d < 4; ++d) {
              const uint32_t o = dup[u] < 4u * d ? 0u : dup[u] - 4u * d;
              wa[u][t][d] = o < 4u ? wa[u][t][d] & (int)(0xffffffffu << (8 * o)) : 0;
            }
          }
#pragma unroll
          for (int d = 0; d < 4; ++d) wsum[t] = __builtin_amdgcn_sdot4(wa[u][t][d], 0x01010101, wsum[t], false);
        }
#pragma unroll
        for (int i = 0; i < TP; ++i) {
#pragma unroll
          for (int d = 0; d < 4; ++d) pa[u][i][d] ^= (int)flip[u][i];
#pragma unroll
          for (int t = 0; t < TC; ++t) acc[i][t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wa[u][t], pa[u][i], acc[i][t], 0, 0, 0);
        }
      }
    }
  }

  // partial sums and weight sums of every wavefront
#pragma unroll
  for (int t = 0; t < TC; ++t) {
    const int32_t ws = wsum[t] + __shfl_xor(wsum[t], 32);  // the two chunks of a step
    if (h == 0) s_wsum[wave][32 * t + channel_of_row(n)] = ws;
  }
  if constexpr (KS > 1) {
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int t = 0; t < TC; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          s_part[((wave * NTILE + i * TC + t) * 4 + g) * 64 + lane] = v4i{acc[i][t][4 * g], acc[i][t][4 * g + 1], acc[i][t][4 * g + 2], acc[i][t][4 * g + 3]};
  }
  if (threadIdx.x == 0) s_general = 0;
  __syncthreads();
  // the channels' terms.  Folded as in the 1x1 kernel: every term of an output that does not depend on it in one constant,
  // where all channels of the tile allow it.
  const RequantScalars rs = p.rs;
  if (threadIdx.x < 32 * TC) {
    const int c = threadIdx.x, ch = n0 + c < p.N ? n0 + c : p.N - 1;
    int32_t ws = 0;
#pragma unroll
    for (int w = 0; w < KS; ++w) ws += s_wsum[w][c];
    const int32_t corr = (p.bias ? p.bias[ch] : 0) + p.corr_coef * ws;
    s_corr[c] = corr;
    if constexpr (MODE == 0) {
      const int32_t m = rq_mult(p.mult, p.per_channel ? ch : 0), sh = rq_shift(p.mult, p.shift, p.per_channel ? ch : 0);
      s_m[c] = m;
      s_sh[c] = sh;
      s_k64[c] = (int64_t)corr * m + ((int64_t)1 << (30 + sh)) + ((int64_t)rs.z_out << (31 + sh));
      const bool ok = sh >= 0 && sh <= 19 && corr >= -(1 << 30) && corr <= (1 << 30) && (int)kbytes < (1 << 15) && rs.z_out >= -256 &&
                      rs.z_out <= 255 && !rs.half_away && p.acc_wrap_shift == 0;
      if (!ok) atomicOr(&s_general, 1);
    }
  }
  __syncthreads();

  // unit u of a wavefront: registers 4 g .. 4 g + 3 of a tile
  const int unit0 = wave * UPW, tile = unit0 >> 2, g0 = unit0 & 3;
  const int ti = tile / TC, tc = tile % TC;
  const int m = m0 + 32 * ti + n, c0 = 32 * tc + 16 * h + 4 * g0;  // first channel of the lane's 4 UPW, in the workgroup's tile
  const bool general = MODE == 0 && s_general != 0;
  int32_t v[UPW][4];
#pragma unroll
  for (int u = 0; u < UPW; ++u) {
    v4i s = {0, 0, 0, 0};
    if constexpr (KS > 1) {
#pragma unroll
      for (int w = 0; w < KS; ++w) s += s_part[((w * NTILE + tile) * 4 + g0 + u) * 64 + lane];
    }
    const v4i cc = *reinterpret_cast<const v4i*>(s_corr + c0 + 4 * u);
    if constexpr (MODE == 0) {
      const v4i mm = *reinterpret_cast<const v4i*>(s_m + c0 + 4 * u), hh = *reinterpret_cast<const v4i*>(s_sh + c0 + 4 * u);
      if (!general) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t pr = (int64_t)s[e] * (int64_t)mm[e] + s_k64[c0 + 4 * u + e];
          v[u][e] = med3((int32_t)(pr >> (31 + hh[e])), rs.lo_rel + rs.z_out, rs.hi_rel + rs.z_out);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[u][e] = requant_general(wrap_acc_bits(s[e] + cc[e], p.acc_wrap_shift), mm[e], hh[e], rs);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[u][e] = wrap_acc_bits(s[e] + cc[e], p.acc_wrap_shift);
    }
  }
  const int ch = n0 + c0;
  if (m >= p.M || ch >= p.N) return;
  constexpr int kEsz = MODE == 0 ? 1 : (MODE == 1 ? 4 : 2);
  uint8_t* o = static_cast<uint8_t*>(p.out) + ((int64_t)m * p.N + ch) * kEsz;
  if (ch + 4 * UPW <= p.N) {
    if constexpr (MODE == 0) {
      uint32_t dw[UPW];
#pragma unroll
      for (int u = 0; u < UPW; ++u) dw[u] = pack4_perm(v[u][0], v[u][1], v[u][2], v[u][3]);
      if constexpr (UPW == 4) *reinterpret_cast<v4i_u*>(o) = v4i{(int)dw[0], (int)dw[1], (int)dw[2], (int)dw[3]};
      else if constexpr (UPW == 2) *reinterpret_cast<v2i_u*>(o) = v2i_u{(int)dw[0], (int)dw[1]};
      else *reinterpret_cast<u32_u*>(o) = dw[0];
    } else {
#pragma unroll
      for (int u = 0; u < UPW; ++u) {
        if constexpr (MODE == 1) *reinterpret_cast<v4i_u*>(o + 16 * u) = v4i{v[u][0], v[u][1], v[u][2], v[u][3]};
        else *reinterpret_cast<v2i_u*>(o + 8 * u) = v2i_u{(v[u][0] & 0xffff) | (int)((uint32_t)v[u][1] << 16), (v[u][2] & 0xffff) | (int)((uint32_t)v[u][3] << 16)};
      }
    }
    return;
  }
#pragma unroll
  for (int u = 0; u < UPW; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (ch + 4 * u + e >= p.N) continue;
      if constexpr (MODE == 0) o[4 * u + e] = (uint8_t)v[u][e];
      else if constexpr (MODE == 1) reinterpret_cast<int32_t*>(o)[4 * u + e] = v[u][e];
      else reinterpret_cast<int16_t*>(o)[4 * u + e] = (int16_t)v[u][e];
    }
}

template <int TP, int TC, int KS>
hipError_t launch_shape(const CgParams& p, int mode, hipStream_t st) {
  CgParams q = p;
  q.tiles_n = (q.N + 32 * TC - 1) / (32 * TC);
  const int64_t ids = (int64_t)((q.M + 32 * TP - 1) / (32 * TP)) * q.tiles_n;
  q.inv_tn = q.tiles_n > 1 && ids * q.tiles_n < (1ll << 32) ? (uint32_t)(((1ull << 32) + q.tiles_n - 1) / q.tiles_n) : 0u;
  auto kern = mode == 0 ? conv_gather_kernel<0, TP, TC, KS> : mode == 1 ? conv_gather_kernel<1, TP, TC, KS> : conv_gather_kernel<2, TP, TC, KS>;
  hipLaunchKernelGGL(kern, dim3((unsigned)ids), dim3(64 * KS), 0, st, q);
  return hipGetLastError();
}

}  // namespace

// Returns false (and launches nothing) when the geometry is not this kernel's, or another kernel is the better one.
// forced_shape: 0 64 pixels x 64 output channels by four wavefronts, 1 the same by eight, 2 32 x 32 by four; -1 by size.
bool try_qconv_gather(const GemmArgs& a, const ConvGeom& cg, int forced_shape, hipStream_t st, hipError_t* err) {
  const int64_t act_bytes = (int64_t)cg.B * cg.C * cg.H * cg.W, wgt_bytes = (int64_t)cg.O * a.K;
  if (!cg.nhwc || cg.C < 16 || cg.KH > 32 || cg.KW > 32 || act_bytes >= (1ll << 31) || wgt_bytes >= (1ll << 31)) return false;
  CgParams p{};
  p.act = static_cast<const uint8_t*>(a.act);
  p.wgt = a.wgt;
  p.bias = a.bias;
  p.out = a.out;
  p.mult = a.rq.multiplier;
  p.shift = a.rq.shift;
  p.M = a.M; p.N = a.N; p.C = cg.C; p.H = cg.H; p.W = cg.W; p.OH = cg.OH; p.OW = cg.OW;
  p.KH = cg.KH; p.KW = cg.KW; p.sh = cg.stride_h; p.sw = cg.stride_w; p.ph = cg.pad_h; p.pw = cg.pad_w;
  p.cpt = (cg.C + 15) / 16;
  p.chunks = cg.KH * cg.KW * p.cpt;
  p.steps = (p.chunks + 1) / 2;
  auto inverse = [](int64_t d, int64_t n) { return d > 1 && n * d < (1ll << 32) ? (uint32_t)(((1ull << 32) + (uint64_t)d - 1) / (uint64_t)d) : 0u; };
  p.inv_ohw = inverse((int64_t)cg.OH * cg.OW, (int64_t)a.M + 64);
  p.inv_ow = inverse(cg.OW, (int64_t)cg.OH * cg.OW);
  p.inv_cpt = inverse(p.cpt, (int64_t)p.chunks + 2);
  p.inv_kw = inverse(cg.KW, (int64_t)cg.KH * cg.KW + 2);
  p.act_bytes = (uint32_t)act_bytes;
  p.wgt_bytes = (uint32_t)wgt_bytes;
  p.x4 = a.act_unsigned ? 0x80808080u : 0u;
  p.pad4 = ((((uint32_t)a.act_zero_point) ^ (a.act_unsigned ? 0x80u : 0u)) & 0xffu) * 0x01010101u;
  p.corr_coef = (a.act_unsigned ? 128 : 0) - a.act_zero_point;
  p.per_channel = a.rq.per_channel;
  p.acc_wrap_shift = a.acc_wrap_shift;
  p.rs = RequantScalars{a.rq.z_out, a.rq.clip_lo - a.rq.z_out, a.rq.clip_hi - a.rq.z_out, a.rq.half_away};
  const int mode = a.has_rq ? 0 : (a.acc16 ? 2 : 1);
  // Microseconds.  Here: 3 and, per CU, 0.042 (about 100 cycles of the memory pipe) for every operand load of a tile, nearly
  // twice that where they are unaligned (the other kernels lose 1.6 there); a step of 64 x 64 is four loads, of 32 x 32 two.  The other kernels: 6 and their
  // rate, or the length of the reduction where there are few tiles.  Measured (here, other): 16 x 28 x 28 64 -> 64 3x3 5.4,
  // 8.4; one image 3.9, 7.1; 32 x 14 x 14 128 -> 128 8.4, 12.0; 8 x 56 x 56 64 -> 128 stride 2 5.8, 10.4; 57 x 56
  // 224 -> 224 7x7 stride 2 31, 66; 4 x 40 x 40 100 -> 200 1x1 stride 2 3.9, 7.8; but 32 x 28 x 28 128 -> 128 22.7, 15.1.
  auto tiles = [&](int64_t edge) { return ((a.M + edge - 1) / edge) * ((a.N + edge - 1) / edge); };
  const double step = 0.042 * p.steps * (cg.C % 4 ? 1.8 : 1.0);
  auto time = [&](int64_t n, int loads) { return 3.0 + step * loads * (n > 256 ? (double)n / 256 : 1.0); };
  const double t64 = time(tiles(64), 4), t32 = time(tiles(32), 2);
  int shape = forced_shape;
  if (shape < 0) {
    const double rate = (double)a.M * a.N * a.K / 0.41e9, length = (double)a.K / 256;
    if ((t64 < t32 ? t64 : t32) >= (6.0 + (rate > length ? rate : length)) * (cg.C % 4 ? 1.6 : 1.0)) return false;
    shape = t32 < t64 ? 2 : tiles(64) <= 256;  // (eight wavefronts fill a CU's LDS)
  }
  switch (shape) {
    case 0: *err = launch_shape<2, 2, 4>(p, mode, st); break;
    case 1: *err = launch_shape<2, 2, 8>(p, mode, st); break;
    default: *err = launch_shape<1, 1, 4>(p, mode, st); break;
  }
  return true;
}

}  // namespace hago
