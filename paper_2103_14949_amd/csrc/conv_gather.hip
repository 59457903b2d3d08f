// Convolution in one launch, without LDS staging.  Channel-last first, of 16 or more channels (NCHW: below): out[b][oy][ox][n] =
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
//   MIS: pixels or weights off multiples of four bytes.  Such a 16-byte load costs four times an aligned one (128 cycles of
//   the memory pipe for the 32 x 2 pieces of a wavefront, 32 so), so the aligned dwords that hold the bytes are loaded, one
//   more per piece, and shifted into place (us as loaded directly and so: 61 -> 64 3x3 on 8 x 41 x 41 7.2, 6.3; 201 -> 120 3x3 on one 14 x 14
//   image 11.0, 8.3; 31 -> 60 5x5 on 3 x 40 x 40 7.8, 6.3).
#include "hago_device.h"
#include "launch.h"

#include <cmath>

namespace hago {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef v4i v4i_u __attribute__((aligned(1)));
typedef uint32_t u32_u __attribute__((aligned(1)));
typedef int v2i_u __attribute__((ext_vector_type(2), aligned(1)));

constexpr uint32_t kOob = 0x80000000u;
constexpr uint32_t kBeyond = 0x80000010u;  // the same behind whole dwords of tensors of up to 2^31 bytes, from any byte

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
template <int MODE, bool MIS, int TP, int TC, int KS>
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
  const uint32_t id = xcd_run(blockIdx.x, gridDim.x);
  const uint32_t tile_m = div_by(id, (uint32_t)p.tiles_n, p.inv_tn);
  const int m0 = (int)tile_m * 32 * TP, n0 = (int)(id - tile_m * (uint32_t)p.tiles_n) * 32 * TC;
  // The constants of the channel whose terms the thread will form, under way during the reduction (us, loaded behind it and so: 64 -> 64 1x1
  // stride 2 on 16 x 28 x 28 3.44, 3.26; 64 -> 96 3x3 stride 2 on 4 x 41 x 43 4.24, 4.05; the bias of raw layers alone is better loaded behind it, 3.95, 4.00).
  int32_t c_bias = 0, c_mult = 0, c_shift = 0;
  if (MODE == 0 && threadIdx.x < 32 * TC) {
    const int ch = n0 + (int)threadIdx.x < p.N ? n0 + (int)threadIdx.x : p.N - 1;
    if (p.bias) c_bias = p.bias[ch];
    c_mult = rq_mult(p.mult, p.per_channel ? ch : 0);
    c_shift = rq_shift(p.mult, p.shift, p.per_channel ? ch : 0);
  }

  // MIS: descriptors of the whole dwords that hold the tensors (their first and last hold bytes of the tensor)
  const uint32_t a0 = MIS ? (uint32_t)reinterpret_cast<uintptr_t>(p.act) & 3u : 0u;
  const uint32_t w0 = MIS ? (uint32_t)reinterpret_cast<uintptr_t>(p.wgt) & 3u : 0u;
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(p.act) - a0, 0, (int)(MIS ? (p.act_bytes + a0 + 3u) & ~3u : p.act_bytes), 0x00020000);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t*>(p.wgt) - w0, 0, (int)(MIS ? (p.wgt_bytes + w0 + 3u) & ~3u : p.wgt_bytes), 0x00020000);
  struct Piece {  // 16 bytes as loaded
    v4i v;
    uint32_t more;
    __device__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
      const uint32_t at = MIS ? off & ~3u : off;
      v = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(r, at, 0, 0));
      if constexpr (MIS) more = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, at + 16, 0, 0);
    }
    __device__ void settle(uint32_t off) {  // the offset, modulo 4
      if constexpr (MIS) {
#pragma unroll
        for (int d = 0; d < 4; ++d)
          v[d] = (int)__builtin_amdgcn_alignbyte(d < 3 ? (uint32_t)v[d + 1] : more, (uint32_t)v[d], off);
      }
    }
  };
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
    poff[t] = (uint32_t)((((int)b * p.H + iy) * p.W + ix) * p.C) + a0;
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
    woff[t] = ch < p.N ? (uint32_t)ch * kbytes + w0 : kBeyond;
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
    Piece pa[U][TP], wa[U][TC];
    uint32_t flip[U][TP], dup[U], ptap[U], wtap[U];  // (ptap, wtap: what the step adds to the offsets)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < s_last) {  // uniform
        const uint32_t q = 2u * (uint32_t)(s0 + u) + (uint32_t)h;
        const uint32_t tap = div_by(q, (uint32_t)p.cpt, p.inv_cpt), j = q - tap * (uint32_t)p.cpt;
        const uint32_t ky = div_by(tap, (uint32_t)p.KW, p.inv_kw), kx = tap - ky * (uint32_t)p.KW;
        const uint32_t c0 = 16 * j < (uint32_t)p.C - 16 ? 16 * j : (uint32_t)p.C - 16;
        dup[u] = 16 * j - c0;  // channels of the chunk before it, repeated
        ptap[u] = (ky * (uint32_t)p.W + kx) * (uint32_t)p.C + c0;
        wtap[u] = tap * (uint32_t)p.C + c0;
        const bool real = q < (uint32_t)p.chunks;
#pragma unroll
        for (int t = 0; t < TP; ++t) {
          const bool ok = real && ((rows_in[t] >> ky) & (cols_in[t] >> kx) & 1u);
          flip[u][t] = ok ? p.x4 : p.pad4;
          pa[u][t].load(ra, ok ? poff[t] + ptap[u] : kBeyond);
        }
#pragma unroll
        for (int t = 0; t < TC; ++t)
          wa[u][t].load(rw, real && woff[t] != kBeyond ? woff[t] + wtap[u] : kBeyond);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < s_last) {  // uniform
#pragma unroll
        for (int t = 0; t < TC; ++t) {
          wa[u][t].settle(woff[t] + wtap[u]);
          if (p.C & 15) {  // uniform
#pragma unroll
            for (int d = 0; d < 4; ++d) {
              const uint32_t o = dup[u] < 4u * d ? 0u : dup[u] - 4u * d;
              wa[u][t].v[d] = o < 4u ? wa[u][t].v[d] & (int)(0xffffffffu << (8 * o)) : 0;
            }
          }
#pragma unroll
          for (int d = 0; d < 4; ++d) wsum[t] = __builtin_amdgcn_sdot4(wa[u][t].v[d], 0x01010101, wsum[t], false);
        }
#pragma unroll
        for (int i = 0; i < TP; ++i) {
          pa[u][i].settle(poff[i] + ptap[u]);
#pragma unroll
          for (int d = 0; d < 4; ++d) pa[u][i].v[d] ^= (int)flip[u][i];
#pragma unroll
          for (int t = 0; t < TC; ++t) acc[i][t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wa[u][t].v, pa[u][i].v, acc[i][t], 0, 0, 0);
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
    if (MODE != 0) c_bias = p.bias ? p.bias[ch] : 0;
    const int32_t corr = c_bias + p.corr_coef * ws;
    s_corr[c] = corr;
    if constexpr (MODE == 0) {
      const int32_t m = c_mult, sh = c_shift;
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
  auto run = [&]<bool MIS>() {
    auto kern = mode == 0 ? conv_gather_kernel<0, MIS, TP, TC, KS> : mode == 1 ? conv_gather_kernel<1, MIS, TP, TC, KS> : conv_gather_kernel<2, MIS, TP, TC, KS>;
    return launch_kernel(kern, dim3((unsigned)ids), dim3(64 * KS), 0, st, q);
  };
  // (one step is over before the shifts pay: 22 -> 20 1x1 stride 2 on 59 x 27 x 25 3.15 us, 3.25 with them)
  if (q.steps > 1 && (q.C % 4 != 0 || ((reinterpret_cast<uintptr_t>(q.act) | reinterpret_cast<uintptr_t>(q.wgt)) & 3u) != 0)) return run.template operator()<true>();
  return run.template operator()<false>();
}

// ---- NCHW, and channel-last of fewer than 16 channels.  The 16 reduction elements of a lane (k = (c, ky, kx), or
// (ky, kx, c): the order of the weights) are 16 bytes at 16 places,
// loaded one by one: neighbouring lanes are neighbouring pixels, so a byte load of a wavefront touches two or three lines.
// What an element adds to the address of a pixel's window is the same for every lane of a half, and comes with its tap's
// number from a table in LDS (26 and 6 bits) that the workgroup builds once; whether the tap is inside the image is bit 63 of a mask of
// the pixel's missing taps, shifted by that number, and goes into the offset's sign bit (out of the descriptor's range).
// The weights of a wavefront's steps stay in registers while the workgroup goes from tile to tile, if they are at most
// five steps.
//   KS = 4: four wavefronts share a tile as above; KS = 1: each has one of its own (short reductions).
constexpr int kResident = 5;
struct CnParams {
  const uint8_t* act;
  const int8_t* wgt;
  const int32_t* bias;
  void* out;
  const int32_t* mult;
  const int32_t* shift;
  int32_t B, C, H, W, N, OW, OHW, KH, KW, sh, sw, ph, pw;
  int32_t K, steps, nhwc;
  uint32_t minor;                               // inner extent of the reduction: taps (NCHW) or C
  int32_t tiles_per_img, tiles, nblocks;        // pixel tiles; blocks of output channels
  uint32_t inv_tpi, inv_ow, inv_minor, inv_kw;   // as above
  uint32_t x4, zbyte;                           // sign flip of uint8 bytes; the zero point's byte as stored
  int32_t corr_coef, per_channel, acc_wrap_shift;
  RequantScalars rs;
};

template <int MODE, int TC, int KS, bool ZP>
__global__ __launch_bounds__(KS == 8 ? 512 : 256, 2) void conv_gather_nchw_kernel(CnParams p) {
  constexpr int NW = KS == 8 ? 8 : 4;                          // wavefronts
  constexpr int UPW = KS == 1 ? 4 : (4 * TC < KS ? 1 : 4 * TC / KS);  // groups of four registers a wavefront finishes at a time
  constexpr int NFIN = KS == 1 ? 0 : 4 * TC / UPW;             // wavefronts that finish (KS > 1)
  extern __shared__ __align__(16) int32_t smem[];
  uint32_t* const s_tab = reinterpret_cast<uint32_t*>(smem);                          // steps * 32
  int32_t* const s_wsum = smem + p.steps * 32;                                        // NW x 32 TC (KS > 1)
  v4i* const s_part = reinterpret_cast<v4i*>(s_wsum + (KS == 1 ? 0 : NW * 32 * TC));   // NW TC 4 64 (KS > 1)
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blk = (int)(blockIdx.x % (unsigned)p.nblocks), first = (int)(blockIdx.x / (unsigned)p.nblocks);
  const int stride = (int)(gridDim.x / (unsigned)p.nblocks);
  const int n0 = blk * 32 * TC;
  const int K = p.K;

  if constexpr (MODE == 0 && TC == 2 && KS == 4 && !ZP) HAGO_SPARE_REGISTER("v223");  // (216 needed; two wavefronts on a SIMD either way)

  // the table
  for (int k = threadIdx.x; k < p.steps * 32; k += 64 * NW) {
    const uint32_t major = div_by((uint32_t)k, p.minor, p.inv_minor), minor = (uint32_t)k - major * p.minor;
    const uint32_t c = p.nhwc ? minor : major, tap = p.nhwc ? major : minor;
    const uint32_t ky = div_by(tap, (uint32_t)p.KW, p.inv_kw), kx = tap - ky * (uint32_t)p.KW;
    const uint32_t at = p.nhwc ? (ky * (uint32_t)p.W + kx) * (uint32_t)p.C + c : (c * (uint32_t)p.H + ky) * (uint32_t)p.W + kx;
    s_tab[k] = k < K ? at << 6 | (63 - tap) : 0u;
  }

  // this wavefront's steps and their weights
  const int s_first = KS == 1 ? 0 : p.steps * wave / KS, s_last = KS == 1 ? p.steps : p.steps * (wave + 1) / KS;
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(p.wgt), 0, p.N * K, 0x00020000);
  // (the last, incomplete step byte by byte: none of the next channel)
  v4i wtail[TC];
  const int whole = K >> 5;
  if (s_last > whole) {
#pragma unroll
    for (int t = 0; t < TC; ++t)
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int ch = n0 + 32 * t + n, k0 = 32 * whole + 16 * h + 4 * d;
        uint32_t v = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v |= (uint32_t)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(rw, ch < p.N && k0 + e < K ? (uint32_t)(ch * K + k0 + e) : kOob, 0, 0) << (8 * e);
        wtail[t][d] = (int)v;
      }
  }
  auto load_w = [&](int s, int t) -> v4i {
    const int ch = n0 + 32 * t + n;
    if (s >= whole) return wtail[t];  // uniform
    return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, ch < p.N ? (uint32_t)(ch * K + 32 * s + 16 * h) : kOob, 0, 0));
  };
  const bool resident = s_last - s_first <= kResident;
  v4i wres[kResident][TC];
  int32_t wsum[TC];
#pragma unroll
  for (int t = 0; t < TC; ++t) wsum[t] = 0;
  auto sum_w = [&](const v4i& w, int t) {
#pragma unroll
    for (int d = 0; d < 4; ++d) wsum[t] = __builtin_amdgcn_sdot4(w[d], 0x01010101, wsum[t], false);
  };
  if (resident) {
#pragma unroll
    for (int u = 0; u < kResident; ++u)
      if (s_first + u < s_last)
#pragma unroll
        for (int t = 0; t < TC; ++t) wres[u][t] = load_w(s_first + u, t);
#pragma unroll
    for (int u = 0; u < kResident; ++u)
      if (s_first + u < s_last)
#pragma unroll
        for (int t = 0; t < TC; ++t) sum_w(wres[u][t], t);
  } else {
    for (int s = s_first; s < s_last; ++s)
#pragma unroll
      for (int t = 0; t < TC; ++t) sum_w(load_w(s, t), t);
  }
  // the lane's output channels
  int32_t mult[TC], shift[TC], corr[TC];
#pragma unroll
  for (int t = 0; t < TC; ++t) {
    const int ch = n0 + 32 * t + n < p.N ? n0 + 32 * t + n : p.N - 1;
    corr[t] = p.bias ? p.bias[ch] : 0;
    mult[t] = MODE == 0 ? rq_mult(p.mult, p.per_channel ? ch : 0) : 0;
    shift[t] = MODE == 0 ? rq_shift(p.mult, p.shift, p.per_channel ? ch : 0) : 0;
  }
#pragma unroll
  for (int t = 0; t < TC; ++t) {
    wsum[t] += __shfl_xor(wsum[t], 32);
    if constexpr (KS > 1) {
      if (h == 0) s_wsum[wave * 32 * TC + 32 * t + n] = wsum[t];
    }
  }
  __syncthreads();  // the table (and the sums) are there
  const RequantScalars rs = p.rs;
  bool fold = MODE == 0 && K < (1 << 15) && rs.z_out >= -256 && rs.z_out <= 255 && !rs.half_away && p.acc_wrap_shift == 0;
  int64_t k64[TC];
#pragma unroll
  for (int t = 0; t < TC; ++t) {
    if constexpr (KS > 1) {
      wsum[t] = 0;
#pragma unroll
      for (int w = 0; w < KS; ++w) wsum[t] += s_wsum[w * 32 * TC + 32 * t + n];
    }
    corr[t] += p.corr_coef * wsum[t];
    k64[t] = (int64_t)corr[t] * mult[t] + ((int64_t)1 << (30 + shift[t])) + ((int64_t)rs.z_out << (31 + shift[t]));
    fold = fold && __builtin_amdgcn_ballot_w64(!(shift[t] >= 0 && shift[t] <= 19 && corr[t] >= -(1 << 30) && corr[t] <= (1 << 30))) == 0;
  }

  const int64_t img_in = (int64_t)p.C * p.H * p.W;
  constexpr int AT = KS == 1 ? NW : 1;  // tiles of a workgroup at a time
  for (int tl0 = first * AT; tl0 < p.tiles; tl0 += stride * AT) {
    const int tl = KS == 1 ? tl0 + wave : tl0;
    if (KS == 1 && tl >= p.tiles) break;  // (no barrier in this form's loop)
    const int b = (int)div_by((uint32_t)tl, (uint32_t)p.tiles_per_img, p.inv_tpi);
    int pix0 = (tl - b * p.tiles_per_img) * 32;
    if (p.OHW >= 32 && pix0 > p.OHW - 32) pix0 = p.OHW - 32;  // (the last tile ends with the image)
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.act) + b * img_in, 0, (int)img_in, 0x00020000);
    const int m = pix0 + channel_of_row(n);  // (registers are 16 consecutive pixels)
    const uint32_t oy = div_by((uint32_t)m, (uint32_t)p.OW, p.inv_ow);
    const int iy = (int)oy * p.sh - p.ph, ix = (m - (int)oy * p.OW) * p.sw - p.pw;
    const uint32_t base = (uint32_t)(iy * p.W + ix) * (p.nhwc ? (uint32_t)p.C : 1u);
    const int xl = ix < 0 ? -ix : 0, xr = p.W - ix < p.KW ? p.W - ix : p.KW;  // columns xl .. xr - 1 of the filter are inside
    const uint64_t cols = xl < xr ? ((1ull << xr) - 1) & ~((1ull << xl) - 1) : 0;
    uint64_t missing = 0;  // bit: tap outside the image; bit 63: elements beyond K
    for (int ky = 0; ky < p.KH; ++ky)
      if ((uint32_t)(iy + ky) < (uint32_t)p.H) missing |= cols << (ky * p.KW);
    missing = m < p.OHW ? ~missing : ~0ull;

    v16i acc[TC];
#pragma unroll
    for (int t = 0; t < TC; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[t][r] = 0;
    struct Step { uint32_t byte[16], out; };  // out: bit 15 - e, element e is missing (ZP)
    auto gather = [&](int s, Step& q) {
      q.out = 0;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const uint32_t at = s_tab[32 * s + 16 * h + e];
        const uint32_t miss = (uint32_t)((missing << (at & 63u)) >> 32);
        if constexpr (ZP) q.out = __builtin_amdgcn_alignbit(q.out, miss, 31);
        q.byte[e] = (uint32_t)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(ra, (miss & kOob) | ((base + (at >> 6)) & 0x7fffffffu), 0, 0);
      }
    };
    auto operand = [&](const Step& q) {
      v4i a;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        uint32_t v = q.byte[4 * d] | q.byte[4 * d + 1] << 8 | q.byte[4 * d + 2] << 16 | q.byte[4 * d + 3] << 24;
        if constexpr (ZP) {  // missing taps read 0
#pragma unroll
          for (int e = 0; e < 4; ++e) v |= ((uint32_t)__builtin_amdgcn_sbfe((int)q.out, 15 - 4 * d - e, 1) & p.zbyte) << (8 * e);
        }
        a[d] = (int)(v ^ p.x4);
      }
      return a;
    };
    if (resident) {
#pragma unroll
      for (int u = 0; u < kResident; ++u) {
        if (s_first + u < s_last) {
          Step q;
          gather(s_first + u, q);
          const v4i a = operand(q);
#pragma unroll
          for (int t = 0; t < TC; ++t) acc[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, wres[u][t], acc[t], 0, 0, 0);
        }
      }
    } else {
      Step q[2];
      v4i w[2][TC];
      auto fetch = [&](int s, Step& q_, v4i (&w_)[TC]) {
#pragma unroll
        for (int t = 0; t < TC; ++t) w_[t] = load_w(s, t);
        gather(s, q_);
      };
      auto use = [&](const Step& q_, const v4i (&w_)[TC]) {
        const v4i a = operand(q_);
#pragma unroll
        for (int t = 0; t < TC; ++t) acc[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, w_[t], acc[t], 0, 0, 0);
      };
      fetch(s_first, q[0], w[0]);
      for (int s = s_first; s < s_last; s += 2) {
        if (s + 1 < s_last) fetch(s + 1, q[1], w[1]);
        __builtin_amdgcn_sched_barrier(0);
        use(q[0], w[0]);
        if (s + 1 < s_last) {
          if (s + 2 < s_last) fetch(s + 2, q[0], w[0]);
          __builtin_amdgcn_sched_barrier(0);
          use(q[1], w[1]);
        }
      }
    }

    // results: lane n has channel n0 + 32 t + n, registers 4 g + e pixel 16 h + 4 g + e of the tile
    constexpr int kEsz = MODE == 0 ? 1 : (MODE == 1 ? 4 : 2);
    auto finish = [&](int g0, int t, int32_t mu, int32_t sf, int32_t co, int64_t kk, auto&& sums) {
      const int ch = n0 + 32 * t + n, px = pix0 + 16 * h + 4 * g0;
      int32_t v[UPW][4];
#pragma unroll
      for (int u = 0; u < UPW; ++u) {
        const v4i s = sums(u);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (MODE == 0 && fold) v[u][e] = med3((int32_t)(((int64_t)s[e] * (int64_t)mu + kk) >> (31 + sf)), rs.lo_rel + rs.z_out, rs.hi_rel + rs.z_out);
          else {
            v[u][e] = wrap_acc_bits(s[e] + co, p.acc_wrap_shift);
            if constexpr (MODE == 0) v[u][e] = requant_general(v[u][e], mu, sf, rs);
          }
        }
      }
      if (ch >= p.N || px >= p.OHW) return;
      if (p.nhwc) {  // uniform; a pixel's channels lie across the lanes
        uint8_t* o = static_cast<uint8_t*>(p.out) + (((int64_t)b * p.OHW + px) * p.N + ch) * kEsz;
#pragma unroll
        for (int u = 0; u < UPW; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (px + 4 * u + e >= p.OHW) continue;
            uint8_t* at = o + (int64_t)(4 * u + e) * p.N * kEsz;
            if constexpr (MODE == 0) *at = (uint8_t)v[u][e];
            else if constexpr (MODE == 1) *reinterpret_cast<int32_t*>(at) = v[u][e];
            else *reinterpret_cast<int16_t*>(at) = (int16_t)v[u][e];
          }
        return;
      }
      uint8_t* o = static_cast<uint8_t*>(p.out) + (((int64_t)b * p.N + ch) * p.OHW + px) * kEsz;
      if (px + 4 * UPW <= p.OHW) {
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
          if (px + 4 * u + e >= p.OHW) continue;
          if constexpr (MODE == 0) o[4 * u + e] = (uint8_t)v[u][e];
          else if constexpr (MODE == 1) reinterpret_cast<int32_t*>(o)[4 * u + e] = v[u][e];
          else reinterpret_cast<int16_t*>(o)[4 * u + e] = (int16_t)v[u][e];
        }
    };
    if constexpr (KS == 1) {
#pragma unroll
      for (int t = 0; t < TC; ++t)
        finish(0, t, mult[t], shift[t], corr[t], k64[t],
               [&](int u) { return v4i{acc[t][4 * u], acc[t][4 * u + 1], acc[t][4 * u + 2], acc[t][4 * u + 3]}; });
    } else {
#pragma unroll
      for (int t = 0; t < TC; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          s_part[((wave * TC + t) * 4 + g) * 64 + lane] = v4i{acc[t][4 * g], acc[t][4 * g + 1], acc[t][4 * g + 2], acc[t][4 * g + 3]};
      __syncthreads();
      if (wave < NFIN) {
        const int unit0 = wave * UPW, tc = unit0 >> 2, g0 = unit0 & 3;
        int32_t mu = mult[0], sf = shift[0], co = corr[0];
        int64_t kk = k64[0];
#pragma unroll
        for (int t = 1; t < TC; ++t)
          if (tc == t) { mu = mult[t]; sf = shift[t]; co = corr[t]; kk = k64[t]; }
        finish(g0, tc, mu, sf, co, kk, [&](int u) {
          v4i s = {0, 0, 0, 0};
#pragma unroll
          for (int w = 0; w < KS; ++w) s += s_part[((w * TC + tc) * 4 + g0 + u) * 64 + lane];
          return s;
        });
      }
      __syncthreads();  // the partial sums have been read
    }
  }
}

template <int TC, int KS, bool ZP>
hipError_t launch_nchw_zp(const CnParams& p, int mode, hipStream_t st) {
  constexpr int NW = KS == 8 ? 8 : 4, AT = KS == 1 ? NW : 1;
  CnParams q = p;
  q.nblocks = (q.N + 32 * TC - 1) / (32 * TC);
  const size_t lds = (size_t)q.steps * 128 + (KS == 1 ? 0 : NW * 32 * TC * 4 + (size_t)NW * TC * 4 * 64 * 16);
  auto kern = mode == 0 ? conv_gather_nchw_kernel<0, TC, KS, ZP> : mode == 1 ? conv_gather_nchw_kernel<1, TC, KS, ZP> : conv_gather_nchw_kernel<2, TC, KS, ZP>;
  static std::atomic<uint64_t> attr_set[3];
  hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), 160 * 1024, attr_set[mode]);
  if (e != hipSuccess) return e;
  const int64_t groups = ((int64_t)q.tiles + AT - 1) / AT;
  int64_t per_blk = (lds <= 80 * 1024 && NW == 4 ? 512 : 256) / q.nblocks;
  per_blk = per_blk < 1 ? 1 : (per_blk > groups ? groups : per_blk);
  return launch_kernel(kern, dim3((unsigned)(per_blk * q.nblocks)), dim3(64 * NW), lds, st, q);
}

template <int TC, int KS>
hipError_t launch_nchw(const CnParams& p, int mode, hipStream_t st) {
  return p.zbyte ? launch_nchw_zp<TC, KS, true>(p, mode, st) : launch_nchw_zp<TC, KS, false>(p, mode, st);
}

}  // namespace

const GatherTimes& qconv_gather_times(const GemmArgs& a, const ConvGeom& cg, bool has_workspace, GatherTimes& times) {
  if (times.t64 >= 0) return times;
  const int32_t steps = (cg.KH * cg.KW * ((cg.C + 15) / 16) + 1) / 2;
  // Microseconds, fitted to 333 layers drawn at random (over 333 others the kernel so chosen is 2.5 % from the best on average,
  // half as long again in the worst).  Here: a start, and per tile of a CU 2.2 and 0.075 a step for 64 x 64, of which a CU has whole rounds up to the third and several side by side
  // beyond, 0.62 and 0.049 for 32 x 32; a step's part is 1.65 times that where the operands' rows are unaligned.  The other
  // kernels: 5.9, their rate, the length of the reduction and the tensors' bytes, all but the last 1.2 times for unaligned rows
  // without a workspace.  Measured (here, other): 16 x 28 x 28 64 -> 64 3x3 5.4, 8.4; one image 3.9, 7.1; 32 x 14 x 14 128 -> 128 8.4,
  // 12.0; 8 x 56 x 56 64 -> 128 stride 2 5.8, 10.4; 57 x 56 224 -> 224 7x7 stride 2 31, 66; 4 x 40 x 40 100 -> 200 1x1 stride 2
  // 3.9, 7.8; 22 x 41 x 41 32 -> 32 3x3 6.8, 8.6; 5 x 74 x 72 48 -> 39 5x5 10.1, 17.2; but 32 x 28 x 28 128 -> 128 22.7, 15.1;
  // 20 x 69 x 72 21 -> 33 5x5 28.8, 17.4; 7 x 72 x 72 113 -> 60 3x3 22.7, 17.5.  (Over 50 more layers of both layouts the kernel chosen by this
  // and the other rules is 1.9 % from the best where requantized, 2.0 % raw.)
  auto tiles = [&](int64_t edge) { return ((a.M + edge - 1) / edge) * ((a.N + edge - 1) / edge); };
  const double step = steps * (cg.C % 4 ? 1.65 : 1.0);
  const double x64 = (double)tiles(64) / 256, x32 = (double)tiles(32) / 256;
  const double t64 = 1.9 + (2.2 + 0.075 * step) * (x64 <= 1 ? 1.0 : x64 <= 3 ? 0.95 * std::ceil(x64) : 2.85 + 0.8 * (x64 - 3));
  const double t32 = 2.5 + (0.62 + 0.049 * step) * (x32 <= 1 ? 1.0 : std::pow(x32, 0.93));
  const double bytes = (double)cg.B * cg.C * cg.H * cg.W + (double)a.M * a.N * (a.has_rq ? 1 : a.acc16 ? 2 : 4);
  const double rate = (double)a.M * a.N * a.K / 0.41e9, length = (double)a.K / 175;
  const double steps_and_rate = rate > length ? rate + 0.8 * length : length + 0.8 * rate;
  const double other = (5.9 + steps_and_rate) * (cg.C % 4 && !has_workspace ? 1.2 : 1.0) + bytes / 4e6;
  times = GatherTimes{t64, t32, other, tiles(64)};
  return times;
}

// Returns false (and launches nothing) when the geometry is not this kernel's, or another kernel is the better one.
// forced_shape: 0 64 pixels x 64 output channels by four wavefronts, 1 the same by eight, 2 32 x 32 by four; -1 by size.
bool try_qconv_gather(const GemmArgs& a, const ConvGeom& cg, bool has_workspace, int forced_shape, GatherTimes& times, hipStream_t st, hipError_t* err) {
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
  int shape = forced_shape;
  if (shape < 0) {
    const GatherTimes& e = qconv_gather_times(a, cg, has_workspace, times);
    if ((e.t64 < e.t32 ? e.t64 : e.t32) >= e.other) return false;
    shape = e.t32 < e.t64 ? 2 : e.tiles64 <= 256;  // (eight wavefronts fill a CU's LDS)
  }
  switch (shape) {
    case 0: *err = launch_shape<2, 2, 4>(p, mode, st); break;
    case 1: *err = launch_shape<2, 2, 8>(p, mode, st); break;
    default: *err = launch_shape<1, 1, 4>(p, mode, st); break;
  }
  return true;
}

// The same for NCHW, any channel count, and for channel-last of fewer than 16 channels.  forced_shape, pixels x output channels: 0 32 x 32 by eight wavefronts, 1 32 x 64 by
// four, 2 32 x 32 by four, 3 32 x 64 by one; -1 by size.
bool try_qconv_gather_nchw(const GemmArgs& a, const ConvGeom& cg, bool has_workspace, int forced_shape, hipStream_t st, hipError_t* err) {
  const int64_t img = (int64_t)cg.C * cg.H * cg.W;
  const int64_t ohw = (int64_t)cg.OH * cg.OW;
  // The table's offsets have 26 bits.  The filter's far corner may lie beyond the image, whose offsets count from the
  // pixel's own corner: a filter taller than the image reaches further than the image is large.
  const int64_t far = cg.nhwc ? ((cg.KH - 1) * (int64_t)cg.W + cg.KW - 1) * cg.C + cg.C - 1
                              : ((cg.C - 1) * (int64_t)cg.H + cg.KH - 1) * cg.W + cg.KW - 1;
  if ((cg.nhwc && cg.C >= 16) || cg.KH * cg.KW > 63 || a.K > 28000 || img >= (1ll << 26) || far >= (1ll << 26) || (int64_t)cg.O * a.K >= (1ll << 31) ||
      (int64_t)cg.B * ((ohw + 31) / 32) >= (1ll << 30))
    return false;
  CnParams p{};
  p.act = static_cast<const uint8_t*>(a.act);
  p.wgt = a.wgt;
  p.bias = a.bias;
  p.out = a.out;
  p.mult = a.rq.multiplier;
  p.shift = a.rq.shift;
  p.B = cg.B; p.C = cg.C; p.H = cg.H; p.W = cg.W; p.N = cg.O; p.OW = cg.OW; p.OHW = (int32_t)ohw;
  p.KH = cg.KH; p.KW = cg.KW; p.sh = cg.stride_h; p.sw = cg.stride_w; p.ph = cg.pad_h; p.pw = cg.pad_w;
  p.K = a.K;
  const int taps = cg.KH * cg.KW;
  p.nhwc = cg.nhwc;
  p.minor = (uint32_t)(cg.nhwc ? cg.C : taps);
  p.steps = (a.K + 31) / 32;
  auto inverse = [](int64_t d, int64_t n) { return d > 1 && n * d < (1ll << 32) ? (uint32_t)(((1ull << 32) + (uint64_t)d - 1) / (uint64_t)d) : 0u; };
  p.inv_ow = inverse(cg.OW, ohw + 64);
  p.inv_minor = inverse(p.minor, a.K + 32);
  p.inv_kw = inverse(cg.KW, taps + 32);
  p.x4 = a.act_unsigned ? 0x80808080u : 0u;
  p.zbyte = (uint32_t)a.act_zero_point & 0xffu;
  p.corr_coef = (a.act_unsigned ? 128 : 0) - a.act_zero_point;
  p.per_channel = a.rq.per_channel;
  p.acc_wrap_shift = a.acc_wrap_shift;
  p.rs = RequantScalars{a.rq.z_out, a.rq.clip_lo - a.rq.z_out, a.rq.clip_hi - a.rq.z_out, a.rq.half_away};
  const int mode = a.has_rq ? 0 : (a.acc16 ? 2 : 1);
  p.tiles_per_img = (int32_t)((ohw + 31) / 32);
  p.tiles = cg.B * p.tiles_per_img;
  p.inv_tpi = inverse(p.tiles_per_img, p.tiles);
  // Microseconds: 3.8 and, per CU, 0.4 for every tile and 0.12 (32 channels) or 0.15 (64) for every step, nearly twice that
  // where neighbouring pixels are not neighbouring bytes; long reductions lose more, as a wavefront has two steps' loads
  // under way.  The other kernels: 8.5 and their rate and the length of the reduction (which costs the one-launch
  // kernel more for filters other than 3x3, and is its only cost without a workspace).  Measured (here, other): 5 x 38 x 38 13 -> 42 5x5 6.7, 14.2; 16 x 25 x 26 132 -> 137 1x1 stride 2 5.9,
  // 9.8; 2 x 18 x 16 63 -> 147 5x5 14.1, 10.7 with and 39.5 without a workspace; 8 x 224 x 224 3 -> 64 7x7 stride 2 24.8, 14.3;
  // 64 x 32 x 32 3 -> 16 6.6, 8.6.
  const double step = cg.stride_w > 1 ? 1.8 * p.steps : (double)p.steps;
  const double r32 = (double)p.tiles * ((a.N + 31) / 32) / 256, r64 = (double)p.tiles * ((a.N + 63) / 64) / 256;
  // (long reductions of neighbouring pixels: blocks of 32 by eight wavefronts, 34 -> 140 5x5 on 88 x 87 18.8, with 64 by four 25.6,
  // but with one round of the latter, 128 -> 34 5x5 on 2 x 51 x 52, 25.9 and 20.1)
  const bool deep = p.steps >= 24 && cg.stride_w == 1;
  const double t32 = (r32 > 1 ? r32 : 1.0) * (0.4 + 0.12 * step), t64 = (r64 > 1 ? r64 : 1.0) * (0.4 + 0.15 * step) * (deep && r64 > 1 ? 1.4 : 1.0);
  const bool alone = p.steps <= 2 && r64 >= 4;
  int shape = forced_shape;
  if (shape < 0) {
    // (results leave in pieces of 4 to 16 pixels of different channels' planes, as fast whatever their width: 20 -> 64 5x5 on 16 x 40 x 41
    // 12.4 in 8 and 12.5 in 32 bits, there 21.2 and 22.8; channel-last one element per lane and store)
    const double t = 3.8 + (double)a.M * a.N * (cg.nhwc ? 2.4 : 1.0) / 1.2e6 + (alone ? 0.35 * r64 : t32 < t64 ? t32 : t64) + (p.steps > 18 ? 0.1 * (p.steps - 18) : 0.0);
    const double base = has_workspace && (cg.nhwc || cg.W % 4 == 0) ? 7.5 : 8.5;  // (the rewrite is fast there)
    if (t >= base + (double)a.M * a.N * a.K / 0.41e9 + (double)a.K / (has_workspace || taps == 9 || taps == 1 ? 450 : 70)) return false;
    shape = alone ? 3 : t64 < t32 ? 1 : deep || (p.steps >= 12 && r32 <= 1) ? 0 : 2;
  }
  switch (shape) {
    case 0: *err = launch_nchw<1, 8>(p, mode, st); break;
    case 1: *err = launch_nchw<2, 4>(p, mode, st); break;
    case 2: *err = launch_nchw<1, 4>(p, mode, st); break;
    default: *err = launch_nchw<2, 1>(p, mode, st); break;
  }
  return true;
}

}  // namespace hago
