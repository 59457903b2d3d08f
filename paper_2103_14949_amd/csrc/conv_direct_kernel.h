// Convolution (groups == 1) of any geometry in ONE launch, straight from the caller's tensors: no rewritten copy, no
// scratch memory.  NCHW or NHWC, any kernel, stride and padding, any channel count, images at least four pixels wide.
//
// A workgroup (eight wavefronts) owns a tile of output pixels - TR rows of the stacked images (row R = b * OH + oy; a
// tile of small images spans several) x TW columns - and a block of 64 or 128 output channels.  Per chunk of CC input
// channels it stages in LDS
//   - the input rows the tile needs, channel-last: [row][column][CC + 16] bytes, int8 (uint8 flipped), taps outside the
//     image filled with the zero point, so that padding contributes 0 under the zero-point identity;
//     NCHW: a thread loads the dword of four pixels for 16 channels and transposes 16 x 4 bytes in registers;
//     NHWC: 16 channel bytes of a pixel are one load;
//   - the weights as [output channel][tap][CC];
// and runs the implicit GEMM over 32-byte reduction groups of contiguous LDS bytes.  The next chunk's (or tile's)
// input loads are in flight meanwhile.  16 bytes of padding per pixel and per output channel keep the fragment reads
// spread over the banks.
//
// Up to 16 input channels a group of one tap would be mostly padding (the three-channel first layer of a network: 3 of
// 32 bytes).  Such inputs are staged with 4, 8 or 16 bytes per pixel and a group is then a run of 8, 4 or 2
// neighbouring taps of one filter row.
//
// What bounds it: at the sizes of these layers one or two tiles per CU, so the chain launch - weights and first
// tile - matrix instructions - stores; the matrix pipe only for deep layers.  Measured (the general kernel, the two-launch
// form through a workspace, here; us): 3 -> 64 7x7 stride 2 on 8 x 224 x 224 46, 26, 13.5; 64 -> 128 3x3 stride 2 on
// 32 x 56 x 56 53, 14.2, 10.5; channel-last 65 -> 55 3x3 stride 2 on 31 x 101 x 99 131, 59, 35.
#pragma once

#include "conv_direct.h"

namespace hago {

namespace {

typedef uint32_t u32_any __attribute__((aligned(1)));
typedef uint16_t u16_any __attribute__((aligned(1)));

__device__ __forceinline__ uint32_t divide(uint32_t n, uint32_t d, uint32_t inv, uint32_t& rem) {
  uint32_t q = __umulhi(n, inv);  // q - 2 <= this <= q
  uint32_t r = n - q * d;
  if (r >= d) { ++q; r -= d; }
  if (r >= d) { ++q; r -= d; }
  rem = r;
  return q;
}

// rows a..d = four channels of four pixels -> per pixel the dword of its four channels
__device__ __forceinline__ void transpose4(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t (&o)[4]) {
  const uint32_t t0 = __builtin_amdgcn_perm(b, a, 0x05010400u), t1 = __builtin_amdgcn_perm(b, a, 0x07030602u);
  const uint32_t t2 = __builtin_amdgcn_perm(d, c, 0x05010400u), t3 = __builtin_amdgcn_perm(d, c, 0x07030602u);
  o[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
  o[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
  o[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
  o[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
}

// WT: how weights are staged.  9: NCHW 3x3, four channels' nine taps at once; 2: contiguous channels (1x1, NHWC); 0: byte
// by byte (any kernel; the few-channel form).  MULTI: several chunks of channels.  WPX x WCH wavefronts over pixels and channels, each AF x 32
// pixels by 64 channels.  OUT: sums go out, as 16 or 32 bits; or codes clipped to their container's
// whole range (and terms small enough to fold but for single channels'); or any codes.  (Us in one kernel, with the raw form apart, and so: 64 -> 128
// 3x3 stride 2 on 32 x 56 x 56 10.7, 10.0, 10.0; 3 -> 64 7x7 on 8 x 224 x 224 9.9, 9.7 with the two kinds of codes apart; 3 -> 72 5x5 on 8 x 112 x 112 11.5, 11.3.)
template <bool NHWC, bool SMALL, bool MULTI, int WT, int WPX, int WCH, int AF, int OUT>
__global__ __launch_bounds__(64 * WPX * WCH, 2) void conv_direct_kernel(CdParams p) {
  constexpr int NT = 64 * WPX * WCH;
  constexpr int NU = NHWC ? 8 : (AF == 2 ? 2 : 3);  // staging units per thread
  constexpr int NV = NHWC ? 4 : 16;   // dwords per unit
  constexpr int OB = 64 * WCH;        // output channels per workgroup
  // 512 pixels channel-last: every register is taken (253 of 256).  Its channel constants wait in LDS, and it finds a row's
  // image by division: with the form of one comparison it spilled 62 registers (us, so and then: 3 -> 64 7x7 on 8 x 224 x 224
  // 13.0, 14.5, raw 20.4, 21.5; 64 -> 64 3x3 on 32 x 56 x 56 13.4, 14.6).
  constexpr bool kTight = NHWC && AF == 2;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  constexpr bool RAW = OUT == kSums;
  const int out_mode = RAW ? (p.out_mode == 1 ? 1 : 2) : 0;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wpx = wave % WPX, wch = wave / WPX;
  const int j = lane & 31, h = lane >> 5;
  const int Wp = 4 * p.Wq, PS = p.PS, HW = p.H * p.W;
  const int rowB = Wp * PS;                          // bytes per staged row
  const int wstride = p.groups * 32 + 16;            // bytes per staged output channel
  uint8_t* s_w = smem;
  uint8_t* s_in = smem + OB * wstride;
  int32_t* s_sum = reinterpret_cast<int32_t*>(s_in + p.in_room);
  int32_t* s_corr = s_sum + OB;
  int32_t* s_mu = s_corr + OB;
  int32_t* s_sh = s_mu + OB;
  int32_t* s_flag = s_sh + OB;  // (four words)
  int4* s_fold = reinterpret_cast<int4*>(s_flag + 4);  // folded requantize constants: k64 (two dwords), multiplier, shift - 1

  // tiles: workgroups that share one sit on one XCD, which walks a contiguous eighth (as in conv3x3.hip)
  int blk, tile, tile_end, tile_step;
  const int nwg = (int)gridDim.x / p.nblk;
  if (nwg % 8 == 0) {
    const int xcd = (int)blockIdx.x & 7, q = (int)blockIdx.x >> 3;
    const int per_xcd = (p.ntiles + 7) / 8;
    blk = q % p.nblk;
    tile = xcd * per_xcd + q / p.nblk;
    tile_end = (xcd + 1) * per_xcd < p.ntiles ? (xcd + 1) * per_xcd : p.ntiles;
    tile_step = nwg / 8;
  } else {
    blk = (int)blockIdx.x % p.nblk;
    tile = (int)blockIdx.x / p.nblk;
    tile_end = p.ntiles;
    tile_step = nwg;
  }
  if (tile >= tile_end) return;  // workgroup-uniform
  const int o0 = blk * OB;

  // ---- staging units.  NCHW: (16-channel group, staged row, quad of columns); few channels: one group.
  // NHWC: (staged row, column, 16-channel group).
  const int cgroups = SMALL ? 1 : p.CC >> 4;
  const int per_row = NHWC ? Wp * cgroups : p.Wq;
  const int units = NHWC ? p.rows * per_row : cgroups * p.rows * p.Wq;
  uint32_t raw[NU][NV];
  int u_v[NU], u_x[NU], u_c[NU], u_lds[NU];  // staged row (-1: none), first column, first channel of the chunk, LDS offset
#pragma unroll
  for (int n = 0; n < NU; ++n) {
    const int u = t + NT * n;
    u_v[n] = -1; u_x[n] = 0; u_c[n] = 0; u_lds[n] = 0;
    if (n > 0 && NT * n >= units) continue;  // uniform
    if (u < units) {
      if constexpr (NHWC) {
        uint32_t r, cg;
        const int v = (int)divide((uint32_t)u, (uint32_t)per_row, p.inv_unit1, r);
        const int x = (int)divide(r, (uint32_t)cgroups, p.inv_unit2, cg);
        u_v[n] = v; u_x[n] = x; u_c[n] = 16 * (int)cg;
        u_lds[n] = v * rowB + x * PS + 16 * (int)cg;
      } else {
        uint32_t r, q;
        const int cg = (int)divide((uint32_t)u, (uint32_t)(p.rows * p.Wq), p.inv_unit1, r);
        const int v = (int)divide(r, (uint32_t)p.Wq, p.inv_unit2, q);
        u_v[n] = v; u_x[n] = 4 * (int)q; u_c[n] = 16 * cg;
        u_lds[n] = v * rowB + 4 * (int)q * PS + 16 * cg;
      }
    }
  }
  // first stacked row, first column, first staged row of the stack; the image that row lies in, and its row there
  struct TilePos { int R0, x0, V0, b0, hv0; };
  auto tile_pos = [&](int tl) {
    uint32_t seg, oy;
    const int rt = (int)divide((uint32_t)tl, (uint32_t)p.nseg, p.inv_nseg, seg);
    TilePos q;
    q.R0 = rt * p.TR;
    q.x0 = (int)seg * p.TW;
    const uint32_t b = divide((uint32_t)q.R0, (uint32_t)p.OH, p.inv_oh, oy);
    q.V0 = (int)(b * (uint32_t)p.HV + oy * (uint32_t)p.sr);
    q.b0 = (int)b;
    q.hv0 = (int)oy * p.sr;
    return q;
  };
  // image row of staged row v: whether it exists, and its offset (b * C * H + iy rows for NCHW, (b * H + iy) * W pixels for NHWC)
  auto image_row = [&](const TilePos& q, int v, uint32_t& off) {
    uint32_t hv = (uint32_t)(q.hv0 + v), b = (uint32_t)q.b0;
    if (!kTight && p.rows <= p.HV) {  // uniform: the tile crosses one image boundary at most
      const bool over = hv >= (uint32_t)p.HV;
      hv -= over ? (uint32_t)p.HV : 0u;
      b += over ? 1u : 0u;
    } else {
      b = divide((uint32_t)(q.V0 + v), (uint32_t)p.HV, p.inv_hv, hv);
    }
    int iy = (int)hv - p.ph;
    if (p.sr != p.sh) {  // stride beyond the kernel: only the rows the taps touch are staged
      const int oy = (int)hv / p.KH;
      iy = oy * p.sh + ((int)hv - oy * p.KH) - p.ph;
    }
    const bool ok = v >= 0 && b < (uint32_t)p.B && (unsigned)iy < (unsigned)p.H;
    off = NHWC ? (b * (uint32_t)p.H + (uint32_t)iy) * (uint32_t)p.W : b * (uint32_t)(p.C * HW) + (uint32_t)(iy * p.W);
    return ok;
  };
  const __amdgpu_buffer_rsrc_t rs_act =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.act), 0, (int)p.act_bytes, 0x00020000);
  uint32_t u_mask[NHWC ? 1 : NU];  // NCHW: bytes of the loaded dwords that lie inside the image
  int32_t u_shift[NU];  // NCHW: bits that move them into place (> 0: right); NHWC: bytes, -1: outside the image
  auto load_input = [&](const TilePos& q, int c0) {
#pragma unroll
    for (int n = 0; n < NU; ++n) {
      if (n > 0 && NT * n >= units) break;  // uniform
      uint32_t off;
      const bool row_ok = image_row(q, u_v[n], off);
      const int ix = q.x0 * p.sw + u_x[n] - p.pw - p.off_x;
      if constexpr (NHWC) {
        const bool ok = row_ok && (unsigned)ix < (unsigned)p.W;
        u_shift[n] = ok ? 0 : -1;
        v4i v = {0, 0, 0, 0};
        if (ok) {
          // (16 bytes that would run past the tensor's end are read from its last 16 and moved into place later)
          const uint32_t at = (off + (uint32_t)ix) * (uint32_t)p.C + (uint32_t)(c0 + u_c[n]), most = (uint32_t)p.act_bytes - 16u;
          if (at > most) u_shift[n] = (int32_t)(at - most);  // bytes; at most 16 beyond: nothing is left
          v = *reinterpret_cast<const v4i_any*>(p.act + (at < most ? at : most));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) raw[n][i] = (uint32_t)v[i];
      } else {
        // the quad's dword, pulled inside the row; channels beyond C read what follows, or nothing beyond the tensor (their
        // weights are 0).  A quad without a byte in the image is out of the descriptor's range and reads 0.
        const int ixc = ix < 0 ? 0 : (ix > p.W - 4 ? p.W - 4 : ix);
        const int d = ix - ixc;
        u_mask[n] = !row_ok || d >= 4 || d <= -4 ? 0u : (d >= 0 ? 0xffffffffu >> (8 * d) : 0xffffffffu << (-8 * d));
        u_shift[n] = d >= 4 || d <= -4 ? 0 : 8 * d;
        if constexpr (MULTI) {
          // (by address, channels beyond C repeating the last one: 247 -> 77 3x3 on 63 x 64 18.9 us, by descriptor 20.2; 163 -> 93
          // stride 2 on 10 x 44 x 44 17.1, 18.0)
          const int c = c0 + u_c[n] < p.C ? c0 + u_c[n] : p.C - 1;
          const int left = p.C - 1 - c;
          uint32_t at = off + (uint32_t)c * (uint32_t)HW + (uint32_t)ixc;
#pragma unroll
          for (int k = 0; k < 16; ++k) raw[n][k] = 0;
          if (u_mask[n]) {
#pragma unroll
            for (int k = 0; k < 16; ++k) {
              raw[n][k] = *reinterpret_cast<const u32_any*>(p.act + at);
              at += k < left ? (uint32_t)HW : 0u;
            }
          }
          continue;
        }
        const uint32_t at = u_mask[n] ? off + (uint32_t)(c0 + u_c[n]) * (uint32_t)HW + (uint32_t)ixc : 0x80000000u;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          if (SMALL && k % 4 == 0 && k >= p.small_c) break;  // uniform
          raw[n][k] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs_act, at + (uint32_t)(k * HW), 0, 0);
        }
      }
    }
  };
  auto store_input = [&]() {
#pragma unroll
    for (int n = 0; n < NU; ++n) {
      if (n > 0 && NT * n >= units) break;  // uniform
      __builtin_amdgcn_sched_barrier(0);    // one unit's registers at a time
      if (u_v[n] < 0) continue;
      const uint32_t mask = NHWC ? (u_shift[n] < 0 ? 0u : 0xffffffffu) : u_mask[n], pad = p.pad4 & ~mask;
      uint8_t* dst = s_in + u_lds[n];
      if constexpr (NHWC) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = raw[n][i];
        if (u_shift[n] > 0) {
#pragma unroll
          for (int b = 0; b < 3; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = ((u_shift[n] >> (2 + b)) & 1) ? (i + (1 << b) < 4 ? w[i + (1 << b)] : 0u) : w[i];
#pragma unroll
          for (int i = 0; i < 4; ++i) w[i] = __builtin_amdgcn_alignbyte(i < 3 ? w[i + 1] : 0u, w[i], (uint32_t)(u_shift[n] & 3));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = ((w[i] ^ p.act_xor4) & mask) | pad;
        if constexpr (SMALL) {
          if (p.small_c == 4) *reinterpret_cast<uint32_t*>(dst) = w[0];
          else if (p.small_c == 8) *reinterpret_cast<uint2*>(dst) = make_uint2(w[0], w[1]);
          else *reinterpret_cast<uint4*>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
        } else {
          *reinterpret_cast<uint4*>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
        }
      } else {
        const int rs_ = u_shift[n] > 0 ? u_shift[n] : 0, ls_ = u_shift[n] < 0 ? -u_shift[n] : 0;
        auto write = [&](auto fix) {
          auto group = [&](int g, uint32_t (&o)[4]) {
            transpose4(fix(raw[n][4 * g]), fix(raw[n][4 * g + 1]), fix(raw[n][4 * g + 2]), fix(raw[n][4 * g + 3]), o);
          };
          uint32_t o[4][4];
          group(0, o[0]);
          if (SMALL && p.small_c == 4) {
            *reinterpret_cast<uint4*>(dst) = make_uint4(o[0][0], o[0][1], o[0][2], o[0][3]);
            return;
          }
          group(1, o[1]);
          if (SMALL && p.small_c == 8) {
            *reinterpret_cast<uint4*>(dst) = make_uint4(o[0][0], o[1][0], o[0][1], o[1][1]);
            *reinterpret_cast<uint4*>(dst + 16) = make_uint4(o[0][2], o[1][2], o[0][3], o[1][3]);
            return;
          }
          group(2, o[2]);
          group(3, o[3]);
#pragma unroll
          for (int i = 0; i < 4; ++i) *reinterpret_cast<uint4*>(dst + i * PS) = make_uint4(o[0][i], o[1][i], o[2][i], o[3][i]);
        };
        const uint32_t flip = p.act_xor4 & mask, whole = mask ? p.act_xor4 : p.pad4;
        if (p.aligned) write([&](uint32_t v) { return v ^ whole; });  // uniform: a dword lies inside the image or outside
        else write([&](uint32_t v) { return ((((v >> rs_) << ls_) & mask) ^ flip) | pad; });
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- weights of chunk c0, in batches of UB units per thread whose loads are issued together; channels and output
  // channels that do not exist are zero.  A unit: four channels' nine taps (WT 9), 16 channels of a tap (2), one dword (0).
  const int T = p.KH * p.KW;
  constexpr int UB = WT == 9 ? (WCH == 2 && !MULTI ? 4 : 2) : (SMALL ? 6 : 4), WD = WT == 9 ? 9 : (WT == 2 ? 4 : 1);
  uint32_t wraw[UB][WD];
  const int c4n = p.CC >> 2, c16n = p.CC >> 4;
  const int wper = WT == 9 ? c4n : (WT == 2 ? T * c16n : p.groups * 8);  // units per output channel
  const int wunits = OB * wper;
  // Units that are whole or nothing are loaded by descriptor, the ones beyond the channels out of its range (us with a
  // 64-bit address and conditions per unit and so: 48 -> 64 3x3 stride 2 on 16 x 56 x 56 9.1, 8.4, channel-last, all in
  // this kernel, 10.5, 9.1; 64 -> 128 on as many 8.9, 8.6).  Not units of nine dwords where channels come in chunks: 190 -> 132 3x3
  // stride 2 on 18 x 38 x 40 25.0, 24.3 without; 242 -> 244 on 13 x 27 x 30 22.1, 21.7.
  const int w_left = p.O - o0 < OB ? p.O - o0 : OB;
  const __amdgpu_buffer_rsrc_t rs_wgt = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t*>(p.wgt) + (int64_t)o0 * p.C * T, 0, w_left * p.C * T, 0x00020000);
  const bool w_whole = !SMALL && ((WT == 9 && !MULTI && p.C % 4 == 0) || (WT == 2 && p.C % 16 == 0));
  auto load_weights = [&](int c0, int i0) {
    if (w_whole) {  // uniform
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int i = i0 + u * NT + t;
        uint32_t ru;
        const int o = (int)divide((uint32_t)i, (uint32_t)wper, p.inv_wper, ru);
        if constexpr (WT == 9) {
          const int c = c0 + 4 * (int)ru;
          const uint32_t at = i < wunits && c < p.C ? (uint32_t)((o * p.C + c) * 9) : 0x80000000u;
#pragma unroll
          for (int k = 0; k < 9; ++k) wraw[u][k] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs_wgt, at + 4 * k, 0, 0);
        } else if constexpr (WT == 2) {
          uint32_t cu;
          const int tap = (int)divide(ru, (uint32_t)c16n, p.inv_c16, cu), c = c0 + 16 * (int)cu;
          const uint32_t at = i < wunits && c < p.C ? (uint32_t)((o * T + tap) * p.C + c) : 0x80000000u;
          const v4i v = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs_wgt, at, 0, 0));
#pragma unroll
          for (int k = 0; k < 4; ++k) wraw[u][k] = (uint32_t)v[k];
        }
      }
      return;
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int i = i0 + u * NT + t;
#pragma unroll
      for (int k = 0; k < WD; ++k) wraw[u][k] = 0;
      uint32_t ru;
      const int o = (int)divide((uint32_t)i, (uint32_t)wper, p.inv_wper, ru), r = (int)ru;
      if (i >= wunits || o0 + o >= p.O) continue;
      if constexpr (WT == 9) {
        const int left = p.C - c0 - 4 * r;
        const int8_t* src = p.wgt + ((int64_t)(o0 + o) * p.C + c0 + 4 * r) * 9;
        if (left >= 4) {
#pragma unroll
          for (int k = 0; k < 9; ++k) wraw[u][k] = *reinterpret_cast<const u32_any*>(src + 4 * k);
        } else {
#pragma unroll
          for (int b = 0; b < 27; ++b)
            if (b < 9 * left) wraw[u][b >> 2] |= (uint32_t)(uint8_t)src[b] << (8 * (b & 3));
        }
      } else if constexpr (WT == 2) {
        uint32_t cu;
        const int tap = (int)divide(ru, (uint32_t)c16n, p.inv_c16, cu);
        const int c16 = (int)cu * 16, left = p.C - c0 - c16;
        const int8_t* src = p.wgt + ((int64_t)(o0 + o) * T + tap) * p.C + c0 + c16;
        if (left >= 16) {
          const v4i v = *reinterpret_cast<const v4i_any*>(src);
#pragma unroll
          for (int k = 0; k < 4; ++k) wraw[u][k] = (uint32_t)v[k];
        } else {
#pragma unroll
          for (int b = 0; b < 15; ++b)
            if (b < left) wraw[u][b >> 2] |= (uint32_t)(uint8_t)src[b] << (8 * (b & 3));
        }
      } else {
        uint32_t cu;
        const int tap = (int)divide(4 * ru, (uint32_t)p.CC, p.inv_line, cu), c = (int)cu;  // (four channels of one tap)
        const int64_t first_c = ((int64_t)(o0 + o) * p.C + c0 + c) * T + tap;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (c0 + c + e < p.C) wraw[u][0] |= (uint32_t)(uint8_t)p.wgt[first_c + e * T] << (8 * e);
      }
    }
  };
  auto store_weights = [&](int i0, bool sums) {
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int i = i0 + u * NT + t;
      if (i >= wunits) continue;
      uint32_t ru;
      const int o = (int)divide((uint32_t)i, (uint32_t)wper, p.inv_wper, ru), r = (int)ru;
      int32_t part = 0;
      if constexpr (WT == 9) {
        // 36 bytes in memory: byte 9 j + k = channel j, tap k; tap k's dword is bytes (k, 9 + k, 18 + k, 27 + k)
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          constexpr uint32_t kKeep = 0x0c0c0000u;  // upper half zero
          const int i0_ = k, i1 = 9 + k, i2 = 18 + k, i3 = 27 + k;
          const uint32_t* dw = wraw[u];
          const uint32_t lo = __builtin_amdgcn_perm(dw[i1 >> 2], dw[i0_ >> 2], kKeep | (uint32_t)(i0_ & 3) | ((uint32_t)(4 + (i1 & 3)) << 8));
          const uint32_t hi = __builtin_amdgcn_perm(dw[i3 >> 2], dw[i2 >> 2], kKeep | (uint32_t)(i2 & 3) | ((uint32_t)(4 + (i3 & 3)) << 8));
          const uint32_t tap = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
          *reinterpret_cast<uint32_t*>(s_w + o * wstride + k * p.CC + 4 * r) = tap;
        }
      } else if constexpr (WT == 2) {
        *reinterpret_cast<uint4*>(s_w + o * wstride + 16 * r) = make_uint4(wraw[u][0], wraw[u][1], wraw[u][2], wraw[u][3]);
      } else {
        *reinterpret_cast<uint32_t*>(s_w + o * wstride + 4 * r) = wraw[u][0];
      }
      if (sums) {
#pragma unroll
        for (int k = 0; k < WD; ++k) part = __builtin_amdgcn_sdot4((int)wraw[u][k], 0x01010101, part, false);
        atomicAdd(&s_sum[o], part);
      }
    }
  };

  TilePos pos = tile_pos(tile);
  // few channels: the block's weights as one run of bytes
  const int small_bytes = SMALL ? (p.O - o0 < OB ? p.O - o0 : OB) * p.C * T : 0;
  auto load_run = [&](int i) {
    const int8_t* src = p.wgt + (int64_t)o0 * p.C * T + i;
    uint32_t w = 0;
    if (i + 4 <= small_bytes) w = *reinterpret_cast<const u32_any*>(src);
    else
      for (int e = 0; i + e < small_bytes; ++e) w |= (uint32_t)(uint8_t)src[e] << (8 * e);
    return w;
  };
  if constexpr (SMALL) {
#pragma unroll
    for (int u = 0; u < UB; ++u) wraw[u][0] = load_run(4 * (t + u * NT));
  }
  if constexpr (!MULTI && !SMALL) load_weights(0, 0);  // both in flight before anything is waited for
  load_input(pos, 0);
  const bool need_sum = p.corr_coef != 0;
  if (t == 0) *s_flag = 0;
  // a channel's constants stay in registers until its terms are formed: storing them here would wait for every load
  // before them
  static_assert(OB <= NT, "a thread has one output channel");
  int32_t c_bias = 0, c_mu = 0, c_sh = 1;
  if (t < OB) {
    const int o = o0 + t;
    s_sum[t] = 0;
    if (o < p.O) {
      if (p.bias) c_bias = p.bias[o];
      if (!RAW) {
        c_mu = rq_mult(p.mult, p.per_channel ? o : 0);
        c_sh = rq_shift(p.mult, p.shift, p.per_channel ? o : 0);
      }
    }
    if constexpr (kTight) {
      s_corr[t] = c_bias;
      s_mu[t] = c_mu;
      s_sh[t] = c_sh;
    }
  }

  // MFMA rows and columns: NCHW pixels x channels, row r of a 32-row block is pixel pix_perm(r) of it (a lane's 16
  // registers: 16 consecutive pixels of one channel); NHWC channels x pixels, row r is channel pix_perm(r).
  const int jp = NHWC ? j : pix_perm(j), jc = NHWC ? pix_perm(j) : j;
  const int pt = p.TR * p.TW;
  const uint8_t* b_ptr = s_w + (64 * wch + jc) * wstride + 16 * h;
  auto stage_weights = [&](int c0, bool loaded, bool sums) {  // loaded: the first batch is in registers
    for (int i0 = 0; i0 < wunits; i0 += UB * NT) {
      if (!loaded) load_weights(c0, i0);
      loaded = false;
      store_weights(i0, sums);
    }
  };
  // Few channels: the block's weights are one contiguous run of OB * C * T bytes; it is copied to LDS (where the input
  // goes later) and regrouped from there, a dword (four channels of a tap) at a time.
  auto stage_weights_small = [&](bool sums) {
    for (int i = 4 * (t + UB * NT); i < small_bytes; i += 4 * NT) *reinterpret_cast<uint32_t*>(s_in + i) = load_run(i);
#pragma unroll
    for (int u = 0; u < UB; ++u)
      if (4 * (t + u * NT) < small_bytes) *reinterpret_cast<uint32_t*>(s_in + 4 * (t + u * NT)) = wraw[u][0];
    __syncthreads();
    // a thread keeps its place in the row of an output channel (64 .. NT threads share the row)
    int shift = 6;
    while ((1 << shift) < wper && (1 << shift) < NT) ++shift;
    for (int r = t & ((1 << shift) - 1); r < wper; r += 1 << shift) {
      uint32_t rr, c;
      const int ky = (int)divide(4u * (uint32_t)r, (uint32_t)(p.NX * 32), p.inv_line, rr);  // filter row, byte in it
      const int kx = (int)divide(rr, (uint32_t)p.small_c, p.inv_bpp, c);
      const int tap = ky * p.KW + kx, at0 = NHWC ? tap * p.C + (int)c : (int)c * T + tap, step = NHWC ? 1 : T;
      const int nc = kx < p.KW ? p.C - (int)c : 0;  // channels of the dword that exist
      const uint32_t keep = nc >= 4 ? 0xffffffffu : nc <= 0 ? 0u : (1u << (8 * nc)) - 1u;
      // (Several output channels' bytes are read before the first dword is written, and addresses are only added to: one
      // channel at a time, with its addresses multiplied out and its bytes under conditions, took 2.4 us of a 7x7 layer, 1.2 so.)
      const int rows = p.O - o0 < OB ? p.O - o0 : OB, ostep = NT >> shift;
      int o = t >> shift, from = o * p.C * T + at0, to = o * wstride + 4 * r;
      for (int n = 0; n < OB / ostep; n += 4) {
        uint32_t w[4];
        auto read = [&](auto nconst) {
          constexpr int NC = decltype(nconst)::value;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            w[u] = s_in[from];
            if constexpr (NC > 1) w[u] |= (uint32_t)s_in[from + step] << 8;
            if constexpr (NC > 2) w[u] |= (uint32_t)s_in[from + 2 * step] << 16;
            if constexpr (NC > 3) w[u] |= (uint32_t)s_in[from + 3 * step] << 24;
            from += ostep * p.C * T;
          }
        };
        if (p.C == 1) read(std::integral_constant<int, 1>{});
        else if (p.C == 2) read(std::integral_constant<int, 2>{});
        else if (p.C == 3) read(std::integral_constant<int, 3>{});
        else read(std::integral_constant<int, 4>{});
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t v = o < rows ? w[u] & keep : 0u;
          if (o < OB) {
            *reinterpret_cast<uint32_t*>(s_w + to) = v;
            if (sums) atomicAdd(&s_sum[o], __builtin_amdgcn_sdot4((int)v, 0x01010101, 0, false));
          }
          o += ostep;
          to += ostep * wstride;
        }
      }
    }
  };
  bool first = true;  // the workgroup's first tile
  bool fold = false;
  const int32_t lo_abs = p.rs.lo_rel + p.rs.z_out, hi_abs = p.rs.hi_rel + p.rs.z_out;
  // results clipped to the container's whole range: shift, clip and pack of two are one instruction (the lane's channels
  // differ in the channel-last form, so it shifts first)
  constexpr bool sat = OUT == kFullCodes;
  const int32_t zc = p.rs.z_out + (sat ? sat_bias(p.rs) : 0);
  const uint32_t sflip = sat_flip(p.rs);
  int ch = 0;         // chunk
  v16i acc[AF][2];
  // The block's terms, when its weight sums are complete.  Folded requantize (32-bit accumulator, constants small enough in
  // every channel of the block): correction, rounding term and output zero point go into one 64-bit constant, the result is
  // the high dword of acc * m + k64 shifted by sh - 1; |acc| < 2^30 for reductions up to 2^16, so acc + corr cannot wrap.
  // Without chunks they are formed behind the staging of the weights, and the barrier behind the input's staging serves
  // them too (64 -> 128 3x3 stride 2 on 32 x 56 x 56: 10.3 us, 10.4 before; 3 -> 64 7x7 on 8 x 224 x 224,
  // with the input's loads by descriptor, one addition each, 10.6, 12.2 before).
  auto form_terms = [&]() {
    int bad = RAW || p.acc_wrap_shift != 0 || p.rs.half_away || p.rs.z_out < -256 || p.rs.z_out > 255 || p.C * T > 65536;
    if (t < OB) {
      if constexpr (kTight) {
        c_bias = s_corr[t];
        c_mu = s_mu[t];
        c_sh = s_sh[t];
      }
      const int32_t corr = c_bias + (need_sum ? p.corr_coef * s_sum[t] : 0), mu = c_mu, sh = c_sh;
      bad |= sh < 1 || sh > 19 || corr < -(1 << 30) || corr > (1 << 30);
      const int64_t k64 = (int64_t)corr * mu + ((int64_t)1 << (30 + (sh & 31))) + ((int64_t)zc << (31 + (sh & 31)));
      s_corr[t] = corr;
      s_mu[t] = mu;
      s_sh[t] = sh;
      s_fold[t] = make_int4((int)(uint32_t)k64, (int)(k64 >> 32), mu, sh - 1);
    }
    if (!RAW && bad) atomicOr(s_flag, 1);
    if (MULTI) __syncthreads();
  };
  if constexpr (!MULTI) {  // resident for every tile
    __syncthreads();
    if constexpr (SMALL) stage_weights_small(need_sum);
    else stage_weights(0, true, need_sum);
  }
  for (;;) {
    __syncthreads();   // the previous chunk has been consumed
    if constexpr (MULTI) stage_weights(ch * p.CC, false, first && need_sum);
    if (!MULTI && first) form_terms();
    store_input();     // registers -> LDS
    __syncthreads();
    // the next chunk's or tile's loads go out now
    const bool last = !MULTI || ch + 1 == p.nchunk;
    const bool more = !last || tile + tile_step < tile_end;
    const TilePos next_pos = last && more ? tile_pos(tile + tile_step) : pos;
    if (more) load_input(next_pos, last ? 0 : (ch + 1) * p.CC);

    // the lane's pixels: LDS offset of the first tap
    uint32_t a_base[AF];
#pragma unroll
    for (int f = 0; f < AF; ++f) {
      const int q = 32 * (AF * wpx + f) + jp;
      uint32_t x, oy;
      const uint32_t r = divide((uint32_t)(q < pt ? q : 0), (uint32_t)p.TW, p.inv_tw, x);  // (rows beyond the tile read pixel 0)
      uint32_t R = (uint32_t)pos.R0 + r;
      const uint32_t Rmax = (uint32_t)(p.B * p.OH - 1);
      if (R > Rmax) R = Rmax;
      const uint32_t b = divide(R, (uint32_t)p.OH, p.inv_oh, oy);
      a_base[f] = (b * (uint32_t)p.HV + oy * (uint32_t)p.sr - (uint32_t)pos.V0) * (uint32_t)rowB + (x * (uint32_t)p.sw + (uint32_t)p.off_x) * (uint32_t)PS + 16u * h;
    }
    if (!MULTI || ch == 0) {
#pragma unroll
      for (int f = 0; f < AF; ++f)
#pragma unroll
        for (int tn = 0; tn < 2; ++tn)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[f][tn][r] = 0;
    }
      // ---- implicit GEMM over the chunk's groups; the fragments of the next group are requested before the
      // matrix instructions of the current one
      {
        v4i bq[2][2], aq[2][AF];
        int x = 0, c = 0, g = 0;
        uint32_t a_off = 0, a_line = 0;
        auto fetch = [&](int buf) {
          const uint8_t* bp = b_ptr + 32 * g;
          bq[buf][0] = *reinterpret_cast<const v4i*>(bp);
          bq[buf][1] = *reinterpret_cast<const v4i*>(bp + 32 * wstride);
          typedef int v4i_dword __attribute__((ext_vector_type(4), aligned(4)));
          if constexpr (SMALL) {
#pragma unroll
            for (int f = 0; f < AF; ++f) aq[buf][f] = *reinterpret_cast<const v4i_dword*>(s_in + a_base[f] + a_off);
          } else {
#pragma unroll
            for (int f = 0; f < AF; ++f) aq[buf][f] = *reinterpret_cast<const v4i*>(s_in + a_base[f] + a_off);
          }
          // advance (scalar): 32 bytes along the channels, then along the filter row, then the next row
          ++g;
          if (++c < p.CK) {
            a_off += 32;
          } else {
            c = 0;
            if (++x < p.NX) {
              a_off = a_line + (uint32_t)(x * p.xB);
            } else {
              x = 0;
              a_line += (uint32_t)rowB;
              a_off = a_line;
            }
          }
        };
        auto mul = [&](int buf) {
#pragma unroll
          for (int f = 0; f < AF; ++f)
#pragma unroll
            for (int tn = 0; tn < 2; ++tn)
              acc[f][tn] = NHWC ? __builtin_amdgcn_mfma_i32_32x32x32_i8(bq[buf][tn], aq[buf][f], acc[f][tn], 0, 0, 0)
                                : __builtin_amdgcn_mfma_i32_32x32x32_i8(aq[buf][f], bq[buf][tn], acc[f][tn], 0, 0, 0);
        };
        const int n = p.groups;
        fetch(0);
        int s = 0;
        for (; s + 2 < n; s += 2) {
          fetch(1);
          __builtin_amdgcn_sched_barrier(0);
          mul(0);
          __builtin_amdgcn_sched_barrier(0);
          fetch(0);
          __builtin_amdgcn_sched_barrier(0);
          mul(1);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (s + 1 < n) {
          fetch(1);
          mul(0);
          mul(1);
        } else {
          mul(0);
        }
      }
    if (!last) {
      ++ch;
      continue;
    }
    ch = 0;
    if (first && MULTI) form_terms();  // (the sums of the last chunk are complete)
    if (first) fold = !RAW && *s_flag == 0;
    first = false;

    // ---- epilogue
    const uint32_t Rend = (uint32_t)(p.B * p.OH);
    const int esz = out_mode == 0 ? 1 : (out_mode == 1 ? 4 : 2);
    if constexpr (NHWC) {
#pragma unroll
      for (int f = 0; f < AF; ++f) {
        const int q = 32 * (AF * wpx + f) + j;
        uint32_t x;
        const uint32_t r = divide((uint32_t)q, (uint32_t)p.TW, p.inv_tw, x);
        const uint32_t R = (uint32_t)pos.R0 + r;
        const int ox = pos.x0 + (int)x;
        const bool px_ok = q < pt && R < Rend && ox < p.OW;
        const int64_t prow = ((int64_t)R * p.OW + ox) * p.O;
        if (p.through && (out_mode != 0 || (fold && sat))) {  // (uniform) four lanes write 64 consecutive bytes of a pixel
          // through the L2 (3 -> 64 7x7 stride 2 on 8 x 224 x 224: raw 20.5 us with 16 bytes per lane to 32 pixels, 13.3 so, 16 bits 15.7, 11.8, one byte
          // 12.8, 12.2)
          // pixel q of the tile, which another lane has the results of
          auto at_pixel = [&](int q, int64_t& row) {
            uint32_t x;
            const uint32_t r = divide((uint32_t)q, (uint32_t)p.TW, p.inv_tw, x);
            const uint32_t R = (uint32_t)pos.R0 + r;
            const int ox = pos.x0 + (int)x;
            row = ((int64_t)R * p.OW + ox) * p.O;
            return q < pt && R < Rend && ox < p.OW;
          };
          const int at = stay_here(lane), q_first = 32 * (AF * wpx + f);
          if (out_mode == 0) {
            uint32_t dw[2][4];
#pragma unroll
            for (int tn = 0; tn < 2; ++tn)
#pragma unroll
              for (int g = 0; g < 4; ++g) {
                int32_t y[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  const int4 k = s_fold[64 * wch + 32 * tn + 16 * h + 4 * g + e];
                  y[e] = (int32_t)(((int64_t)acc[f][tn][4 * g + e] * (int64_t)k.z + (int64_t)(((uint64_t)(uint32_t)k.y << 32) | (uint32_t)k.x)) >> 32) >> k.w;
                }
                ashr_sat_pair<0>(dw[tn][g], y[0], y[1], 0);
                ashr_sat_pair<1>(dw[tn][g], y[2], y[3], 0);
                dw[tn][g] ^= sflip;
                __builtin_amdgcn_sched_barrier(0);  // (four products at a time)
              }
            swap_sixteens(dw[0], dw[1]);
            const int o = o0 + 64 * wch + 32 * ((at >> 4) & 1) + 16 * (at >> 5);
#pragma unroll
            for (int g = 0; g < 2; ++g) {
              int64_t row;
              if (at_pixel(q_first + 16 * g + (at & 15), row) && o < p.O)
                store_through(static_cast<uint8_t*>(p.out) + row + o, v4i{(int)dw[g][0], (int)dw[g][1], (int)dw[g][2], (int)dw[g][3]});
            }
            continue;
          }
#pragma unroll
          for (int tn = 0; tn < 2; ++tn) {
            __builtin_amdgcn_sched_barrier(0);  // one group of results at a time
            const int32_t* const corr = s_corr + 64 * wch + 32 * tn + 16 * h;
            if (out_mode == 1) {
              uint32_t v[4][4];
#pragma unroll
              for (int g = 0; g < 4; ++g) {
                const int4 c4 = *reinterpret_cast<const int4*>(corr + 4 * g);
                const int32_t cc[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) v[g][e] = (uint32_t)wrap_acc_bits(acc[f][tn][4 * g + e] + cc[e], p.acc_wrap_shift);
              }
              quad_transpose(v, lane);
              const int o = o0 + 64 * wch + 32 * tn + 16 * (at >> 5) + 4 * (at & 3);
#pragma unroll
              for (int t4 = 0; t4 < 4; ++t4) {
                int64_t row;
                if (at_pixel(q_first + (at & 28) + t4, row) && o < p.O)
                  store_through(static_cast<int32_t*>(p.out) + row + o, v4i{(int)v[t4][0], (int)v[t4][1], (int)v[t4][2], (int)v[t4][3]});
              }
            } else {
              uint32_t dq[2][4];
#pragma unroll
              for (int y = 0; y < 8; ++y)
                dq[y >> 2][y & 3] = ((uint32_t)(acc[f][tn][2 * y] + corr[2 * y]) & 0xffffu) | ((uint32_t)(acc[f][tn][2 * y + 1] + corr[2 * y + 1]) << 16);
              swap_sixteens(dq[0], dq[1]);
              const int o = o0 + 64 * wch + 32 * tn + 16 * (at >> 5) + 8 * ((at >> 4) & 1);
#pragma unroll
              for (int g = 0; g < 2; ++g) {
                int64_t row;
                if (at_pixel(q_first + 16 * g + (at & 15), row) && o < p.O)
                  store_through(static_cast<int16_t*>(p.out) + row + o, v4i{(int)dq[g][0], (int)dq[g][1], (int)dq[g][2], (int)dq[g][3]});
              }
            }
          }
          continue;
        }
#pragma unroll
        for (int tn = 0; tn < 2; ++tn) {
          __builtin_amdgcn_sched_barrier(0);  // one group of results at a time
          const int cl = 64 * wch + 32 * tn + 16 * h, o = o0 + cl;  // 16 consecutive channels
          if (!px_ok || o >= p.O) continue;
          const int left = p.O - o;
          if (fold && sat) {  // uniform
            uint32_t dw[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              int32_t y[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const int4 k = s_fold[cl + 4 * g + e];
                y[e] = (int32_t)(((int64_t)acc[f][tn][4 * g + e] * (int64_t)k.z + (int64_t)(((uint64_t)(uint32_t)k.y << 32) | (uint32_t)k.x)) >> 32) >> k.w;
              }
              ashr_sat_pair<0>(dw[g], y[0], y[1], 0);
              ashr_sat_pair<1>(dw[g], y[2], y[3], 0);
              dw[g] ^= sflip;
              __builtin_amdgcn_sched_barrier(0);  // (four products at a time)
            }
            uint8_t* dst = static_cast<uint8_t*>(p.out) + prow + o;
            if (left >= 16) {  // one store of 16 bytes: a store per dword is a pass of the memory pipe per lane each
              *reinterpret_cast<v4i_any*>(dst) = v4i{(int)dw[0], (int)dw[1], (int)dw[2], (int)dw[3]};
            } else {
#pragma unroll
              for (int g = 0; g < 4; ++g) {
                if (4 * g + 4 <= left) {
                  *reinterpret_cast<u32_any*>(dst + 4 * g) = dw[g];
                } else {
#pragma unroll
                  for (int e = 0; e < 3; ++e)
                    if (4 * g + e < left) dst[4 * g + e] = (uint8_t)(dw[g] >> (8 * e));
                }
              }
            }
            continue;
          }
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            int32_t v[4];
            if (!sat && fold) {
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const int4 k = s_fold[cl + 4 * g + e];
                const int64_t pr = (int64_t)acc[f][tn][4 * g + e] * (int64_t)k.z + (int64_t)(((uint64_t)(uint32_t)k.y << 32) | (uint32_t)k.x);
                v[e] = med3((int32_t)(pr >> 32) >> k.w, lo_abs, hi_abs);
              }
            } else {
              const int4 c4 = *reinterpret_cast<const int4*>(s_corr + cl + 4 * g);
              const int4 m4 = *reinterpret_cast<const int4*>(s_mu + cl + 4 * g);
              const int4 h4 = *reinterpret_cast<const int4*>(s_sh + cl + 4 * g);
              const int32_t cc[4] = {c4.x, c4.y, c4.z, c4.w}, mm[4] = {m4.x, m4.y, m4.z, m4.w}, hh[4] = {h4.x, h4.y, h4.z, h4.w};
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                v[e] = acc[f][tn][4 * g + e] + cc[e];
                if (p.acc_wrap_shift) v[e] = wrap_acc_bits(v[e], p.acc_wrap_shift);
                if (out_mode == 0) v[e] = requant_general(v[e], mm[e], hh[e], p.rs);
              }
            }
            uint8_t* dst = static_cast<uint8_t*>(p.out) + (prow + o + 4 * g) * esz;
            if (4 * g + 4 <= left) {
              if (out_mode == 0) {
                *reinterpret_cast<u32_any*>(dst) = pack4_perm(v[0], v[1], v[2], v[3]);
              } else if (out_mode == 1) {
                *reinterpret_cast<v4i_any*>(dst) = v4i{v[0], v[1], v[2], v[3]};
              } else {
                *reinterpret_cast<u32_any*>(dst) = ((uint32_t)v[0] & 0xffffu) | ((uint32_t)v[1] << 16);
                *reinterpret_cast<u32_any*>(dst + 4) = ((uint32_t)v[2] & 0xffffu) | ((uint32_t)v[3] << 16);
              }
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (4 * g + e < left) {
                  if (out_mode == 0) dst[e] = (uint8_t)v[e];
                  else if (out_mode == 1) reinterpret_cast<int32_t*>(dst)[e] = v[e];
                  else reinterpret_cast<int16_t*>(dst)[e] = (int16_t)v[e];
                }
            }
          }
        }
      }
    } else {
      const int OHW = p.OH * p.OW;
#pragma unroll
      for (int tn = 0; tn < 2; ++tn) {
        const int cl = 64 * wch + 32 * tn + j, o = o0 + cl;
        if (AF == 2 && fold && sat && p.through) {  // (uniform)
          // Sixteen pixels of both row blocks: 64 bytes of a channel by four lanes, through the L2 (3 -> 64 7x7 stride 2 on 8 x 224 x 224 10.6 us
          // with a lane's own sixteen bytes left there, 9.7 so).
          const int4 k = s_fold[cl];
          const int64_t k64 = (int64_t)(((uint64_t)(uint32_t)k.y << 32) | (uint32_t)k.x);
          uint32_t dw[AF][4];
#pragma unroll
          for (int f = 0; f < AF; ++f)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              int32_t y[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) y[e] = (int32_t)(((int64_t)acc[f][tn][4 * g + e] * (int64_t)k.z + k64) >> 32);
              ashr_sat_pair<0>(dw[f][g], y[0], y[1], k.w);
              ashr_sat_pair<1>(dw[f][g], y[2], y[3], k.w);
              dw[f][g] ^= sflip;
              __builtin_amdgcn_sched_barrier(0);  // (four products at a time: all sixteen would spill)
            }
          swap_sixteens(dw[0], dw[AF - 1]);
          const int at = stay_here(lane), q0 = 32 * (AF * wpx + ((at >> 4) & 1)) + 16 * (at >> 5);
          uint32_t x, oy;
          const uint32_t r = divide((uint32_t)q0, (uint32_t)p.TW, p.inv_tw, x);
          const uint32_t R = (uint32_t)pos.R0 + r;
          const uint32_t b = divide(R, (uint32_t)p.OH, p.inv_oh, oy);
          const int ox = pos.x0 + (int)x, from = o0 + 64 * wch + 32 * tn + (at & 15);
          if (q0 < pt && R < Rend && ox < p.OW) {
            uint8_t* const dst = static_cast<uint8_t*>(p.out) + (((int64_t)b * p.O + from) * OHW + (int)oy * p.OW + ox);
            typedef uint32_t v4u __attribute__((ext_vector_type(4)));
            if (from < p.O) store_through(dst, v4u{dw[0][0], dw[0][1], dw[0][2], dw[0][3]});
            if (from + 16 < p.O) store_through(dst + (int64_t)16 * OHW, v4u{dw[AF - 1][0], dw[AF - 1][1], dw[AF - 1][2], dw[AF - 1][3]});
          }
          continue;
        }
        if (out_mode != 0 && p.through) {  // (uniform) raw: pieces of 16 bytes by lanes that write 64 consecutive ones of a channel
          // (3 -> 64 7x7 stride 2 on 8 x 224 x 224, 16 bytes per lane to 32 channels and so: 17.8 us, 11.5, 16 bits 12.4, 10.85; 64 -> 128 3x3
          // stride 2 on 32 x 56 x 56 15.1, 11.65)
#pragma unroll
          for (int f = 0; f < AF; ++f) {
            __builtin_amdgcn_sched_barrier(0);  // one group of results at a time
            const int32_t corr = s_corr[stay_here(cl)];
            const int at = stay_here(lane), wide = out_mode == 1;
            const int q0 = 32 * (AF * wpx + f) + 16 * (at >> 5) + (wide ? 4 * (at & 3) : 8 * ((at >> 4) & 1));
            const int from = o0 + 64 * wch + 32 * tn + (wide ? at & 28 : at & 15);
            uint32_t x, oy;
            const uint32_t r = divide((uint32_t)q0, (uint32_t)p.TW, p.inv_tw, x);
            const uint32_t R = (uint32_t)pos.R0 + r;
            const uint32_t b = divide(R, (uint32_t)p.OH, p.inv_oh, oy);
            const int ox = pos.x0 + (int)x;
            const bool ok = q0 < pt && R < Rend && ox < p.OW;
            uint8_t* const dst = static_cast<uint8_t*>(p.out) + (((int64_t)b * p.O + from) * OHW + (int)oy * p.OW + ox) * esz;
            if (wide) {
              uint32_t v[4][4];
#pragma unroll
              for (int e = 0; e < 16; ++e) v[e >> 2][e & 3] = (uint32_t)wrap_acc_bits(acc[f][tn][e] + corr, p.acc_wrap_shift);
              quad_transpose(v, lane);
#pragma unroll
              for (int t4 = 0; t4 < 4; ++t4)
                if (ok && from + t4 < p.O) store16(true, dst + (int64_t)t4 * OHW * 4, v[t4][0], v[t4][1], v[t4][2], v[t4][3]);
            } else {
              uint32_t dq[2][4];
#pragma unroll
              for (int y = 0; y < 8; ++y)  // (the low sixteen bits are the wrapped sum's for any accumulator of at least that width)
                dq[y >> 2][y & 3] = ((uint32_t)(acc[f][tn][2 * y] + corr) & 0xffffu) | ((uint32_t)(acc[f][tn][2 * y + 1] + corr) << 16);
              swap_sixteens(dq[0], dq[1]);
#pragma unroll
              for (int g = 0; g < 2; ++g)
                if (ok && from + 16 * g < p.O) store16(true, dst + (int64_t)(16 * g) * OHW * 2, dq[g][0], dq[g][1], dq[g][2], dq[g][3]);
            }
          }
          continue;
        }
        const int32_t corr = s_corr[cl], mu = s_mu[cl], sh = s_sh[cl], s1 = sh - 1;
        const int4 k = s_fold[cl];
        const int64_t k64 = (int64_t)(((uint64_t)(uint32_t)k.y << 32) | (uint32_t)k.x);
        // the clip moved in front of the shift, which then drops each result into its byte of the output dword
        const int32_t lo_s = clip_lo_before_shift(lo_abs, s1 & 31), hi_s = clip_hi_before_shift(hi_abs, s1 & 31);
#pragma unroll
        for (int f = 0; f < AF; ++f) {
          __builtin_amdgcn_sched_barrier(0);  // one group of results at a time
          const int q0 = 32 * (AF * wpx + f) + 16 * h;  // the lane's 16 consecutive pixels of the tile
          if (o >= p.O || q0 >= pt) continue;
          uint32_t x, oy;
          const uint32_t r = divide((uint32_t)q0, (uint32_t)p.TW, p.inv_tw, x);
          const uint32_t R = (uint32_t)pos.R0 + r;
          if (R >= Rend) continue;
          const uint32_t b = divide(R, (uint32_t)p.OH, p.inv_oh, oy);
          int32_t v[16];
          uint32_t dw[4];
          if (fold && sat) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              int32_t y[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) y[e] = (int32_t)(((int64_t)acc[f][tn][4 * g + e] * (int64_t)mu + k64) >> 32);
              ashr_sat_pair<0>(dw[g], y[0], y[1], s1);
              ashr_sat_pair<1>(dw[g], y[2], y[3], s1);
              dw[g] ^= sflip;
              __builtin_amdgcn_sched_barrier(0);  // (four products at a time: all sixteen would spill)
            }
          } else if (!sat && fold) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              auto one = [&]<int E>() {
                const int64_t pr = (int64_t)acc[f][tn][4 * g + E] * (int64_t)mu + k64;
                ashr_into_byte<E>(dw[g], med3((int32_t)(pr >> 32), lo_s, hi_s), s1);
              };
              one.template operator()<0>();
              one.template operator()<1>();
              one.template operator()<2>();
              one.template operator()<3>();
              __builtin_amdgcn_sched_barrier(0);  // (four products at a time: all sixteen would spill)
            }
          } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              v[e] = acc[f][tn][e] + corr;
              if (p.acc_wrap_shift) v[e] = wrap_acc_bits(v[e], p.acc_wrap_shift);
              if (out_mode == 0) v[e] = requant_general(v[e], mu, sh, p.rs);
            }
            if (out_mode == 0)
#pragma unroll
              for (int g = 0; g < 4; ++g) dw[g] = pack4_perm(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]);
          }
          // The 16 pixels are contiguous in the image when the tile is as wide as it, or inside one row of a segment
          // (16 divides TW then); they may end with the image, the segment or the tile.
          const int ox = pos.x0 + (int)x;
          const int pix = (int)oy * p.OW + ox;
          int cnt = pt - q0;                                  // pixels left in the tile
          const int in_img = p.nseg == 1 ? OHW - pix : p.OW - ox;  // ... in the image / in the row
          if (p.nseg > 1 && ox >= p.OW) continue;
          uint8_t* dst = static_cast<uint8_t*>(p.out) + (((int64_t)b * p.O + o) * OHW + pix) * esz;
          if (cnt >= 16 && in_img >= 16) {
            if (out_mode == 0) {
              *reinterpret_cast<v4i_any*>(dst) = v4i{(int)dw[0], (int)dw[1], (int)dw[2], (int)dw[3]};
            } else if (out_mode == 1) {
#pragma unroll
              for (int g = 0; g < 4; ++g) *reinterpret_cast<v4i_any*>(dst + 16 * g) = v4i{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
            } else {
#pragma unroll
              for (int g = 0; g < 2; ++g) {
                int dq[4];
#pragma unroll
                for (int y = 0; y < 4; ++y) dq[y] = (int)(((uint32_t)v[8 * g + 2 * y] & 0xffffu) | ((uint32_t)v[8 * g + 2 * y + 1] << 16));
                *reinterpret_cast<v4i_any*>(dst + 16 * g) = v4i{dq[0], dq[1], dq[2], dq[3]};
              }
            }
          } else {
            // in fours or one by one; past the end of an image the next one's plane of this channel follows C planes later
            int64_t rest = (int64_t)(Rend - R) * p.OW - (int64_t)x;  // pixels until the last image ends (nseg == 1)
            if (p.nseg > 1) rest = in_img;
            if (cnt > rest) cnt = (int)rest;
            const int64_t jump = (int64_t)(p.O - 1) * OHW;
            uint8_t* d = dst;
            int until = in_img;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              if (4 * g + 4 <= cnt && until >= 4) {
                if (out_mode == 0) *reinterpret_cast<u32_any*>(d) = dw[g];
                else if (out_mode == 1) *reinterpret_cast<v4i_any*>(d) = v4i{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
                else {
                  *reinterpret_cast<u32_any*>(d) = ((uint32_t)v[4 * g] & 0xffffu) | ((uint32_t)v[4 * g + 1] << 16);
                  *reinterpret_cast<u32_any*>(d + 4) = ((uint32_t)v[4 * g + 2] & 0xffffu) | ((uint32_t)v[4 * g + 3] << 16);
                }
                d += 4 * esz;
                until -= 4;
                if (until == 0) { d += jump * esz; until = OHW; }
              } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                  if (4 * g + e < cnt) {
                    if (out_mode == 0) *d = (uint8_t)(dw[g] >> (8 * e));
                    else if (out_mode == 1) *reinterpret_cast<int32_t*>(d) = v[4 * g + e];
                    else *reinterpret_cast<int16_t*>(d) = (int16_t)v[4 * g + e];
                    d += esz;
                    if (--until == 0) { d += jump * esz; until = OHW; }
                  }
              }
            }
          }
        }
      }
    }
    if (!more) break;
    tile += tile_step;
    pos = next_pos;
  }
}

template <bool NHWC, bool SMALL, bool MULTI, int WT, int WPX, int WCH, int AF, int OUT>
hipError_t launch_cd(const CdParams& p, size_t lds, int64_t grid, hipStream_t st) {
  auto kern = conv_direct_kernel<NHWC, SMALL, MULTI, WT, WPX, WCH, AF, OUT>;
  static std::atomic<uint64_t> attr_set{0};
  hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), 160 * 1024, attr_set);
  if (e != hipSuccess) return e;
  return launch_kernel(kern, dim3((unsigned)grid), dim3(64 * WPX * WCH), lds, st, p);
}

template <bool NHWC, bool SMALL, int WT, int OUT>
hipError_t launch_cd_shape(const CdParams& p, int shape, size_t lds, int64_t grid, hipStream_t st) {
  if constexpr (!SMALL) {
    if (p.nchunk > 1)  // (64 pixels per wavefront and weights restaged in the loop do not fit the registers)
      return shape == 1 ? launch_cd<NHWC, false, true, WT, 8, 1, 1, OUT>(p, lds, grid, st)
                        : launch_cd<NHWC, false, true, WT, 4, 2, 1, OUT>(p, lds, grid, st);
  }
  switch (shape) {
    case 0: return launch_cd<NHWC, SMALL, false, WT, 8, 1, 2, OUT>(p, lds, grid, st);
    case 1: return launch_cd<NHWC, SMALL, false, WT, 8, 1, 1, OUT>(p, lds, grid, st);
    default: return launch_cd<NHWC, SMALL, false, WT, 4, 2, 1, OUT>(p, lds, grid, st);
  }
}

}  // namespace

template <int OUT>
hipError_t launch_conv_direct(const CdParams& p, bool nhwc, int wt, int shape, size_t lds, int64_t grid, hipStream_t st) {
  if (nhwc) return p.small_c ? launch_cd_shape<true, true, 0, OUT>(p, shape, lds, grid, st) : launch_cd_shape<true, false, 2, OUT>(p, shape, lds, grid, st);
  if (p.small_c) return launch_cd_shape<false, true, 0, OUT>(p, shape, lds, grid, st);
  if (wt == 2) return launch_cd_shape<false, false, 2, OUT>(p, shape, lds, grid, st);
  if (wt == 9) return launch_cd_shape<false, false, 9, OUT>(p, shape, lds, grid, st);
  return launch_cd_shape<false, false, 0, OUT>(p, shape, lds, grid, st);
}

}  // namespace hago
