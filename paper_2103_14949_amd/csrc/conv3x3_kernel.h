// 3x3 stride-1 pad-1 convolution (groups == 1) on NCHW tensors in ONE launch, straight from the
// caller's buffers: no rewritten copy of the input, no scratch memory.
//
// The int8 matrix instruction wants 16 consecutive reduction bytes per lane, and in NCHW the
// reduction index (input channel) is the slow one.  The transposition therefore happens on the
// way into LDS: a workgroup owns TR whole output rows of one image (TR * W <= 32 * NW * AF pixels) and
// a block of 32 or 64 output channels.  It stages
//   - the input rows it needs, with their one-pixel halo, channel-last: [TR + 2][W + 2][C + 16]
//     bytes (uint8 inputs flipped to int8, everything outside the image filled with the zero
//     point, so padded taps contribute 0 under the zero-point identity of the GEMM kernels).  The
//     TR + 2 rows of one channel are one contiguous run in memory; a thread loads, for 16
//     channels, the dword of four pixels of that run (consecutive lanes, consecutive dwords),
//     transposes the 16 x 4 bytes in registers and writes 16 bytes per pixel;
//   - its weights, once, as [o][tap][C] (+16 bytes per o): the workgroup is persistent and walks
//     over pixel tiles with the weights resident.
// The loads of the NEXT tile are issued before the current one is multiplied and are written to
// LDS after it, so memory latency hides behind the matrix instructions and the epilogue.  The
// start-up chain is what bounds small layers and half of a layer of one tile per workgroup: all first loads, of the
// weights, the tile and the per-channel constants, go out by descriptor before any is waited for, divisions are
// multiplications by inverses (us before and so: 64 -> 64 on one 56 x 56 image 5.06, 4.65, on 16 of uint8 7.5, 6.8; 32 ->
// 72 on 28 x 48 x 48 7.7, 6.85; 128 -> 128 on 64 x 28 x 28 14.2, 13.6), and the weight sums of the zero-point term are added up
// (LDS atomics) by the threads that stage the weights, only when that term is not zero.  (Weights loaded as they lie and
// regrouped through LDS: 0.1 to 0.3 us slower; the tile's loads first: 0.1 to 0.4.)
// The 16 bytes of padding per pixel / per output channel make the 16-byte fragment reads of 32
// consecutive pixels (or channels) conflict-free (strides of 20 or 36 dwords).  A filter tap is
// then just an address offset into the staged tile, so every input byte is fetched once.
//
// MFMA orientation: pixels are the P operand (rows of the 32x32 tile), output channels the Q
// operand, so a lane owns one output channel and, per accumulator, 16 pixels.  Row r of a 32-row
// block holds pixel perm(r) of the block, chosen so that a lane's 16 registers are 16 CONSECUTIVE
// pixels: one 16-byte store per channel.
#pragma once

#include "conv3x3.h"

namespace hago {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef int v4i_any __attribute__((ext_vector_type(4), aligned(1)));  // results go out at any alignment
typedef uint32_t u32_any __attribute__((aligned(1)));

constexpr uint32_t kOob = 0x80000000u;  // a buffer offset that reads as 0

// n / d for n * d < 2^32 (inv == 0: d is 1, or n too large for that)
__device__ __forceinline__ uint32_t div_by(uint32_t n, uint32_t d, uint32_t inv) {
  return inv ? __umulhi(n, inv) : n / d;
}

// row r of a 32-row block <-> pixel of the block (see the header)
__device__ __forceinline__ constexpr int pix_of_row(int r) {
  return 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3);
}

// 4 channels x 4 pixels (a..d: the dwords of four consecutive channels) -> per pixel the dword
// of its four channels
__device__ __forceinline__ void transpose4(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t flip,
                                           uint32_t (&o)[4]) {
  const uint32_t t0 = __builtin_amdgcn_perm(b, a, 0x05010400u);  // a0 b0 a1 b1
  const uint32_t t1 = __builtin_amdgcn_perm(b, a, 0x07030602u);  // a2 b2 a3 b3
  const uint32_t t2 = __builtin_amdgcn_perm(d, c, 0x05010400u);
  const uint32_t t3 = __builtin_amdgcn_perm(d, c, 0x07030602u);
  o[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u) ^ flip;
  o[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u) ^ flip;
  o[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u) ^ flip;
  o[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u) ^ flip;
}

// NW: wavefronts per workgroup; AF: 32-pixel MFMA row blocks per wavefront (tiles of 32 * NW * AF
// pixels); NU: staging units per thread; CK: input channels / 32.
// OUT: the results, each in a kernel of its own (us in one kernel for all and so: raw 64 -> 64 on 64 x 56 x 56 17.3, 16.85, 16 bits 14.15, 13.6;
// 128 -> 128 on 64 x 28 x 28, 16 bits, 14.9, 14.2; 64 -> 64 on 16 x 56 x 56 7.04, 6.83).  kFull: codes clipped to their container's whole
// range, of a 32-bit accumulator; kClipped: all others (one kernel for both and so: one image of 64 -> 64 on 56 x 56 4.67 us, 4.52, 32 -> 96 on
// 8 x 28 x 28 4.29, 4.12, 128 -> 128 on 64 x 28 x 28 13.3, 13.0).
template <int NW, int AF, int NU, int CK, int TN, int OUT>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) void conv3x3_nchw_kernel(C3Params p) {
  constexpr int NT = 64 * NW;
  constexpr bool kBytes = OUT == kFull || OUT == kClipped;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  constexpr int C = 32 * CK;
  const int H = p.H, W = p.W, O = p.O;
  constexpr int Cp = C + 16;           // bytes per staged pixel
  const int Wp = W + 2;
  constexpr int wstride = 9 * C + 16;  // bytes per staged output channel
  const int HW = H * W;
  // Workgroups that share a pixel tile (one per block of output channels) read the same input,
  // and neighbouring tiles of an image share their halo rows.  Consecutive workgroup ids go round
  // the 8 XCDs, each with an L2 of its own, so the block index is taken from the id divided by 8
  // (the sharers land on one XCD) and each XCD walks a contiguous eighth of the tiles.
  int blk, tile, tile_end, tile_step;
  const int nwg = (int)gridDim.x / p.nblk;
  if (nwg % 8 == 0) {
    const int xcd = (int)blockIdx.x & 7, q = (int)blockIdx.x >> 3;
    const int per_xcd = (p.ntiles + 7) / 8;
    const int share = (int)div_by((uint32_t)q, (uint32_t)p.nblk, p.inv_nblk);
    blk = q - share * p.nblk;
    tile = xcd * per_xcd + share;
    tile_end = (xcd + 1) * per_xcd < p.ntiles ? (xcd + 1) * per_xcd : p.ntiles;
    tile_step = nwg / 8;
  } else {
    tile = (int)div_by(blockIdx.x, (uint32_t)p.nblk, p.inv_nblk);
    blk = (int)blockIdx.x - tile * p.nblk;
    tile_end = p.ntiles;
    tile_step = nwg;
  }
  constexpr int OB = 32 * TN;
  const int o0 = blk * OB;                             // this workgroup's block of output channels

  uint8_t* s_w = smem;                                 // [OB][wstride]
  uint8_t* s_in = smem + OB * wstride;                 // [(TR + 2)][Wp][Cp]
  int32_t* s_sum = reinterpret_cast<int32_t*>(s_in + (p.TR + 2) * Wp * Cp);  // [OB] weight sums

  // ---- staging units of a tile: (16-channel group, dword of the channel's run of TR + 2 rows)
  const int w4 = W >> 2;
  const int run4 = (p.TR + 2) * w4;                    // dwords per channel run
  const int units = (C >> 4) * run4;
  uint32_t raw[NU][16];                                // as loaded: [unit][channel] = four pixels
  int u_row[NU], u_off[NU];                            // row inside the tile (-1: no unit), LDS byte offset of the first pixel
  uint32_t u_src[NU];                                  // byte offset of the unit's first channel row start + column
#pragma unroll
  for (int n = 0; n < NU; ++n) {
    const int u = t + NT * n;
    u_row[n] = -1; u_off[n] = 0; u_src[n] = 0;
    if (u < units) {
      const int c16 = (int)div_by((uint32_t)u, (uint32_t)run4, p.inv_run4), d = u - c16 * run4;
      const int r = (int)div_by((uint32_t)d, (uint32_t)w4, p.inv_w4), x4 = d - r * w4;
      u_row[n] = r;
      u_off[n] = (r * Wp + 1 + 4 * x4) * Cp + 16 * c16;
      u_src[n] = (uint32_t)(c16 * 16) * (uint32_t)HW + (uint32_t)(4 * x4);   // + (y0 - 1 + r) * W
    }
  }
  // (by descriptor: one offset register per unit, the channel in a scalar; rows outside the image read as 0)
  auto load_tile = [&](int tile) {
    const int b = (int)div_by((uint32_t)tile, (uint32_t)p.tiles_per_img, p.inv_tpi);
    const int y0 = (tile - b * p.tiles_per_img) * p.TR;
    const __amdgpu_buffer_rsrc_t rin =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.act) + (int64_t)b * C * HW, 0, C * HW, 0x00020000);
#pragma unroll
    for (int n = 0; n < NU; ++n) {
      const int iy = y0 - 1 + u_row[n];
      const uint32_t at = u_row[n] >= 0 && (unsigned)iy < (unsigned)H ? u_src[n] + (uint32_t)(iy * W) : kOob;
#pragma unroll
      for (int k = 0; k < 16; ++k) raw[n][k] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rin, at, k * HW, 0);
    }
  };
  auto store_tile = [&](int tile) {
    const int b = (int)div_by((uint32_t)tile, (uint32_t)p.tiles_per_img, p.inv_tpi);
    const int y0 = (tile - b * p.tiles_per_img) * p.TR;
#pragma unroll
    for (int n = 0; n < NU; ++n) {
      if (u_row[n] < 0) continue;
      const int iy = y0 - 1 + u_row[n];
      const uint32_t flip = (unsigned)iy < (unsigned)H ? p.act_xor4 : p.pad4;  // (padding was read as 0)
      uint32_t px[4][4];   // [channel quad][pixel]
#pragma unroll
      for (int g = 0; g < 4; ++g) transpose4(raw[n][4 * g], raw[n][4 * g + 1], raw[n][4 * g + 2], raw[n][4 * g + 3], flip, px[g]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<uint4*>(s_in + u_off[n] + i * Cp) = make_uint4(px[0][i], px[1][i], px[2][i], px[3][i]);
    }
    // the halo columns x = -1 and x = W
    const int c4n = C >> 2;
    for (int u = t; u < (p.TR + 2) * 2 * c4n; u += NT) {
      const int c4 = u % c4n, rs = u / c4n;
      const int r = rs >> 1, side = rs & 1;
      *reinterpret_cast<uint32_t*>(s_in + (r * Wp + (side ? W + 1 : 0)) * Cp + 4 * c4) = p.pad4;
    }
  };
  // weight sums per output channel (only the zero-point term needs them): every thread that
  // stages weights adds its four channels' nine taps
  const bool need_sum = p.corr_coef != 0;
  if (t < OB) s_sum[t] = 0;
  __syncthreads();

  // ---- weights of the block: OIHW (per o: [C][9]) -> [o][tap][C]; channels beyond O are zero.
  // A unit is four channels of one output channel: 36 contiguous bytes in memory (nine dwords), unit i at byte 36 i of the block; byte 9 j + k = channel
  // j, tap k; tap k's dword is bytes (k, 9 + k, 18 + k, 27 + k), picked with three byte permutes.
  // A thread's first unit goes out in front of the tile's loads (whose latency the regrouping hides), the constants behind
  // both: nothing is waited for before all of them are under way.  (Two or four units of a thread together, or the next one
  // under way while one is regrouped: the same or 0.2 us slower, 128 -> 128.)  The sums of eight neighbouring lanes, always of
  // one output channel, are added up before they go to LDS.
  constexpr int kUnits = OB * (C / 4);
  constexpr int kEach = (kUnits + NT - 1) / NT;  // of a thread
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t*>(p.wgt) + (int64_t)o0 * C * 9, 0, (O - o0 < OB ? O - o0 : OB) * C * 9, 0x00020000);
  uint32_t dw[9];
  auto load_weights = [&](int u) {
#pragma unroll
    for (int k = 0; k < 9; ++k) dw[k] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rw, 36 * (u * NT + t) + 4 * k, 0, 0);
  };
  load_weights(0);
  if (tile < tile_end) load_tile(tile);

  // ---- per-lane constants: output channels o0 + 32 tn + j
  const int j = lane & 31, h = lane >> 5;
  int32_t corr[TN], mu[TN], sh[TN];
  {
    auto table = [&](const int32_t* q, int n) {
      return __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(q), 0, q ? 4 * n : 0, 0x00020000);
    };
    const int rq_n = kBytes ? (p.per_channel ? O : 1) : 0;
    const __amdgpu_buffer_rsrc_t rb = table(p.bias, O), rm = table(p.mult, rq_n), rs_ = table(p.shift, rq_n);
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      const int o = o0 + 32 * tn + j;
      const uint32_t at = o < O ? 4u * (uint32_t)(p.per_channel ? o : 0) : kOob;
      corr[tn] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rb, o < O ? 4 * o : kOob, 0, 0);
      mu[tn] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rm, at, 0, 0);
      sh[tn] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rs_, at, 0, 0);
    }
  }

#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    if (u > 0) load_weights(u);
    const int i = u * NT + t;
    if (kUnits % NT != 0 && i >= kUnits) break;  // (kUnits is a multiple of 64: whole wavefronts)
    const int o = i / (C / 4), c4 = (i - o * (C / 4)) * 4;
    int32_t part = 0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      // selector bytes: 0-3 pick from the second operand, 4-7 from the first
      constexpr uint32_t kKeep = 0x0c0c0000u;  // upper half zero
      const int i0_ = k, i1 = 9 + k, i2 = 18 + k, i3 = 27 + k;
      const uint32_t lo = __builtin_amdgcn_perm(dw[i1 >> 2], dw[i0_ >> 2], kKeep | (uint32_t)(i0_ & 3) | ((uint32_t)(4 + (i1 & 3)) << 8));
      const uint32_t hi = __builtin_amdgcn_perm(dw[i3 >> 2], dw[i2 >> 2], kKeep | (uint32_t)(i2 & 3) | ((uint32_t)(4 + (i3 & 3)) << 8));
      const uint32_t tap = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
      *reinterpret_cast<uint32_t*>(s_w + o * wstride + k * C + c4) = tap;
      part = __builtin_amdgcn_sdot4((int)tap, 0x01010101, part, false);
    }
    if (need_sum) {
      part += __builtin_amdgcn_update_dpp(0, part, 0xB1, 0xf, 0xf, true);   // quad_perm [1,0,3,2]
      part += __builtin_amdgcn_update_dpp(0, part, 0x4E, 0xf, 0xf, true);   // quad_perm [2,3,0,1]
      part += __builtin_amdgcn_update_dpp(0, part, 0x141, 0xf, 0xf, true);  // row_half_mirror
      if ((lane & 7) == 0) atomicAdd(&s_sum[o], part);
    }
  }
  __syncthreads();
  bool lane_ok = true;   // the folded requantize arithmetic is exact for this lane's channels
#pragma unroll
  for (int tn = 0; tn < TN; ++tn) {
    if (o0 + 32 * tn + j < O) {
      corr[tn] += p.corr_coef * s_sum[32 * tn + j];
      if (kBytes && !p.mult) mu[tn] = 1 << 30, sh[tn] -= 1;
    } else {
      sh[tn] = 1;
    }
    lane_ok = lane_ok && sh[tn] >= 1 && sh[tn] <= 19 && corr[tn] >= -(1 << 30) && corr[tn] <= (1 << 30);
  }
  // FOLD (requantized, 32-bit accumulator, every lane's constants small enough): correction term,
  // rounding term and output zero point go into one 64-bit constant per lane and channel, the
  // result is the high dword of acc * m + k64 shifted by sh - 1 (the shift distance is >= 32),
  // clamped BEFORE that shift against limits scaled by 2^(sh-1), so that the shift can drop each
  // result straight into its byte of the output dword.  |acc| <= 9 C 2^14 < 2^30 and
  // |corr| <= 2^30, so acc + corr cannot wrap; with sh <= 19 and an 8-bit z nothing leaves 63 bits.
  const bool exact = kBytes && !p.rs.half_away && p.rs.z_out >= -256 &&
                    p.rs.z_out <= 255 && __builtin_amdgcn_ballot_w64(!lane_ok) == 0;   // wavefront-uniform
  const bool fold = exact && (OUT == kFull || p.acc_wrap_shift == 0);
  // Clipped to the container's whole range: shift, clip and pack of two results are one instruction and no clip in front of
  // it (9 cycles of a SIMD per output instead of 13.4).
  // With a narrow accumulator the correction term is added in front of its wrapping instead (128 -> 128 on 64 x 28 x 28,
  // 16 bits: the general form's results took 4.6 us of 17.0, these 1.9 of 13.9).
  const bool sat = exact && (OUT == kFull || sat_range(p.rs));
  const int32_t zc = p.rs.z_out + (sat ? sat_bias(p.rs) : 0);
  const uint32_t sflip = sat_flip(p.rs);
  int64_t k64[TN];
  int32_t lo_s[TN], hi_s[TN], s1[TN];
#pragma unroll
  for (int tn = 0; tn < TN; ++tn) {
    s1[tn] = sh[tn] - 1;
    k64[tn] = (fold ? (int64_t)corr[tn] * mu[tn] : 0) + ((int64_t)1 << (30 + (sh[tn] & 31))) + ((int64_t)zc << (31 + (sh[tn] & 31)));
    lo_s[tn] = clip_lo_before_shift(p.rs.lo_rel + p.rs.z_out, s1[tn] & 31);
    hi_s[tn] = clip_hi_before_shift(p.rs.hi_rel + p.rs.z_out, s1[tn] & 31);
  }

  // fragment addresses: the lane's pixels of the tile as MFMA rows
  const int pt = p.TR * W;                             // pixels of a full tile (<= 32 * NW * AF)
  uint32_t a_base[AF];
#pragma unroll
  for (int f = 0; f < AF; ++f) {
    const int q = 32 * (AF * wave + f) + pix_of_row(j);  // the lane's pixel in row block f
    const int qc = q < pt ? q : 0;                       // rows beyond the tile read pixel 0 (results dropped)
    const int qr = (int)div_by((uint32_t)qc, (uint32_t)W, p.inv_w), qx = qc - qr * W;
    a_base[f] = (uint32_t)((qr * Wp + qx) * Cp + 16 * h);
  }
  const uint32_t b_base = (uint32_t)(j * wstride + 16 * h);

  for (; tile < tile_end; tile += tile_step) {
    const int b = (int)div_by((uint32_t)tile, (uint32_t)p.tiles_per_img, p.inv_tpi);
    const int y0 = (tile - b * p.tiles_per_img) * p.TR;          // first output row
    const int rows = (H - y0 < p.TR) ? H - y0 : p.TR;            // output rows of this tile
    __syncthreads();       // the previous tile has been consumed
    store_tile(tile);      // registers -> LDS (waits for this tile's loads)
    __syncthreads();
    if (tile + tile_step < tile_end) load_tile(tile + tile_step);   // the next tile's loads go out now

    // ---- implicit GEMM: 9 taps x C / 32 steps, TN AF MFMAs (32 TN output channels) per step
    v16i acc[AF][TN];
#pragma unroll
    for (int f = 0; f < AF; ++f)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[f][tn][r] = 0;
    // Fully unrolled, the fragments of step s + 1 are requested before the matrix instructions of
    // step s are issued, so the LDS latency hides behind them; all offsets of the weight
    // fragments are immediates, a tap costs one address addition per row block.
    {
      v4i bq[2][TN], aq[2][AF];
      uint32_t a_addr[AF];
      auto fetch = [&](int buf, int tap, int c) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) bq[buf][tn] = *reinterpret_cast<const v4i*>(s_w + b_base + 32 * tn * wstride + tap * C + 32 * c);
#pragma unroll
        for (int f = 0; f < AF; ++f) aq[buf][f] = *reinterpret_cast<const v4i*>(s_in + a_addr[f] + 32 * c);
      };
#pragma unroll
      for (int f = 0; f < AF; ++f) a_addr[f] = a_base[f];
      fetch(0, 0, 0);
#pragma unroll
      for (int step = 0; step < 9 * CK; ++step) {
        const int cur = step & 1;
        if (step + 1 < 9 * CK) {
          const int ntap = (step + 1) / CK, nc = (step + 1) % CK;
          if (nc == 0) {
            const int ky = ntap / 3, kx = ntap - 3 * ky;
            const uint32_t a_tap = (uint32_t)((ky * Wp + kx) * Cp);
#pragma unroll
            for (int f = 0; f < AF; ++f) a_addr[f] = a_base[f] + a_tap;
          }
          fetch(cur ^ 1, ntap, nc);
        }
        __builtin_amdgcn_sched_barrier(0);   // keep the requests ahead of this step's matrix instructions
#pragma unroll
        for (int f = 0; f < AF; ++f)
#pragma unroll
          for (int tn = 0; tn < TN; ++tn) acc[f][tn] = __builtin_amdgcn_mfma_i32_32x32x32_i8(aq[cur][f], bq[cur][tn], acc[f][tn], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }

    // ---- epilogue: the lane's 16 consecutive pixels of channel o0 + 32 tn + j, per row block
    const int npix = rows * W;                           // valid pixels of this tile (a multiple of 4, as W is)
    if (32 * AF * wave >= npix) continue;                // (uniform: a wavefront beyond the tile's pixels)
    const uint32_t obase = (uint32_t)(b * O) * (uint32_t)HW + (uint32_t)(y0 * W);  // (less than 2^31 results)
    if constexpr (kBytes) {
      auto codes = [&](int f, int tn, uint32_t (&dw)[4]) {
        // (opaque: the sums and products that forms have in common are formed in front of all of them otherwise)
        if (OUT != kFull && sat && !fold) {
          const int32_t c = opaque(corr[tn]), m = opaque(mu[tn]);
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            int32_t r[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
              r[e] = (int32_t)(((int64_t)wrap_acc_bits(acc[f][tn][4 * g + e] + c, p.acc_wrap_shift) * (int64_t)m + k64[tn]) >> 32);
            ashr_sat_pair<0>(dw[g], r[0], r[1], s1[tn]);
            ashr_sat_pair<1>(dw[g], r[2], r[3], s1[tn]);
            dw[g] ^= sflip;
          }
        } else if (sat) {
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            int32_t r[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = (int32_t)(((int64_t)acc[f][tn][4 * g + e] * (int64_t)mu[tn] + k64[tn]) >> 32);
            ashr_sat_pair<0>(dw[g], r[0], r[1], s1[tn]);
            ashr_sat_pair<1>(dw[g], r[2], r[3], s1[tn]);
            dw[g] ^= sflip;
          }
        } else if (OUT != kFull && fold) {
          const int32_t m = opaque(mu[tn]);
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            auto one = [&]<int E>() {
              const int64_t pr = (int64_t)acc[f][tn][4 * g + E] * (int64_t)m + k64[tn];
              ashr_into_byte<E>(dw[g], med3((int32_t)(pr >> 32), lo_s[tn], hi_s[tn]), s1[tn]);
            };
            one.template operator()<0>();
            one.template operator()<1>();
            one.template operator()<2>();
            one.template operator()<3>();
          }
        } else {
          const int32_t c = opaque(corr[tn]), m = opaque(mu[tn]);
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            int32_t v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              v[e] = requant_general(OUT == kFull ? acc[f][tn][4 * g + e] + c : wrap_acc_bits(acc[f][tn][4 * g + e] + c, p.acc_wrap_shift), m, sh[tn], p.rs);
            }
            dw[g] = pack4(v[0], v[1], v[2], v[3]);
          }
        }
      };
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) {
        uint32_t dw[AF][4];
#pragma unroll
        for (int f = 0; f < AF; ++f) codes(f, tn, dw[f]);
        if constexpr (AF == 2) swap_sixteens(dw[0], dw[1]);
#pragma unroll
        for (int f = 0; f < AF; ++f) {
          const int at = stay_here(lane);
          const int o = o0 + 32 * tn + (AF == 2 ? 16 * f + (at & 15) : at & 31);
          const int pix = 32 * (AF * wave + (AF == 2 ? (at >> 4) & 1 : 0)) + 16 * (at >> 5), left = npix - pix;
          if (o >= O || left <= 0) continue;
          uint8_t* dst = static_cast<uint8_t*>(p.out) + (obase + (uint32_t)(o * HW + pix));
          if (left >= 16) {
            store16(AF == 2 && p.through, dst, dw[f][0], dw[f][1], dw[f][2], dw[f][3]);
          } else {
#pragma unroll
            for (int g = 0; g < 4; ++g)
              if (4 * g < left) reinterpret_cast<u32_any*>(dst)[g] = dw[f][g];
          }
        }
      }
      continue;
    }
#pragma unroll
    for (int f = 0; f < AF; ++f) {
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) {
        if constexpr (OUT == kWords) {
          // a lane's 64 bytes go out by the quad: its channel t's from all four lanes
          uint32_t v[4][4];
          const int32_t c = opaque(corr[tn]);
          // (the four channels' addresses, kept through the loop over the tiles, were up to 20 registers, and with them went the second
          // workgroup on a CU: 32 -> 64 on 64 x 56 x 56 11.1 us, 10.8 so; 128 -> 256 on 16 x 56 x 56 21.5, 21.0)
          const int at = stay_here(lane), pix = 32 * (AF * wave + f) + 16 * (at >> 5) + 4 * (at & 3), oq0 = o0 + 32 * tn + (at & 28);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            v[r >> 2][r & 3] = (uint32_t)wrap_acc_bits(acc[f][tn][r] + c, p.acc_wrap_shift);
          }
          quad_transpose(v, lane);
#pragma unroll
          for (int t4 = 0; t4 < 4; ++t4) {
            const int oq = oq0 + t4;
            if (oq < O && pix < npix) {
              int32_t* const dst = static_cast<int32_t*>(p.out) + (obase + (uint32_t)(oq * HW + pix));
              const v4i r = {(int)v[t4][0], (int)v[t4][1], (int)v[t4][2], (int)v[t4][3]};
              if (p.through) store_through(dst, r);
              else __builtin_nontemporal_store(r, reinterpret_cast<v4i_any*>(dst));
            }
          }
        } else {
          uint32_t dq[2][4];
          const int32_t c = opaque(corr[tn]);
#pragma unroll
          for (int x = 0; x < 8; ++x) {
            // (the low sixteen bits are the wrapped sum's for any accumulator of at least that width)
            dq[x >> 2][x & 3] = ((uint32_t)(acc[f][tn][2 * x] + c) & 0xffffu) | ((uint32_t)(acc[f][tn][2 * x + 1] + c) << 16);
          }
          swap_sixteens(dq[0], dq[1]);
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            const int at = stay_here(lane), o = o0 + 32 * tn + 16 * g + (at & 15);
            const int pix = 32 * (AF * wave + f) + 16 * (at >> 5) + 8 * ((at >> 4) & 1), left = npix - pix;
            if (o >= O || left <= 0) continue;
            int16_t* dst = static_cast<int16_t*>(p.out) + (obase + (uint32_t)(o * HW + pix));
            if (left >= 8) {
              store16(p.through, dst, dq[g][0], dq[g][1], dq[g][2], dq[g][3]);
            } else {
              reinterpret_cast<u32_any*>(dst)[0] = dq[g][0];
              reinterpret_cast<u32_any*>(dst)[1] = dq[g][1];
            }
          }
        }
      }
    }
  }
}

template <int NW, int AF, int NU, int CK, int TN, int OUT>
hipError_t launch_c3_ck(const C3Params& p, size_t lds, int64_t grid, hipStream_t st) {
  static std::atomic<uint64_t> attr_set{0};
  // the LDS size depends on the geometry, not only on the template arguments: raise the kernel's
  // limit to the CU's 160 KB once, whatever this call needs
  auto kern = conv3x3_nchw_kernel<NW, AF, NU, CK, TN, OUT>;
  hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), 160 * 1024, attr_set);
  if (e != hipSuccess) return e;
  return launch_kernel(kern, dim3((unsigned)grid), dim3(64 * NW), lds, st, p);
}

template <int NW, int AF, int NU, int TN, int OUT>
hipError_t launch_c3(const C3Params& p, size_t lds, int64_t grid, hipStream_t st) {
  switch (p.C / 32) {
    case 1: return launch_c3_ck<NW, AF, NU, 1, TN, OUT>(p, lds, grid, st);
    case 2: return launch_c3_ck<NW, AF, NU, 2, TN, OUT>(p, lds, grid, st);
    case 3: return launch_c3_ck<NW, AF, NU, 3, TN, OUT>(p, lds, grid, st);
    default: return launch_c3_ck<NW, AF, NU, 4, TN, OUT>(p, lds, grid, st);
  }
}

}  // namespace

template <int OUT>
hipError_t launch_conv3x3(const C3Params& p, int nw, int af, int nu, int tn, size_t lds, int64_t grid, hipStream_t st) {
#define HAGO_C3(NWV, AFV, NUV) \
  if (nw == NWV && af == AFV && nu == NUV) return tn == 1 ? launch_c3<NWV, AFV, NUV, 1, OUT>(p, lds, grid, st) : launch_c3<NWV, AFV, NUV, 2, OUT>(p, lds, grid, st);
  HAGO_C3(8, 2, 1) HAGO_C3(8, 2, 2) HAGO_C3(8, 2, 3)
  HAGO_C3(8, 1, 1) HAGO_C3(8, 1, 2) HAGO_C3(8, 1, 3)
  HAGO_C3(4, 1, 1) HAGO_C3(4, 1, 2) HAGO_C3(4, 1, 3)
#undef HAGO_C3
  return hipErrorInvalidValue;
}

}  // namespace hago
