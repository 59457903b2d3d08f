// Depthwise quantized convolution (groups == C == O) with the fused requantize
// epilogue: each output byte needs one input byte from HBM and nine multiply-adds.
//
//   rows3x3  : NCHW, 3x3, stride 1, pad 1, W > 32.  One WAVEFRONT per (image, channel, band of rows, segment of up to 64
//              columns) and no LDS: a lane loads one dword per input row and gets its neighbours' by DPP; see the kernel.
//   mfma     : NCHW, 3x3, pad 1, stride 2, and stride 1 up to W = 32: banded products on the matrix cores.
//   nhwc3x3  : channel-last, stride 1 and 2, pad 1, C >= 4: four channels, four columns and a run of rows per thread.
//   direct   : every other geometry / layout: one output per lane straight
//              from global memory (cache-served), same arithmetic.
#include "dw_split.h"
#include "hago_device.h"
#include "launch.h"

namespace hago {

namespace {

constexpr int kThreads = 256;

// Forms of the requantize arithmetic: see dw_rows3x3_kernel.
enum { kGeneral, kFold, kSat };
// CODES: kernels for codes that are clipped to their container's whole range (of a 32-bit accumulator, rounding half up), of activations
// that need a flip or none, and for everything else; a wavefront waits for the instructions of the forms that its kernel holds
// (us in one kernel and so, of a block with its 1x1 layers: 42 x 28 x 28 x 432 29.1, 28.6; 32 x 56 x 56 x 144 at stride 2 17.4, 17.1).
// The folded form stays beside the saturating one, for channels of shift 0 (in the general form and so: 32 x 56 x 56 x 144 11.6, 9.1; 42 x 28 x 28 x
// 432 14.3, 10.0, channel-last 13.7, 10.4; layers without such channels the same within 1 %).
enum { kOther, kFullPlain, kFullFlipped };

struct DwArgs {
  const uint8_t* act;
  const int8_t* wgt;
  const int32_t* bias;
  void* out;
  ConvGeom g;
  uint32_t act_xor;    // 0x80 for a uint8 container (maps it to int8 = a - 128)
  int32_t act_off;     // 128 for uint8, 0 for int8
  int32_t z_a;
  int32_t acc16;
  int32_t acc_wrap_shift;  // 32 - accumulator bits (0, 16 or 8); the register kernels know 0 and 16 only
  int32_t has_rq;
  int32_t out_mode;    // 0: requantized 8-bit, 1: raw int32, 2: raw int16
  const int32_t* mult;
  const int32_t* shift;
  int32_t per_channel;
  RequantScalars rs;
};

// The work of a launch of gx * mid * outer workgroups, the outermost index first: images, in all three kernels, so
// that each keeps to the XCD that its neighbours in a network of 1x1 layers use for it.  Us of an expansion, a depthwise
// layer and a projection, with the workgroups in launch order (an image's channels on all XCDs) and so, buffers kept
// and three sets of them in turn: 24 -> 144 -> 24 on 8 x 56 x 56 14.2, 12.0 and 14.5, 11.9; on 32 x 56 x 56 29.9, 22.5 and 23.8,
// 23.8 (14 MB between the layers: rewriting lines that other XCDs still hold is what cost the first).
// What a workgroup finds its place by comes as the kernel's leading arguments, which are in scalar registers when it starts: from
// behind the others, where the launch's own dimensions are too, it took 0.1 to 0.2 us of a layer.
struct DwPlace { int32_t x, mid, outer; };
__device__ __forceinline__ uint32_t over(uint32_t n, uint32_t d, uint32_t inv) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)(d == 1 ? n : inv ? __umulhi(n, inv) : n / d));
}
// Of workgroups of equal work, launched as gx x mid x outer.
__device__ __forceinline__ DwPlace xcd_place(uint32_t gx, uint32_t mid, uint32_t count, uint32_t inv_x, uint32_t inv_mid) {
  const uint32_t id = xcd_run(blockIdx.x + gx * (blockIdx.y + mid * blockIdx.z), count);
  const uint32_t rest = over(id, gx, inv_x), outer = over(rest, mid, inv_mid);
  return DwPlace{(int32_t)(id - rest * gx), (int32_t)(rest - outer * mid), (int32_t)outer};
}
// ceil(2^32 / d) for quotients of numbers below n; 0: not exact (or d is 1).
uint32_t inverse(int64_t d, int64_t n) { return d > 1 && n * d < (1ll << 32) ? (uint32_t)(((1ull << 32) + (uint64_t)d - 1) / (uint64_t)d) : 0u; }

__device__ __forceinline__ int32_t wrap_acc(int32_t acc, int wrap_shift) {
  return wrap_shift ? wrap_acc_bits(acc, wrap_shift) : acc;
}

__device__ __forceinline__ void store_one(const DwArgs& p, int64_t idx, int32_t acc, int32_t m,
                                          int32_t sh) {
  if (p.out_mode == 0)
    static_cast<uint8_t*>(p.out)[idx] = (uint8_t)requant_general(acc, m, sh, p.rs);
  else if (p.out_mode == 1)
    static_cast<int32_t*>(p.out)[idx] = acc;
  else
    static_cast<int16_t*>(p.out)[idx] = (int16_t)acc;
}

__global__ __launch_bounds__(kThreads) void dw_direct_kernel(DwArgs p) {
  const ConvGeom& g = p.g;
  const int64_t total = (int64_t)g.B * g.O * g.OH * g.OW;
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < total; i += stride) {
    int32_t b, c, oy, ox;
    int64_t r = i;
    if (g.nhwc) {
      c = (int32_t)(r % g.O); r /= g.O;
      ox = (int32_t)(r % g.OW); r /= g.OW;
      oy = (int32_t)(r % g.OH); b = (int32_t)(r / g.OH);
    } else {
      ox = (int32_t)(r % g.OW); r /= g.OW;
      oy = (int32_t)(r % g.OH); r /= g.OH;
      c = (int32_t)(r % g.O); b = (int32_t)(r / g.O);
    }
    int32_t acc = p.bias ? p.bias[c] : 0;
    for (int ky = 0; ky < g.KH; ++ky) {
      const int iy = oy * g.stride_h + ky - g.pad_h;
      if (iy < 0 || iy >= g.H) continue;
      for (int kx = 0; kx < g.KW; ++kx) {
        const int ix = ox * g.stride_w + kx - g.pad_w;
        if (ix < 0 || ix >= g.W) continue;
        const int64_t ai = g.nhwc ? (((int64_t)b * g.H + iy) * g.W + ix) * g.C + c
                                  : (((int64_t)b * g.C + c) * g.H + iy) * g.W + ix;
        const int64_t wi = g.nhwc ? ((int64_t)c * g.KH + ky) * g.KW + kx
                                  : ((int64_t)c * g.KH + ky) * g.KW + kx;
        const int32_t av = (int32_t)(int8_t)(p.act[ai] ^ p.act_xor) + p.act_off - p.z_a;
        acc += av * (int32_t)p.wgt[wi];
      }
    }
    acc = wrap_acc(acc, p.acc_wrap_shift);
    const int pc = p.per_channel ? c : 0;
    store_one(p, i, acc, p.has_rq ? rq_mult(p.mult, pc) : 0, p.has_rq ? rq_shift(p.mult, p.shift, pc) : 0);
  }
}

// A channel's constants, through scalar loads (the addresses are the same for the whole
// wavefront; scalar loads have their own counter, so waiting for them here, behind the row
// loads, does not wait for a row).  The nine weights: the three aligned dwords that hold bytes
// 9c .. 9c+8.  Each of the three holds at least one of the nine bytes, and an aligned dword
// lies within one page, so the bytes read before and after the channel's weights are never a
// fault.  A pointer the mode does not use is replaced by the weights' address.
struct DwChannel {
  int32_t w[3];       // weight rows, three bytes each
  int32_t wsum, wl, wr;  // sums: all, left column, right column
  int32_t bias, m, sh;
};
template <int MODE>
__device__ __forceinline__ DwChannel dw_channel(const DwArgs& p, int c) {
  const uintptr_t wb = reinterpret_cast<uintptr_t>(p.wgt) + (uint64_t)(uint32_t)c * 9u;
  const int pc = p.per_channel ? c : 0;
  const uint32_t* wp = reinterpret_cast<const uint32_t*>(wb & ~(uintptr_t)3);
  const uint32_t* bp = p.bias ? reinterpret_cast<const uint32_t*>(p.bias + c) : wp;
  const uint32_t* mp = (MODE == 0 && p.mult) ? reinterpret_cast<const uint32_t*>(p.mult + pc) : wp;
  const uint32_t* sp = MODE == 0 ? reinterpret_cast<const uint32_t*>(p.shift + pc) : wp;
  uint64_t d01;
  uint32_t d2, bias_raw, m_raw, sh_raw;
  asm volatile(
      "s_load_dwordx2 %0, %5, 0x0\n\t"
      "s_load_dword %1, %5, 0x8\n\t"
      "s_load_dword %2, %6, 0x0\n\t"
      "s_load_dword %3, %7, 0x0\n\t"
      "s_load_dword %4, %8, 0x0\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&s"(d01), "=&s"(d2), "=&s"(bias_raw), "=&s"(m_raw), "=&s"(sh_raw)
      : "s"(wp), "s"(bp), "s"(mp), "s"(sp));
  const uint32_t d0 = (uint32_t)d01, d1 = (uint32_t)(d01 >> 32);
  const uint32_t o8 = (uint32_t)(wb & 3u) * 8u;
  const uint32_t w03 = (uint32_t)((((uint64_t)d1 << 32) | d0) >> o8);  // weights 0..3
  const uint32_t w47 = (uint32_t)((((uint64_t)d2 << 32) | d1) >> o8);  // weights 4..7
  const uint32_t w8 = (d2 >> o8) & 0xffu;
  DwChannel k;
  k.w[0] = (int32_t)(w03 & 0xffffffu);
  k.w[1] = (int32_t)((w03 >> 24) | ((w47 & 0xffffu) << 8));
  k.w[2] = (int32_t)((w47 >> 16) | (w8 << 16));
  int32_t col[3] = {0, 0, 0};
#pragma unroll
  for (int ky = 0; ky < 3; ++ky)
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) col[kx] += (int32_t)(int8_t)(k.w[ky] >> (8 * kx));
  k.wl = col[0];
  k.wr = col[2];
  k.wsum = col[0] + col[1] + col[2];
  k.bias = p.bias ? (int32_t)bias_raw : 0;
  // (no multiplier array: power-of-two scales, i.e. multiplier one half and the shift one less)
  k.m = MODE == 0 ? (p.mult ? (int32_t)m_raw : (1 << 30)) : 0;
  k.sh = MODE == 0 ? (int32_t)sh_raw - (p.mult ? 0 : 1) : 0;
  return k;
}

// NCHW 3x3 stride 1 pad 1, W >= 4, planes below 2 GB: no LDS.  One wavefront per (plane, band of 4 * rpc rows), rpc <= 16.  Lane (q, rc):
// strip of four output columns q, quarter rc of the band's rows.  A lane loads ONE dword per
// input row (its own strip) and takes the left and right neighbours' dwords by DPP row shifts
// (the 16 lanes of a DPP row are the strips of one image row; lanes without a strip hold the
// zero point, which is also what a shift from outside the row yields).  All rpc + 2 loads are
// in flight together.  Loads and stores go through buffer descriptors of the plane, so a lane
// that has nothing to load or store just uses an out-of-range offset.
// The kernel is bound by vector-ALU instruction issue (about 40 per row of four outputs against
// 5 bytes of traffic), so everything that is the same for the whole wavefront -- the channel's
// weights, bias and multiplier -- comes through scalar loads and scalar arithmetic, and the
// per-output work is three dot products, one 64-bit multiply-add, one shift and one clamp.
// MODE 0: requantized 8-bit, 1: raw int32, 2: raw int16; ACC16: accumulator wraps to 16 bits.
// WIDE: images wider than 64 columns are cut into segments of segw <= 64;
// the lanes at the ends of a segment fetch the neighbouring segment's dword with one more load
// per row, which replaces what the DPP shift cannot deliver.
// RAGGED: rows that are not whole dwords (or tensors at any byte).  Loads and stores are unaligned; the last strip of a
// row is loaded from the row's last four bytes and shifted into place, and stored as those four bytes together with the
// end of its left neighbour's results (16 x 288 planes of 41 x 41: 24.8 us through LDS, 8.6 here).
// OUT (MODE 0): how a row's results go out, a dword per lane: kL2 left in the L2, whose lines the kernel's end writes back; kThrough
//   through it to memory, while other wavefronts work; kFours the same by four rows of a quarter, which are one run of the image: they
//   meet in LDS and its lanes with a strip write 16 bytes each.
enum { kL2, kThrough, kFours };
template <int MODE, bool ACC16, bool WIDE, bool RAGGED, int OUT = kL2, int CODES = kOther>
__global__ __launch_bounds__(kThreads) void dw_rows3x3_kernel(uint32_t gx, uint32_t mid, uint32_t count, uint32_t inv_x, uint32_t inv_mid,
                                                               DwArgs p, int32_t rpc, int32_t nsegs, int32_t segw) {
  // grid: x = groups of four channels, of each its column segments (which are not equally wide: next to each other, every XCD has as
  // many of both; 96 -> 576 -> depthwise -> 96 on one 112 x 112 image, segments of 64 and 48 columns, 25.6 us with a segment's groups of
  // all channels in a row, 22.5 so), y = band, z = image
  const ConvGeom& g = p.g;
  const int H = g.H, W = g.W;
  const int lane = threadIdx.x & 63;
  const DwPlace at = xcd_place(gx, mid, count, inv_x, inv_mid);
  const int cgrp = WIDE ? (int)((uint32_t)at.x / (uint32_t)nsegs) : at.x;
  const int seg = WIDE ? at.x - cgrp * nsegs : 0, band = at.mid;
  const int c = __builtin_amdgcn_readfirstlane(cgrp * 4 + (int)(threadIdx.x >> 6));
  if (c >= g.C) return;  // wavefront-uniform; the kernel has no barrier
  const int64_t plane = (int64_t)at.outer * g.C + c;
  const int cb = WIDE ? seg * segw : 0;  // first column of the segment
  constexpr uint32_t kOob = 0x80000000u;
  constexpr int kEsz = MODE == 0 ? 1 : (MODE == 1 ? 4 : 2);
  constexpr int kPass = 16;  // most output rows per lane

  const int q = lane & 15;
  const int rc = lane >> 4;
  const int y0 = (band * 4 + rc) * rpc;  // first output row of the lane
  const int x0 = cb + (q << 2);          // first column of the strip
  const bool has_strip = x0 < W && (!WIDE || (q << 2) < segw);
  // RAGGED: columns by which the row's last strip is pulled back to end with the row
  const int pull = RAGGED && has_strip && x0 + 4 > W ? x0 + 4 - W : 0;
  const uint32_t lane_off = has_strip ? (uint32_t)(x0 - pull) : kOob;  // byte column of the strip's dword
  const uint32_t pull_bits = (uint32_t)(8 * pull), col_mask = 0xffffffffu >> pull_bits;
  // the dword beyond the segment's end that this lane stands in for (first lane: left, last: right)
  const bool left_edge = WIDE && q == 0 && seg > 0;
  const bool right_edge = WIDE && (q << 2) + 4 == segw && cb + segw < W;
  const int right_x = RAGGED && cb + segw + 4 > W ? W - 4 : cb + segw;  // (only its first column is used)
  const uint32_t edge_off = left_edge ? (uint32_t)(cb - 4) : (right_edge ? (uint32_t)right_x : kOob);
  const uint32_t edge_bits = RAGGED && right_edge ? (uint32_t)(8 * (cb + segw - right_x)) : 0u;
  const uint32_t x4 = p.act_xor * 0x01010101u;
  const uint32_t pad4 = (((uint32_t)p.z_a ^ p.act_xor) & 0xffu) * 0x01010101u;
  const int64_t pbytes = (int64_t)H * W;
  const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(p.act) + (int64_t)plane * pbytes, 0, (int)pbytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(
      static_cast<uint8_t*>(p.out) + (int64_t)plane * pbytes * kEsz, 0, (int)(pbytes * kEsz), 0x00020000);

  // Row i of the lane is image row y0 + i - 1.  A row outside the image, and a lane without a
  // strip, read as the zero point: their offsets are out of the descriptor's range (a negative
  // row wraps to a huge offset, a row >= H lies beyond the plane, a strip-less lane starts at
  // 2^31), such a load returns 0, and the flip mask turns that into the zero point's byte (in
  // range it is the plain sign flip).  The mask is opaque to the compiler: with a select on the
  // loaded value it builds a branch around every load, each followed by a full wait.
  uint32_t flip_lane = has_strip ? x4 : pad4;
  asm volatile("" : "+v"(flip_lane));
  uint32_t d[kPass + 2];  // as loaded; the flip is applied where a row is used, so that no row waits for a later one
  {
    const uint32_t off0 = lane_off + (uint32_t)((y0 - 1) * W);
#pragma unroll
    for (int i = 0; i < kPass + 2; ++i) {
      uint32_t off = off0 + (uint32_t)(i * W);
      if (i >= 3) off = (i - 1 <= rpc) ? off : kOob;  // uniform: rows beyond the lane's halo
      d[i] = __builtin_amdgcn_raw_buffer_load_b32(rin, off, 0, 0);
    }
  }
  uint32_t de[WIDE ? kPass + 2 : 1];  // the edge lanes' extra dwords, same rows
  if constexpr (WIDE) {
    const uint32_t off0 = edge_off + (uint32_t)((y0 - 1) * W);
#pragma unroll
    for (int i = 0; i < kPass + 2; ++i) {
      uint32_t off = off0 + (uint32_t)(i * W);
      if (i >= 3) off = (i - 1 <= rpc) ? off : kOob;
      de[i] = __builtin_amdgcn_raw_buffer_load_b32(rin, off, 0, 0);
    }
  }
  const int rows_in = H + 1 - y0;  // rows 1 .. rows_in - 1 of the lane lie in the image
  struct Row { uint32_t d, edge; };  // a lane's dword of a row and, for an edge lane (which has a strip: same flip), its edge dword
  auto row = [&](int i) {
    uint32_t flip = (i == 0 ? y0 > 0 : i < rows_in) ? flip_lane : pad4;
    asm volatile("" : "+v"(flip));
    if constexpr (RAGGED)
      return Row{(((d[i] >> pull_bits) ^ flip) & col_mask) | (pad4 & ~col_mask), WIDE ? (de[i] >> edge_bits) ^ flip : 0u};
    return Row{d[i] ^ flip, WIDE ? de[i] ^ flip : 0u};
  };

  const DwChannel k = dw_channel<MODE>(p, c);
  const int32_t* wrow = k.w;
  const int32_t m = k.m, sh = k.sh;
  // sum (a - z) w = sum (a' + off - z) w = sum a' w + (off - z) * sum w, a' = flipped byte
  const int32_t corr = k.bias + (p.act_off - p.z_a) * k.wsum;
  const int64_t rnd = (int64_t)1 << (30 + sh);
  const int32_t z = p.rs.z_out;
  const int32_t away = p.rs.half_away ? -1 : 0;  // mask of the sign-bit correction

  // the four 3-byte windows of a strip: output x = 4q + i reads input columns x-1 .. x+1
  // The shifted copies live in two registers of their own, which start as the zero point in
  // every lane: a shift never writes the lane at the end of a DPP row it has no source for, so
  // that lane keeps the zero point from one shift to the next and needs no fresh copy.
  uint32_t left = pad4, right = pad4;
  auto windows = [&](Row r, uint32_t (&w)[4]) {
    const uint32_t d1 = r.d;
    left = (uint32_t)__builtin_amdgcn_update_dpp((int)left, (int)d1, 0x111, 0xf, 0xf, false);    // row_shr:1
    right = (uint32_t)__builtin_amdgcn_update_dpp((int)right, (int)d1, 0x101, 0xf, 0xf, false);  // row_shl:1
    if constexpr (WIDE) {
      left = left_edge ? r.edge : left;
      right = right_edge ? r.edge : right;
    }
    w[0] = __builtin_amdgcn_alignbyte(d1, left, 3);
    w[1] = d1;
    w[2] = __builtin_amdgcn_alignbyte(right, d1, 1);
    w[3] = __builtin_amdgcn_alignbyte(right, d1, 2);
  };
  // (the builtin, not inline assembly: the compiler has to see the dot instructions to keep the
  // wait states they need before a dependent instruction)
  auto dot4 = [](uint32_t a, int32_t b, int32_t c) {
    return __builtin_amdgcn_sdot4((int)a, b, c, false);
  };
  // A store beyond the image lies beyond the plane, and a strip-less lane's offset starts at
  // 2^31: both are out of the descriptor's range and dropped.
  const uint32_t so0 = has_strip ? (uint32_t)(x0 - (MODE == 0 ? pull : 0) + y0 * W) * kEsz : kOob;
  static_assert(OUT == kL2 || MODE == 0);
  static_assert(OUT != kFours || (!WIDE && !RAGGED));
  constexpr int kOutAux = OUT == kL2 ? 0 : 16;  // sc1
  __shared__ __attribute__((aligned(16))) uint8_t s_fours[OUT == kFours ? kThreads / 16 : 1][256];
  uint8_t* const fours = s_fours[OUT == kFours ? threadIdx.x >> 4 : 0];

  // FOLD (requantized, 32-bit accumulator, and the channel's constants small enough): the
  // correction term, the rounding term and the output zero point all go into one 64-bit
  // constant k64, so that an output is clamp((dots * m + k64) >> (31 + sh)) against the
  // absolute bounds: (acc * m + rnd) >> s + z == (acc * m + rnd + z * 2^s) >> s exactly, and
  // acc = dots + corr cannot wrap when |corr| <= 2^30 (|dots| < 2^19).  With sh <= 19 and an
  // 8-bit z nothing here leaves 63 bits.
  // SAT (the same, sh >= 1 and a clip to the container's whole range): shift, clip and pack of two results are one
  // instruction (config 4's layer, 144 channels of 32 x 56 x 56: 8.7 us, 9.1 before).
  // PLAIN: int8 activations with zero point 0 need no flip at all (the mask is zero everywhere)
  auto rows = [&]<int FORM, bool PLAIN>() {
    constexpr bool FOLD = FORM != kGeneral;
    auto rowp = [&](int i) {
      if constexpr (PLAIN && RAGGED) return Row{d[i] >> pull_bits, WIDE ? de[i] >> edge_bits : 0u};
      else if constexpr (PLAIN) return Row{d[i], WIDE ? de[i] : 0u};
      else return row(i);
    };
    int32_t lo = p.rs.lo_rel + (FOLD ? z : 0), hi = p.rs.hi_rel + (FOLD ? z : 0);
    // vector-register copies: v_med3 takes at most one scalar operand
    asm volatile("" : "+v"(lo), "+v"(hi));
    const int32_t zc = z + (FORM == kSat ? sat_bias(p.rs) : 0), s1 = sh - 1;
    const uint32_t flip = sat_flip(p.rs);
    const int64_t k64 = FOLD ? (int64_t)corr * m + rnd + ((int64_t)zc << (31 + sh)) : rnd;
    const int32_t init = FOLD ? 0 : corr;
    uint32_t w[3][4];  // windows of three consecutive rows, slot = row % 3
    windows(rowp(0), w[0]);
    windows(rowp(1), w[1]);
#pragma unroll
    for (int i = 0; i < kPass; ++i) {
      if (i < rpc) {  // uniform
        windows(rowp(i + 2), w[(i + 2) % 3]);
        int32_t acc[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          int32_t a = dot4(w[i % 3][e], wrow[0], init);
          a = dot4(w[(i + 1) % 3][e], wrow[1], a);
          a = dot4(w[(i + 2) % 3][e], wrow[2], a);
          acc[e] = ACC16 ? (int32_t)(int16_t)a : a;
        }
        const uint32_t so = so0 + (uint32_t)(i * W * kEsz);
        if constexpr (MODE == 0) {
          int32_t r[4];
          uint32_t dw;
          if constexpr (FORM == kSat) {
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = (int32_t)(((int64_t)acc[e] * (int64_t)m + k64) >> 32);
            ashr_sat_pair<0>(dw, r[0], r[1], s1);
            ashr_sat_pair<1>(dw, r[2], r[3], s1);
            dw ^= flip;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              // (general form only: halves away from zero add the accumulator's sign bit)
              const int64_t pr = (int64_t)acc[e] * (int64_t)m + k64 + (FOLD ? 0 : (int64_t)((acc[e] >> 31) & away));
              r[e] = med3((int32_t)(pr >> (31 + sh)), lo, hi) + (FOLD ? 0 : z);
            }
            dw = pack4_perm(r[0], r[1], r[2], r[3]);
          }
          if constexpr (RAGGED) {
            const uint32_t lw = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)dw, 0x111, 0xf, 0xf, true);  // row_shr:1
            dw = (uint32_t)((((uint64_t)dw << 32) | lw) >> (32 - pull_bits));
          }
          if (OUT == kFours && (i | 3) < rpc) {  // (uniform)
            if (has_strip) *reinterpret_cast<uint32_t*>(fours + 4 * q + (i & 3) * W) = dw;
            if ((i & 3) == 3) {
              typedef uint32_t v4u __attribute__((ext_vector_type(4)));
              __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
              const int left = has_strip ? (H - y0 - (i - 3)) * W - 16 * q : 0;  // bytes of the image from the lane's piece on
              if (left > 0) {
                const v4u v = *reinterpret_cast<const v4u*>(fours + 16 * q);
                uint8_t* const dst = static_cast<uint8_t*>(p.out) + plane * pbytes + (uint32_t)((y0 + i - 3) * W + 16 * q);
                if (left >= 16) {
                  store_through(dst, v);
                } else {  // (the image ends with this piece)
#pragma unroll
                  for (int e = 0; e < 3; ++e)
                    if (4 * e < left) reinterpret_cast<uint32_t*>(dst)[e] = v[e];
                }
              }
              __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
          } else {
            __builtin_amdgcn_raw_buffer_store_b32(dw, rout, so, 0, kOutAux);
          }
        } else if constexpr (MODE == 1) {
          typedef int32_t v4i32 __attribute__((ext_vector_type(4)));
          if constexpr (RAGGED) {
            __builtin_amdgcn_raw_buffer_store_b128(v4i32{acc[0], acc[1], acc[2], acc[3]}, rout, pull ? kOob : so, 0, 0);
#pragma unroll
            for (int e = 0; e < 3; ++e) __builtin_amdgcn_raw_buffer_store_b32((uint32_t)acc[e], rout, pull && e < 4 - pull ? so + 4 * e : kOob, 0, 0);
          } else {
            __builtin_amdgcn_raw_buffer_store_b128(v4i32{acc[0], acc[1], acc[2], acc[3]}, rout, so, 0, 0);
          }
        } else {
          typedef uint32_t v2u32 __attribute__((ext_vector_type(2)));
          const v2u32 v = {(uint32_t)(acc[0] & 0xffff) | ((uint32_t)acc[1] << 16), (uint32_t)(acc[2] & 0xffff) | ((uint32_t)acc[3] << 16)};
          if constexpr (RAGGED) {
            __builtin_amdgcn_raw_buffer_store_b64(v, rout, pull ? kOob : so, 0, 0);
#pragma unroll
            for (int e = 0; e < 3; ++e) __builtin_amdgcn_raw_buffer_store_b16((short)acc[e], rout, pull && e < 4 - pull ? so + 2 * e : kOob, 0, 0);
          } else {
            __builtin_amdgcn_raw_buffer_store_b64(v, rout, so, 0, 0);
          }
        }
      }
    }
  };
  const bool fold = MODE == 0 && !ACC16 && sh >= 0 && sh <= 19 && corr >= -(1 << 30) && corr <= (1 << 30) &&
                    z >= -256 && z <= 255 && !p.rs.half_away;
  const bool sat = fold && sh >= 1 && sat_range(p.rs), no_flip = x4 == 0 && pad4 == 0;
  if constexpr (CODES != kOther) {
    if (sat) rows.template operator()<kSat, CODES == kFullPlain>();
    else if (fold) rows.template operator()<kFold, CODES == kFullPlain>();
    else rows.template operator()<kGeneral, false>();
  } else {
    if (fold && no_flip) rows.template operator()<kFold, true>();
    else if (fold) rows.template operator()<kFold, false>();
    else rows.template operator()<kGeneral, false>();
  }
}

// NCHW 3x3 pad 1, stride S = 1 or 2, W >= 4 (OW >= 4), on the matrix cores.
//
// Along a row the convolution is a product with a banded matrix: out(x, y) = sum_ky sum_k A_ky(x, k) in(k, S y + ky - 1),
// where A_ky holds w[ky][k - S x + 1] and k runs over the 32 bytes of a row from column xs on.  So one 32x32x32 int8
// instruction per kernel row makes all nine taps of 32 columns x 32 rows; the vector ALUs, which bounded the dot-product
// form at about 40 instructions per 4 outputs and lane, only requantize (3.75 per output).
//   rows of the product: output columns.  Which accumulator register stands for which column is free (A is built here),
//     so every lane gets runs of consecutive columns and stores them whole; where a tile has fewer columns than its
//     lanes hold, the runs overlap and bytes are written twice with the same value: no store is ever partial.
//   columns of the product: output rows, counted through all images of the channel (a flat index), so that a tile is full
//     however few rows an image has; a lane works out its own image and row.
//   operand bytes: the 16 bytes of a lane come straight from memory at whatever byte they start; the three kernel rows
//     are three loads (the second and third hit the vector cache).  Columns outside the image have no byte in the window:
//     their share, the zero point times their weights, is the initial value of the accumulators.  Rows outside read 0
//     through the descriptor's range check and become the zero point under the flip mask.
//   CPK = 2 (W <= 16): two channels share a tile, each with 16 of the 32 bytes and half of the columns.
// A wavefront keeps its channel, A (12 registers) and column tile for several row tiles.
struct DwTile {
  int32_t C, H, W, OH, OW, B;
  int32_t groups, nt, cw;     // channel groups, column tiles, columns of a tile
  uint32_t inv_nt, inv_oh;    // ceil(2^32 / nt); ceil(2^32 / OH), 0: tiles do not run through images
  int32_t period;             // rows of the tile index per image: OH, or whole tiles if those do not run through images
  int32_t per_wave, longer;   // row tiles of a wavefront (dw_split.h)
};

// NJ: groups of four columns per lane (2 or 4).
template <int MODE, int S, int CPK, int NJ, int CODES>
__global__ __launch_bounds__(kThreads, 4) void dw_mfma_kernel(uint32_t gx, uint32_t ids, uint32_t inv_x, DwArgs p, DwTile q) {
  typedef int32_t v2i __attribute__((ext_vector_type(2)));
  typedef int32_t v4i __attribute__((ext_vector_type(4)));
  typedef int32_t v16i __attribute__((ext_vector_type(16)));
  constexpr uint32_t kOob = 0x80000000u;
  constexpr int kEsz = MODE == 0 ? 1 : (MODE == 1 ? 4 : 2);
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const int C = q.C, H = q.H, W = q.W, OH = q.OH, OW = q.OW;
  // runs of row tiles, in each the groups of channels and column tiles; by XCD, or, ids = 0, in launch order
  const uint32_t launched = blockIdx.x + gx * blockIdx.y;
  const uint32_t id = ids ? xcd_run(launched, ids) : launched;
  const uint32_t tile_run = over(id, gx, inv_x);
  const int wi = (int)(id - tile_run * gx) * 4 + (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = q.nt > 1 ? (int)__umulhi((uint32_t)wi, q.inv_nt) : wi;
  if (grp >= q.groups) return;  // wavefront-uniform; the kernel has no barrier
  const int ct = wi - grp * q.nt;
  const int c0 = grp * CPK;
  const int c = CPK == 1 ? c0 : c0 + h;  // the lane's channel: of its operand bytes and of its results
  const int x0 = CPK == 1 ? (ct * q.cw < OW - q.cw ? ct * q.cw : OW - q.cw) : 0;  // first output column of the tile
  // first column of the window: one left of the first output's, inside the row as far as the row is wide enough
  int xs = x0 * S - 1;
  xs = xs > W - 32 ? W - 32 : xs;
  xs = xs < 0 || CPK == 2 ? 0 : xs;
  // output column of the lane's result 4 j + r: col(h, j) + r
  auto col = [&](int hh, int j) {
    if constexpr (CPK == 1) return x0 + (hh ? q.cw - 4 * NJ : 0) + 4 * j;
    else return j >= NJ / 2 ? OW - 2 * NJ + 4 * (j - NJ / 2) : 4 * j;
  };

  // one tile's operand bytes, one load per kernel row, and where its results go
  const int64_t img_in = (int64_t)C * H * W, img_out = (int64_t)C * OH * OW * kEsz;
  const int64_t in_bytes = (int64_t)q.B * img_in, out_bytes = (int64_t)q.B * img_out;
  const uint32_t x4 = p.act_xor * 0x01010101u;
  const uint32_t pad4 = (((uint32_t)p.z_a ^ p.act_xor) & 0xffu) * 0x01010101u;
  const bool plain = (x4 | pad4) == 0;
  struct Tile {
    v4i b[3];
    uint32_t ok;     // bit i: the lane's input row i exists
    uint32_t so;     // byte offset of the lane's output row
    int32_t img;
  };
  const int tile0 = (int)tile_run * q.per_wave + ((int)tile_run < q.longer ? (int)tile_run : q.longer);
  const int count = q.per_wave + ((int)tile_run < q.longer ? 1 : 0);
  int img = tile0 * 32 / q.period, y0 = tile0 * 32 - img * q.period;  // first image and row of the next tile to load
  auto load = [&](Tile& t) {
    const int64_t ibase = (int64_t)img * img_in + (int64_t)c0 * H * W;
    const int64_t left = in_bytes - ibase;
    const uint32_t end = left > 0x7fffffff ? 0x7fffffffu : (uint32_t)left;
    const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.act) + ibase, 0, (int)end, 0x00020000);
    const int yy = y0 + n;
    const int k = (int)__umulhi((uint32_t)yy, q.inv_oh);  // images beyond the tile's first
    const int y = yy - k * OH;
    const bool valid = y < OH && img + k < q.B && (CPK == 1 || c < C);
    const uint32_t base = (uint32_t)k * (uint32_t)img_in + (uint32_t)((y * S - 1) * W + xs) + (h ? (CPK == 2 ? (uint32_t)(H * W) : 16u) : 0u);
    t.so = valid ? (uint32_t)k * (uint32_t)img_out + (uint32_t)(y * OW) * kEsz + (CPK == 2 && h ? (uint32_t)(OH * OW) * kEsz : 0u) : kOob;
    t.img = img;
    t.ok = 0;
    uint32_t off[3];
    bool past = false;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const bool ok = valid && (uint32_t)(y * S - 1 + i) < (uint32_t)H;
      off[i] = ok ? base + (uint32_t)(i * W) : kOob;
      t.ok |= ok ? 1u << i : 0u;
      past |= ok && off[i] + 16u > end;
    }
    // (a window that is wider than the row can reach past the last row of the tensor)
    if ((CPK == 2 || W < 32) && __builtin_amdgcn_ballot_w64(past) != 0) {
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          // a dword across the end reads as 0 as a whole: its bytes one by one
          const uint32_t o = off[i] + 4u * d;
          const uint32_t rem = off[i] == kOob ? 4u : end - o;
          uint32_t v = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rin, rem < 4u ? kOob : o, 0, 0);
          if (__builtin_amdgcn_ballot_w64(rem < 4u) != 0) {
#pragma unroll
            for (int e = 0; e < 3; ++e)
              v |= (uint32_t)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(rin, rem < 4u ? o + e : kOob, 0, 0) << (8 * e);
          }
          t.b[i][d] = (int32_t)v;
        }
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i) t.b[i] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rin, off[i], 0, 0));
    }
    y0 += 32;
    while (y0 >= q.period) { y0 -= q.period; ++img; }
  };
  Tile t0;
  load(t0);

  // the channels' constants
  const DwChannel ka = dw_channel<MODE>(p, c0);
  DwChannel kb = ka;
  if constexpr (CPK == 2) kb = dw_channel<MODE>(p, c0 + 1 < C ? c0 + 1 : c0);
  auto pick = [&](int32_t a, int32_t b) { return CPK == 1 ? a : (h ? b : a); };

  // A: lane (m = n, h) holds the window bytes 16 h .. 16 h + 15 (CPK 2: the 16 bytes of channel h) of column m's band
  v4i A[3];
  {
    const int j = n >> 3, hm = (n >> 2) & 1;
    const int xc = (col(hm, j) + (n & 3)) * S;  // input column of the middle tap
    const bool used = j < NJ && (CPK == 1 || hm == h);
    const int at = xc - 1 - xs - (CPK == 1 ? 16 * h : 0);  // the lane's byte of the first tap
    uint32_t wk[3];
#pragma unroll
    for (int ky = 0; ky < 3; ++ky) {
      const uint32_t w = (uint32_t)pick(ka.w[ky], kb.w[ky]);
      wk[ky] = used ? (xc + 1 < W ? w : w & 0xffffu) : 0u;  // (no third tap right of the image)
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // the low dword of (w << 24) >> 8 s is w moved to byte at - 4 i, and 0 from s = 6 on
      uint32_t s = (uint32_t)(3 - (at - 4 * i));
      s = s < 7u ? s : 7u;
#pragma unroll
      for (int ky = 0; ky < 3; ++ky) A[ky][i] = (int32_t)(uint32_t)(((uint64_t)wk[ky] << 24) >> (8u * s));
    }
  }

  // sum (a - z) w = sum (a' + off - z) w = sum a' w + (off - z) * sum w, a' = flipped byte
  const int32_t corr_a = ka.bias + (p.act_off - p.z_a) * ka.wsum, corr_b = kb.bias + (p.act_off - p.z_a) * kb.wsum;
  const int32_t z = p.rs.z_out;
  const int32_t away = p.rs.half_away ? -1 : 0;  // mask of the sign-bit correction
  const int32_t corr = pick(corr_a, corr_b), m = pick(ka.m, kb.m), sh = pick(ka.sh, kb.sh);
  const int64_t rnd = (int64_t)1 << (30 + sh);

  // FORM and PLAIN as in the register kernel
  auto run = [&]<int FORM, bool PLAIN>() {
    constexpr bool FOLD = FORM != kGeneral;
    int32_t lo = p.rs.lo_rel + (FOLD ? z : 0), hi = p.rs.hi_rel + (FOLD ? z : 0);
    asm volatile("" : "+v"(lo), "+v"(hi));
    const int32_t zc = z + (FORM == kSat ? sat_bias(p.rs) : 0), s1 = sh - 1;
    const uint32_t sflip = sat_flip(p.rs);
    const int64_t k64 = FOLD ? (int64_t)corr * m + rnd + ((int64_t)zc << (31 + sh)) : rnd;
    v16i init;
#pragma unroll
    for (int i = 0; i < 16; ++i) init[i] = FOLD ? 0 : corr;
    if constexpr (!PLAIN) {
      const int32_t pad = (int32_t)(int8_t)pad4;
      const int32_t pl = pad * pick(ka.wl, kb.wl), pr = pad * pick(ka.wr, kb.wr);
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int xo = col(h, j) + r;
          init[4 * j + r] += (xo == 0 ? pl : 0) + (xo * S + 1 >= W ? pr : 0);
        }
    }
    auto compute = [&](Tile& t) {
      const int64_t obase = (int64_t)t.img * img_out + (int64_t)c0 * OH * OW * kEsz;
      const int64_t oleft = out_bytes - obase;
      const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(
          static_cast<uint8_t*>(p.out) + obase, 0, oleft > 0x7fffffff ? 0x7fffffff : (int)oleft, 0x00020000);
      if constexpr (!PLAIN) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          const uint32_t flip = (t.ok >> i) & 1u ? x4 : pad4;
#pragma unroll
          for (int d = 0; d < 4; ++d) t.b[i][d] ^= (int32_t)flip;
        }
      }
      v16i acc = init;
#pragma unroll
      for (int ky = 0; ky < 3; ++ky) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[ky], t.b[ky], acc, 0, 0, 0);
      auto so = [&](int j) { return t.so + (uint32_t)col(h, j) * kEsz; };
      if constexpr (MODE == 0) {
        uint32_t dw[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          int32_t r[4];
          if constexpr (FORM == kSat) {
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = (int32_t)(((int64_t)acc[4 * j + e] * (int64_t)m + k64) >> 32);
            ashr_sat_pair<0>(dw[j], r[0], r[1], s1);
            ashr_sat_pair<1>(dw[j], r[2], r[3], s1);
            dw[j] ^= sflip;
            continue;
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            int32_t a = acc[4 * j + e];
            if constexpr (!FOLD) a = wrap_acc_bits(a, p.acc_wrap_shift);
            const int64_t pr = (int64_t)a * (int64_t)m + k64 + (FOLD ? 0 : (int64_t)((a >> 31) & away));
            r[e] = med3((int32_t)(pr >> (31 + sh)), lo, hi) + (FOLD ? 0 : z);
          }
          dw[j] = pack4_perm(r[0], r[1], r[2], r[3]);
        }
        if constexpr (CPK == 1 && NJ == 4) {
          __builtin_amdgcn_raw_buffer_store_b128(v4i{(int32_t)dw[0], (int32_t)dw[1], (int32_t)dw[2], (int32_t)dw[3]}, rout, so(0), 0, 0);
        } else if constexpr (NJ == 2 && CPK == 2) {
          if (OW < 4) {  // uniform
            for (int e = 0; e < OW; ++e) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(dw[0] >> (8 * e)), rout, so(0) + e, 0, 0);
            return;
          }
          __builtin_amdgcn_raw_buffer_store_b32(dw[0], rout, so(0), 0, 0);
          __builtin_amdgcn_raw_buffer_store_b32(dw[1], rout, so(1), 0, 0);
        } else {
          __builtin_amdgcn_raw_buffer_store_b64(v2i{(int32_t)dw[0], (int32_t)dw[1]}, rout, so(0), 0, 0);
          if constexpr (NJ == 4) __builtin_amdgcn_raw_buffer_store_b64(v2i{(int32_t)dw[2], (int32_t)dw[3]}, rout, so(2), 0, 0);
        }
      } else {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          int32_t a[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) a[e] = wrap_acc_bits(acc[4 * j + e], p.acc_wrap_shift);
          if (NJ == 2 && CPK == 2 && OW < 4) {  // uniform
#pragma unroll
            for (int e = 0; e < 3; ++e) {
              const uint32_t o = j == 0 && e < OW ? so(0) + e * kEsz : kOob;
              if constexpr (MODE == 1) __builtin_amdgcn_raw_buffer_store_b32((uint32_t)a[e], rout, o, 0, 0);
              else __builtin_amdgcn_raw_buffer_store_b16((short)a[e], rout, o, 0, 0);
            }
            continue;
          }
          if constexpr (MODE == 1)
            __builtin_amdgcn_raw_buffer_store_b128(v4i{a[0], a[1], a[2], a[3]}, rout, so(j), 0, 0);
          else
            __builtin_amdgcn_raw_buffer_store_b64(v2i{(a[0] & 0xffff) | (int32_t)((uint32_t)a[1] << 16),
                                                      (a[2] & 0xffff) | (int32_t)((uint32_t)a[3] << 16)}, rout, so(j), 0, 0);
        }
      }
    };
    Tile t1;
    for (int i = 1; i < count; i += 2) {
      load(t1);
      compute(t0);
      if (i + 1 < count) load(t0);
      compute(t1);
    }
    if (count & 1) compute(t0);
  };
  const bool fold = MODE == 0 && p.acc_wrap_shift == 0 && ka.sh >= 0 && ka.sh <= 19 && kb.sh >= 0 && kb.sh <= 19 &&
                    corr_a >= -(1 << 30) && corr_a <= (1 << 30) && corr_b >= -(1 << 30) && corr_b <= (1 << 30) &&
                    z >= -256 && z <= 255 && !p.rs.half_away;
  const bool sat = fold && ka.sh >= 1 && kb.sh >= 1 && sat_range(p.rs);
  if constexpr (CODES != kOther) {
    if (sat) run.template operator()<kSat, CODES == kFullPlain>();
    else if (fold) run.template operator()<kFold, CODES == kFullPlain>();
    else run.template operator()<kGeneral, false>();
  } else {
    if (fold && plain) run.template operator()<kFold, true>();
    else if (fold) run.template operator()<kFold, false>();
    else run.template operator()<kGeneral, false>();
  }
}

// Channel-last 3x3, pad 1, stride S = 1 or 2, C >= 4, any alignment.  A thread owns four consecutive channels (one dword
// per pixel) of a strip of four output columns and slides down a run of output rows; consecutive threads own consecutive
// channel quads, so a wavefront's loads and stores are contiguous.  The dwords of an input row's 6 (9) columns are
// transposed into rows of one channel (12 (20) byte permutes), from where on it is the dot-product form of the NCHW kernel:
// per channel four windows, three dot products and one requantize per output, 8 instructions per output in all.  (Its
// predecessor multiplied byte by byte, 16 per output, and unpacked the weights of a thread for 8 outputs: 32 x 56 x 56 x 144
// took 30.7 us; stride 2 had no kernel of its own and took 43.)  The last quad of channels and the last strip are moved
// back to end with the pixel or row: bytes written twice get the same value.
template <int MODE, int S, int CODES>
__global__ __launch_bounds__(kThreads) void dw_nhwc3x3_kernel(uint32_t gx, uint32_t mid, uint32_t count, uint32_t inv_x, uint32_t inv_mid,
                                                               DwArgs p, int32_t c4, uint32_t inv_c4, int32_t strips, int32_t run) {
  typedef int32_t v2i __attribute__((ext_vector_type(2)));
  typedef int32_t v4i __attribute__((ext_vector_type(4)));
  typedef uint32_t u32_u __attribute__((aligned(1)));
  constexpr int NC = S == 1 ? 6 : 9;  // input columns of a strip
  constexpr uint32_t kOob = 0x80000000u;
  constexpr int kEsz = MODE == 0 ? 1 : (MODE == 1 ? 4 : 2);
  const ConvGeom& g = p.g;
  const int H = g.H, W = g.W, C = g.C, OH = g.OH, OW = g.OW;
  // grid: x = (strip, channel quad), y = run of rows, z = image
  const DwPlace at = xcd_place(gx, mid, count, inv_x, inv_mid);
  const uint32_t t = (uint32_t)at.x * kThreads + threadIdx.x;
  const int strip = c4 > 1 ? (int)__umulhi(t, inv_c4) : (int)t;
  if (strip >= strips) return;
  const int cq = (int)t - strip * c4;
  const int c = 4 * cq < C - 4 ? 4 * cq : C - 4;
  const int xl = OW - 4 < 0 ? 0 : OW - 4;
  const int x0 = 4 * strip < xl ? 4 * strip : xl;
  const int y0 = at.mid * run;
  const int rows = OH - y0 < run ? OH - y0 : run;
  const uint32_t x4 = p.act_xor * 0x01010101u;
  const uint32_t pad4 = (((uint32_t)p.z_a ^ p.act_xor) & 0xffu) * 0x01010101u;
  const bool plain = (x4 | pad4) == 0;

  // Columns outside the image have an offset out of the descriptor's range, read as 0 and become the zero point under
  // the flip mask; a row outside has a descriptor without bytes.
  uint32_t off[NC], flip[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int x = x0 * S - 1 + i;
    const bool ok = (uint32_t)x < (uint32_t)W;
    off[i] = ok ? (uint32_t)(x * C + c) : kOob;
    flip[i] = ok ? x4 : pad4;
  }
  uint32_t d[NC];
  auto load = [&](int iy) {
    const bool ok = (uint32_t)iy < (uint32_t)H;  // uniform
    const int64_t base = ((int64_t)at.outer * H + (ok ? iy : 0)) * W * C;
    const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.act) + base, 0, ok ? W * C : 0, 0x00020000);
#pragma unroll
    for (int i = 0; i < NC; ++i) d[i] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rin, off[i], 0, 0);
  };
  load(y0 * S - 1);

  // the channels' constants: nine weight bytes each, in three unaligned loads that stay inside the tensor
  int32_t wt[4][3], m[4], sh[4], corr[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint8_t* wp = reinterpret_cast<const uint8_t*>(p.wgt) + (int64_t)(c + j) * 9;
    wt[j][0] = (int32_t)(*reinterpret_cast<const u32_u*>(wp) & 0xffffffu);
    wt[j][1] = (int32_t)(*reinterpret_cast<const u32_u*>(wp + 2) >> 8);
    wt[j][2] = (int32_t)(*reinterpret_cast<const u32_u*>(wp + 5) >> 8);
    const int pc = p.per_channel ? c + j : 0;
    m[j] = MODE == 0 ? rq_mult(p.mult, pc) : 0;
    sh[j] = MODE == 0 ? rq_shift(p.mult, p.shift, pc) : 0;
    corr[j] = p.bias ? p.bias[c + j] : 0;
  }
  auto dot4 = [](uint32_t a, int32_t b, int32_t acc) { return __builtin_amdgcn_sdot4((int)a, b, acc, false); };
  const int32_t z = p.rs.z_out;
  const int32_t away = p.rs.half_away ? -1 : 0;
  bool fold = MODE == 0 && p.acc_wrap_shift == 0 && z >= -256 && z <= 255 && !p.rs.half_away;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int32_t wsum = dot4(0x01010101u, wt[j][0], dot4(0x01010101u, wt[j][1], dot4(0x01010101u, wt[j][2], 0)));
    corr[j] += (p.act_off - p.z_a) * wsum;
    fold = fold && sh[j] >= 0 && sh[j] <= 19 && corr[j] >= -(1 << 30) && corr[j] <= (1 << 30);
  }
  fold = __builtin_amdgcn_ballot_w64(!fold) == 0;
  const bool sat = fold && sat_range(p.rs) && __builtin_amdgcn_ballot_w64(sh[0] < 1 || sh[1] < 1 || sh[2] < 1 || sh[3] < 1) == 0;

  // FORM and PLAIN as in the register kernel
  auto body = [&]<int FORM, bool PLAIN>() {
    constexpr bool FOLD = FORM != kGeneral;
    int32_t lo = p.rs.lo_rel + (FOLD ? z : 0), hi = p.rs.hi_rel + (FOLD ? z : 0);
    asm volatile("" : "+v"(lo), "+v"(hi));
    const uint32_t sflip = sat_flip(p.rs);
    int64_t k64[4];
    int32_t s1[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      s1[j] = sh[j] - 1;
      const int64_t rnd = (int64_t)1 << (30 + sh[j]);
      k64[j] = FOLD ? (int64_t)corr[j] * m[j] + rnd + ((int64_t)(z + (FORM == kSat ? sat_bias(p.rs) : 0)) << (31 + sh[j])) : rnd;
    }
    uint32_t w[3][4][4];  // [row % 3][channel][output column]: the three bytes of a window
    auto windows = [&](bool row_ok, uint32_t (&v)[4][4]) {
      uint32_t e[NC];
#pragma unroll
      for (int i = 0; i < NC; ++i) e[i] = PLAIN ? d[i] : d[i] ^ (row_ok ? flip[i] : pad4);
      // four pixels of four channels to four channels of four pixels
      auto transpose = [](uint32_t a, uint32_t b, uint32_t cc, uint32_t dd, uint32_t (&o)[4]) {
        const uint32_t ab0 = __builtin_amdgcn_perm(b, a, 0x05010400u), ab1 = __builtin_amdgcn_perm(b, a, 0x07030602u);
        const uint32_t cd0 = __builtin_amdgcn_perm(dd, cc, 0x05010400u), cd1 = __builtin_amdgcn_perm(dd, cc, 0x07030602u);
        o[0] = __builtin_amdgcn_perm(cd0, ab0, 0x05040100u);
        o[1] = __builtin_amdgcn_perm(cd0, ab0, 0x07060302u);
        o[2] = __builtin_amdgcn_perm(cd1, ab1, 0x05040100u);
        o[3] = __builtin_amdgcn_perm(cd1, ab1, 0x07060302u);
      };
      uint32_t a[4];
      transpose(e[0], e[1], e[2], e[3], a);
      if constexpr (S == 1) {
        const uint32_t b01 = __builtin_amdgcn_perm(e[5], e[4], 0x05010400u), b23 = __builtin_amdgcn_perm(e[5], e[4], 0x07030602u);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t b = (j < 2 ? b01 : b23) >> (j & 1 ? 16 : 0);
          v[j][0] = a[j];
          v[j][1] = __builtin_amdgcn_alignbyte(b, a[j], 1);
          v[j][2] = __builtin_amdgcn_alignbyte(b, a[j], 2);
          v[j][3] = __builtin_amdgcn_alignbyte(b, a[j], 3);
        }
      } else {
        uint32_t b[4];
        transpose(e[4], e[5], e[6], e[7], b);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          v[j][0] = a[j];
          v[j][1] = __builtin_amdgcn_alignbyte(b[j], a[j], 2);
          v[j][2] = b[j];
          v[j][3] = __builtin_amdgcn_perm(e[8], b[j], 0x0c000302u | (uint32_t)(4 + j) << 16);
        }
      }
    };
    auto emit = [&](int oy, const uint32_t (&r0)[4][4], const uint32_t (&r1)[4][4], const uint32_t (&r2)[4][4]) {
      const int64_t base = ((int64_t)at.outer * OH + oy) * OW * C * kEsz;
      const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(static_cast<uint8_t*>(p.out) + base, 0, OW * C * kEsz, 0x00020000);
      if constexpr (FORM == kSat) {
        // two columns of a channel shift by the same amount; two permutes then sort the pairs into pixels
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
          uint32_t d01, d23;  // channels 0, 1 and 2, 3: columns i and i + 1 of each
          auto pair = [&]<int J>(uint32_t& dst) {
            int32_t r[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const int32_t a = dot4(r2[J][i + e], wt[J][2], dot4(r1[J][i + e], wt[J][1], dot4(r0[J][i + e], wt[J][0], 0)));
              r[e] = (int32_t)(((int64_t)a * (int64_t)m[J] + k64[J]) >> 32);
            }
            ashr_sat_pair<J & 1>(dst, r[0], r[1], s1[J]);
          };
          pair.template operator()<0>(d01);
          pair.template operator()<1>(d01);
          pair.template operator()<2>(d23);
          pair.template operator()<3>(d23);
#pragma unroll
          for (int e = 0; e < 2; ++e)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_amdgcn_perm(d23, d01, e ? 0x07050301u : 0x06040200u) ^ sflip, rout,
                                                  x0 + i + e < OW ? (uint32_t)((x0 + i + e) * C + c) : kOob, 0, 0);
        }
        return;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        int32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          int32_t a = dot4(r2[j][i], wt[j][2], dot4(r1[j][i], wt[j][1], dot4(r0[j][i], wt[j][0], FOLD ? 0 : corr[j])));
          if constexpr (!FOLD) a = wrap_acc_bits(a, p.acc_wrap_shift);
          if constexpr (MODE == 0) {
            const int64_t pr = (int64_t)a * (int64_t)m[j] + k64[j] + (FOLD ? 0 : (int64_t)((a >> 31) & away));
            a = med3((int32_t)(pr >> (31 + sh[j])), lo, hi) + (FOLD ? 0 : z);
          }
          v[j] = a;
        }
        const uint32_t o = x0 + i < OW ? (uint32_t)(((x0 + i) * C + c) * kEsz) : kOob;
        if constexpr (MODE == 0)
          __builtin_amdgcn_raw_buffer_store_b32(pack4_perm(v[0], v[1], v[2], v[3]), rout, o, 0, 0);
        else if constexpr (MODE == 1)
          __builtin_amdgcn_raw_buffer_store_b128(v4i{v[0], v[1], v[2], v[3]}, rout, o, 0, 0);
        else
          __builtin_amdgcn_raw_buffer_store_b64(v2i{(v[0] & 0xffff) | (int32_t)((uint32_t)v[1] << 16),
                                                    (v[2] & 0xffff) | (int32_t)((uint32_t)v[3] << 16)}, rout, o, 0, 0);
      }
    };
    // the next row's loads are under way while a row is worked on
    int iy = y0 * S - 1;
    auto step = [&](uint32_t (&v)[4][4]) {
      windows((uint32_t)iy < (uint32_t)H, v);
      load(++iy);
    };
    if constexpr (S == 1) {
      step(w[0]);
      step(w[1]);
      for (int i = 0; i < rows; i += 3) {
        step(w[2]);
        emit(y0 + i, w[0], w[1], w[2]);
        if (i + 1 >= rows) break;
        step(w[0]);
        emit(y0 + i + 1, w[1], w[2], w[0]);
        if (i + 2 >= rows) break;
        step(w[1]);
        emit(y0 + i + 2, w[2], w[0], w[1]);
      }
    } else {
      step(w[0]);
      for (int i = 0; i < rows; i += 2) {
        step(w[1]);
        step(w[2]);
        emit(y0 + i, w[0], w[1], w[2]);
        if (i + 1 >= rows) break;
        step(w[1]);
        step(w[0]);
        emit(y0 + i + 1, w[2], w[1], w[0]);
      }
    }
  };
  if constexpr (CODES != kOther) {
    if (sat) body.template operator()<kSat, CODES == kFullPlain>();
    else if (fold) body.template operator()<kFold, CODES == kFullPlain>();
    else body.template operator()<kGeneral, false>();
  } else {
    if (fold && plain) body.template operator()<kFold, true>();
    else if (fold) body.template operator()<kFold, false>();
    else body.template operator()<kGeneral, false>();
  }
}

}  // namespace

hipError_t launch_qconv_depthwise(const GemmArgs& a, const ConvGeom& cg, hipStream_t st) {
  DwArgs p{};
  p.act = static_cast<const uint8_t*>(a.act);
  p.wgt = a.wgt;
  p.bias = a.bias;
  p.out = a.out;
  p.g = cg;
  p.act_xor = a.act_unsigned ? 0x80u : 0u;
  p.act_off = a.act_unsigned ? 128 : 0;
  p.z_a = a.act_zero_point;
  p.acc16 = a.acc16;
  p.acc_wrap_shift = a.acc_wrap_shift;
  p.has_rq = a.has_rq;
  p.out_mode = a.has_rq ? 0 : (a.acc16 ? 2 : 1);
  p.mult = a.rq.multiplier;
  p.shift = a.rq.shift;
  p.per_channel = a.rq.per_channel;
  p.rs = RequantScalars{a.rq.z_out, a.rq.clip_lo - a.rq.z_out, a.rq.clip_hi - a.rq.z_out, a.rq.half_away};

  const int64_t total = (int64_t)cg.B * cg.O * cg.OH * cg.OW;
  if (total == 0) return hipSuccess;

  const bool full = a.has_rq && !a.acc16 && a.acc_wrap_shift == 0 && !p.rs.half_away && p.rs.z_out >= -256 && p.rs.z_out <= 255 && sat_range(p.rs);
  const int codes = !full ? kOther : p.act_xor == 0 && (p.z_a & 0xff) == 0 ? kFullPlain : kFullFlipped;

  const size_t esz = a.has_rq ? 1 : (a.acc16 ? 2 : 4);
  const bool k3 = cg.KH == 3 && cg.KW == 3 && cg.pad_h == 1 && cg.pad_w == 1;
  const bool s1 = k3 && cg.stride_h == 1 && cg.stride_w == 1, s2 = k3 && cg.stride_h == 2 && cg.stride_w == 2;
  // (compiled for 32- and 16-bit accumulators; 24-bit ones take the kernels that wrap by a run-time width)
  const bool regs_ok = a.acc_wrap_shift == 0 || a.acc_wrap_shift == 16;
  // channel-last
  if (cg.nhwc && (s1 || s2) && cg.C >= 4 && cg.B <= 65535 && (int64_t)cg.W * cg.C < (1ll << 31) &&
      (int64_t)cg.OW * cg.C * (int64_t)esz < (1ll << 31)) {
    const int32_t c4 = (cg.C + 3) / 4, strips = (cg.OW + 3) / 4;
    const int64_t blocks = ((int64_t)c4 * strips + kThreads - 1) / kThreads;
    // Rows per thread: long runs read few rows twice and fetch the channels' constants seldom; they end where there are
    // fewer workgroups than 1.5 per CU (32 x 56 x 56 x 144: 10.9 us so, 13.0 and 22.8 with twice and four times as many).
    int64_t run = (int64_t)cg.B * blocks * cg.OH / 384;
    run = run < 1 ? 1 : (run > 16 ? 16 : run);
    const int64_t runs = (cg.OH + run - 1) / run;
    run = (cg.OH + runs - 1) / runs;
    if (runs <= 65535 && ((int64_t)c4 * strips + kThreads) * c4 < (1ll << 32)) {
#define HAGO_DW_NHWC(S_) \
  (p.out_mode == 1 ? dw_nhwc3x3_kernel<1, S_, kOther> : p.out_mode == 2 ? dw_nhwc3x3_kernel<2, S_, kOther>      \
   : codes == kFullPlain ? dw_nhwc3x3_kernel<0, S_, kFullPlain>                                        \
   : codes == kFullFlipped ? dw_nhwc3x3_kernel<0, S_, kFullFlipped> : dw_nhwc3x3_kernel<0, S_, kOther>)
      auto kern = s1 ? HAGO_DW_NHWC(1) : HAGO_DW_NHWC(2);
#undef HAGO_DW_NHWC
      return launch_kernel(kern, dim3((unsigned)blocks, (unsigned)runs, (unsigned)cg.B), dim3(kThreads), 0, st,
                         (uint32_t)blocks, (uint32_t)runs, (uint32_t)(blocks * runs * cg.B), inverse(blocks, blocks * runs * cg.B),
                         inverse(runs, runs * cg.B), p, c4,
                         c4 > 1 ? (uint32_t)(((1ull << 32) + c4 - 1) / c4) : 0u, strips, (int32_t)run);
    }
  }
  // NCHW, stride 1, rows of more than 32 bytes: the dot-product form.  (The matrix form reads a row in 16-byte pieces, one
  // memory-pipe pass per lane; with two or more column tiles that, and not the arithmetic, bounds it: 16 x 288 planes of
  // 41 x 41 take 10.8 us there and 8.0 here, 32 x 144 of 56 x 56 the same 9.8.)
  if (regs_ok && !cg.nhwc && s1 && cg.W > 32 && cg.B <= 65535 && (int64_t)cg.H * cg.W * 4 < (1ll << 31)) {
    // bands of 4 * rpc <= 64 rows, as even as they come
    const int64_t nband = (cg.H + 63) / 64;
    const int32_t rpc = (int32_t)((cg.H + 4 * nband - 1) / (4 * nband));
    // Column segments: 64 columns each where rows are whole dwords; else as even as whole strips allow, and never with a
    // last one of fewer than four columns (a row's last strip is loaded and stored as its last four bytes).
    const bool whole = cg.W % 4 == 0 && (reinterpret_cast<uintptr_t>(a.act) & 3u) == 0;
    const bool ragged = !whole || (reinterpret_cast<uintptr_t>(a.out) & (4 * esz - 1)) != 0;
    int32_t nsegs = (cg.W + 63) / 64;
    int32_t segw = whole ? 64 : ((cg.W + nsegs - 1) / nsegs + 3) / 4 * 4;
    while (cg.W > 64 && segw > 12 && cg.W % segw != 0 && cg.W % segw < 4) segw -= 4;
    nsegs = (cg.W + segw - 1) / segw;
    if (segw > 12 && nband * nsegs <= 65535 && (int64_t)(cg.C + 3) / 4 * nsegs <= max_blocks(kThreads)) {
      // Rows in pieces slow the way to memory down from 9 to 11 MB of results on, on buffers that the last-level cache does not hold from fewer on.  Us of 144 channels with results left in the L2, sent
      // through it, and by four rows: 8 x 56 x 56 4.72, 4.42, 5.2; 24 x 56 x 56, 10.8 MB, 7.51, 7.05, 6.99; 32 x 56 x 56 8.65, 9.05, 8.15; 32 x 60 x 60
      // 9.06, 9.96, 8.51; 40 x 48 x 48, 13.3 MB, 9.12, 8.83, 8.17; 26 x 52 x 52, 10.1 MB, 7.13, 6.45, 6.73; rows of 64 bytes on 16 x 64 x 64
      // 6.53, 5.30, 6.32.  Rows off dwords: 24 x 63 x 63, 13.7 MB, 8.75, 9.35; 24 x 49 x 49 7.13, 6.67; 60 x 41 x 41, 14.5 MB, 0.4 less through it.
      // Several segments: 8 x 113 x 113 x 96 8.21, 7.31.  Beyond the last-level cache (and from it): 8 x 56 x 56 5.4, 5.9, 5.9; 16 x 56 x 56 7.2, 8.6, 7.6 (6.1,
      // 5.6, 6.3); 24 x 56 x 56 9.0, 11.2, 9.5 (7.5, 6.9, 7.1); 26 x 52 x 52 8.4, 10.5, 9.0; 32 x 56 x 56 11.0, 14.0, 11.7; 40 x 64 x 64 13.8, 14.9, 13.0 (10.6, 8.0, 9.1);
      // 60 x 41 x 41 13.3, 16.7 (10.9, 9.7); 16 x 112 x 112 x 96 14.9, 18.5 (10.2, 9.7); 8 x 224 x 224 x 64 20.3, 25.1 (13.4, 14.2): so few pieces of large layers go through.
      const int64_t gx = (int64_t)(cg.C + 3) / 4 * nsegs, mid = nband;
      const bool large = total > 11000000;
      const int how = nsegs > 1 || ragged ? (large ? kL2 : kThrough) : cg.W == 64 || total <= 9000000 ? kThrough : kFours;
#define HAGO_DW_ROWS(WIDE_, RAG_, OUT_)                                                                \
  (p.out_mode == 1 ? dw_rows3x3_kernel<1, false, WIDE_, RAG_>                                          \
   : p.out_mode == 2 ? dw_rows3x3_kernel<2, true, WIDE_, RAG_>                                         \
   : p.acc16 ? dw_rows3x3_kernel<0, true, WIDE_, RAG_, OUT_>                                           \
   : codes == kFullPlain ? dw_rows3x3_kernel<0, false, WIDE_, RAG_, OUT_, kFullPlain>                  \
   : codes == kFullFlipped ? dw_rows3x3_kernel<0, false, WIDE_, RAG_, OUT_, kFullFlipped>              \
                           : dw_rows3x3_kernel<0, false, WIDE_, RAG_, OUT_>)
      auto kern = nsegs > 1 ? (how == kL2 ? (ragged ? HAGO_DW_ROWS(true, true, kL2) : HAGO_DW_ROWS(true, false, kL2))
                               : (ragged ? HAGO_DW_ROWS(true, true, kThrough) : HAGO_DW_ROWS(true, false, kThrough)))
                  : ragged ? (how == kL2 ? HAGO_DW_ROWS(false, true, kL2) : HAGO_DW_ROWS(false, true, kThrough))
                           : (how == kFours ? HAGO_DW_ROWS(false, false, kFours) : HAGO_DW_ROWS(false, false, kThrough));
#undef HAGO_DW_ROWS
      return launch_kernel(kern, dim3((unsigned)gx, (unsigned)mid, (unsigned)cg.B), dim3(kThreads), 0, st, (uint32_t)gx, (uint32_t)mid,
                         (uint32_t)(gx * mid * cg.B), inverse(gx, gx * mid * cg.B), inverse(mid, mid * cg.B), p, rpc, nsegs, segw);
    }
  }
  // NCHW on the matrix cores
  if (!cg.nhwc && (s1 || s2)) {
    const int32_t S = cg.stride_w;
    DwTile q{cg.C, cg.H, cg.W, cg.OH, cg.OW, cg.B};
    const bool two = cg.W <= 16;  // (stride 2: at most eight outputs)
    q.groups = two ? (cg.C + 1) / 2 : cg.C;
    // columns: a row of up to 32 bytes is one tile; of a longer one the window gives 30 at most (15 at stride 2)
    q.nt = cg.W <= 32 ? 1 : (S == 1 ? (cg.OW + 29) / 30 : (cg.OW + 14) / 15);
    q.cw = q.nt == 1 ? cg.OW : (cg.OW + q.nt - 1) / q.nt;
    const int32_t up = (q.cw + 3) / 4 * 4;  // (tiles that start on dwords where the window allows it)
    if (q.nt > 1 && up <= (S == 1 ? 30 : 15)) q.cw = up;
    if (q.nt > 1 && S == 1 && q.cw < 16) q.cw = 16;
    q.inv_nt = q.nt > 1 ? (uint32_t)(((1ull << 32) + q.nt - 1) / q.nt) : 0u;
    // tiles run through images where the descriptor of the first reaches the others
    const int64_t span = (int64_t)(32 / cg.OH + 2) * cg.C;
    const bool flat = cg.OH > 1 && cg.OH < 65000 && span * cg.OH * cg.OW * (int64_t)esz < (1ll << 31) && span * cg.H * cg.W < (1ll << 31);
    q.period = flat ? cg.OH : (cg.OH + 31) / 32 * 32;
    q.inv_oh = flat ? (uint32_t)(((1ull << 32) + cg.OH - 1) / cg.OH) : 0u;
    const int64_t tiles = ((int64_t)cg.B * q.period + 31) / 32, waves_x = (int64_t)q.groups * q.nt;
    const int64_t gx = (waves_x + 3) / 4;
    const DwSplit split = dw_split(gx, waves_x, tiles);
    const int64_t gy = split.runs;
    q.per_wave = split.per;
    q.longer = split.longer;
    if (tiles < (1ll << 26) && gy <= 65535 && waves_x * q.nt < (1ll << 32) && gx <= max_blocks(kThreads) &&
        (flat || ((int64_t)cg.H * cg.W * 2 < (1ll << 31) && (int64_t)cg.OH * cg.OW * 2 * (int64_t)esz < (1ll << 31)))) {
#define HAGO_DW_MODE(S_, CPK_, NJ_) \
  (p.out_mode == 1 ? dw_mfma_kernel<1, S_, CPK_, NJ_, kOther> : p.out_mode == 2 ? dw_mfma_kernel<2, S_, CPK_, NJ_, kOther> \
   : codes == kFullPlain ? dw_mfma_kernel<0, S_, CPK_, NJ_, kFullPlain>                                \
   : codes == kFullFlipped ? dw_mfma_kernel<0, S_, CPK_, NJ_, kFullFlipped> : dw_mfma_kernel<0, S_, CPK_, NJ_, kOther>)
      auto kern = S == 2 ? (two ? HAGO_DW_MODE(2, 2, 2) : HAGO_DW_MODE(2, 1, 2))
                         : (!two ? HAGO_DW_MODE(1, 1, 4) : cg.OW > 8 ? HAGO_DW_MODE(1, 2, 4) : HAGO_DW_MODE(1, 2, 2));
#undef HAGO_DW_MODE
      return launch_kernel(kern, dim3((unsigned)gx, (unsigned)gy), dim3(kThreads), 0, st, (uint32_t)gx, split.by_xcd ? (uint32_t)(gx * gy) : 0u,
                         inverse(gx, gx * gy), p, q);
    }
  }
  const int64_t blocks = (total + kThreads - 1) / kThreads;
  const int64_t cap = 256 * 64;
  return launch_kernel(dw_direct_kernel, dim3((unsigned)(blocks < cap ? blocks : cap)), dim3(kThreads), 0, st, p);
}

}  // namespace hago
