// 1x1 convolution (stride 1, no padding, groups == 1) on NCHW tensors, straight from the
// caller's buffers: out[b][n][p] = sum_c (a[b][c][p] - z_a) * w[n][c] + bias[n], p = y * W + x.
//
// In NCHW the reduction index c is the slow one, while the MFMA wants, per lane, 16
// consecutive k-bytes of one row.  The general convolution path therefore rewrites the input
// into a channel-last copy first, which for this operator (few output channels, so hardly any
// reuse of the input) costs more memory traffic than the convolution itself.  Here lanes load dwords (four consecutive
// pixels of one channel) and transpose 4x4 byte blocks in registers.  The MFMA runs with the pixels as its P operand: a
// lane then owns one output channel and, per group of accumulator registers, consecutive pixels, which are packed and
// stored together.  Every block of 32 output channels reads the input again, from the cache; against the forms that read
// it once (conv_direct.hip, or a channel-last copy in the workspace and qgemm_dma.hip) that is the faster one up to the
// largest layers (us here, there without and with a workspace: 64 -> 384 on 8 x 56 x 56 6.5, 12.7; 512 -> 128 on
// 4 x 28 x 28 5.3, 10.6; 256 -> 256 on 32 x 28 x 28 9.8, 11.8, 15.4; 512 -> 512 29.9, 28.2, 28.1; 1024 -> 1024 on
// 32 x 14 x 14 26, 38, 27.5), so it serves every layer of its kind.
//
// Out-of-range channels and pixels are fetched through buffer descriptors with out-of-range
// offsets (they read as 0; the weights of padded channels are 0 as well).
#include "hago_device.h"
#include "launch.h"

namespace hago {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr uint32_t kOob = 0x80000000u;

struct PwArgs {
  const uint8_t* act;
  const int8_t* wgt;
  const int32_t* bias;
  void* out;
  const int32_t* mult;
  const int32_t* shift;
  int32_t C, HW, N;
  int32_t tiles_per_img;
  int32_t per_wave;            // blocks of 32 output channels of a wavefront
  int32_t nblocks;             // such groups of blocks
  uint32_t inv_tpi, inv_nb;    // ceil(2^32 / tiles_per_img) and of nblocks where that divides exactly, else 0
  uint32_t ids;        // wavefronts (or four of them) of the launch
  int32_t corr_coef;   // off - z_a
  uint32_t flags;
  RequantScalars rs;
};
static_assert(sizeof(PwArgs) <= kCheapArguments);
enum : uint32_t { kFlip = 1, kPerChannel = 2, kThrough = 4 };  // uint8 activations; a multiplier per channel; results go through the L2

// MODE 0: requantized 8-bit, 1: raw int32, 2: raw int16; ACC16: accumulator wraps to 16 bits.
// A wavefront owns 128 consecutive pixels of one image and a block (or several) of 32 output channels, as four MFMA row
// tiles.  Lane (i, h) loads, for each of its 16 channels (k-half h), the dword of pixels 4i .. 4i+3:
// consecutive lanes read consecutive dwords, so a load instruction covers 128 contiguous bytes
// of a channel (two channels per instruction).  Four 4x4 byte transposes inside the lane (eight byte permutes each, no
// lane exchange) turn the 16 dwords into the 16 k-bytes of each of the lane's four pixels, and pixel 4i + j becomes row i
// of row tile j: four MFMAs share one weight operand.  On the way out lane (n, h) then holds, for its output channel,
// registers (g, e) of tile j = pixel 4 * (8g + 4h + e) + j: the four tiles pack into one dword and the four e into 16
// contiguous bytes.  64 lanes that store 16 bytes each to 32 channels take 168 cycles of the memory pipe (256 off 16 bytes),
// a bound for large images; so pieces of one channel are brought together first, 64 bytes of it in the four lanes of a
// quad: the two halves of the wavefront swap registers (v_permlane32_swap), the lanes of a quad transpose four by DPP (raw results: a
// lane's four e are 64 or 32 bytes).  Us with the lanes' own pieces stored and so: 24 -> 144 channels on 32 x 56 x 56 8.1, 7.6, on 16 x 55 x 55 6.0, 5.1;
// 64 -> 384 on 8 x 56 x 56 7.75, 6.5; raw 32 -> 192 on 16 x 28 x 28 6.6, 4.6.  (Through LDS: slower than either.)
//   SMALL: images of less than 128 pixels, whose lanes store their own pieces, whole or by fours (64 -> 384 raw on 8 x 9 x
//     9 3.3 us, 3.7 otherwise).
// Rows start at any byte (the loads and stores are unaligned ones).  The last tile of an image is moved back to end with
// it, so that tiles are whole and pixels covered twice get the same value; of an image of less than 128 pixels the last
// four are.
//   CH = 1, 2, 3 (C <= 96): all input channels of a tile are transposed once and stay in registers for several blocks of
//     output channels (88 -> 528 on 8 x 56 x 56: 11.2 us with a wavefront for every block, 9.4 so).
//   CH = 5: five steps of 32 channels are in flight at a time.
//   RANGE: codes clipped to their container's whole range (32-bit accumulator, rounding half up), in a kernel without the other forms (us in
//     one kernel and so: 24 -> 144 on 32 x 56 x 56 6.6, 6.5; 32 -> 192 on 4 x 112 x 112 4.7, 4.55; 432 -> 72 and 72 -> 432 with their depthwise layer 24.2, 24.0).
//     The folded form stays beside the saturating one, for the 32 channels around one of shift 0 (in the general form and so: 24 -> 144 on 32 x 56 x 56
//     11.1, 7.7; 64 -> 384 on 500 x 8 x 8 13.8, 9.8; without such a channel 6.99, 7.04 and 8.99, 9.00).
//   KS = 4: four wavefronts share a tile and block, a quarter of the steps each, and add up through LDS (576 -> 96
//     channels of one 14 x 14 image are six tiles, 18 steps in a row each, else: 8.6 us, 5.8 so).
typedef uint32_t u32_u __attribute__((aligned(1)));
typedef v4i v4i_u __attribute__((aligned(1)));
typedef int v2i_u __attribute__((ext_vector_type(2), aligned(1)));

template <int MODE, bool ACC16, int KS, int CH, bool SMALL, bool RANGE>
__global__ __launch_bounds__(64 * KS, 2) void pw_nchw_kernel(PwArgs p) {
  constexpr int kPart = 65;  // dwords of a lane's partial sums: 64 accumulators and the row sum (odd: no bank conflicts)
  __shared__ int32_t lds[KS == 1 ? 1 : KS * 64 * kPart];
  const int lane = threadIdx.x & 63;
  const int wave = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Workgroups go to the eight XCDs round-robin.  A channel plane is not a multiple of the
  // 128-byte line in general, so neighbouring tiles share lines, and the blocks of output channels of a tile share its
  // input; numbering them so that an XCD gets a run of consecutive ones lets that XCD's L2 serve the shared lines (with
  // the plain order every such line was fetched from memory by two XCDs: 1.5 times the bytes).
  const uint32_t id = xcd_run(blockIdx.x, p.ids);
  const uint32_t tile = p.inv_nb ? __umulhi(id, p.inv_nb) : id / (uint32_t)p.nblocks;
  const int blk0 = (int)(id - tile * (uint32_t)p.nblocks) * p.per_wave;
  const int b = (int)(p.inv_tpi ? __umulhi(tile, p.inv_tpi) : tile / (uint32_t)p.tiles_per_img);
  const int C = p.C, HW = p.HW, N = p.N;
  const uint32_t act_xor4 = p.flags & kFlip ? 0x80808080u : 0u;
  const bool per_channel = p.flags & kPerChannel, through = p.flags & kThrough;
  int pix0 = ((int)tile - b * p.tiles_per_img) * 128;
  if (HW >= 128 && pix0 > HW - 128) pix0 = HW - 128;
  const int i = lane & 31, h = lane >> 5;

  const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(p.act) + (int64_t)b * C * HW, 0, C * HW, 0x00020000);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t*>(p.wgt), 0, N * C, 0x00020000);
  // the lane's four pixels, and its 16 channels of a step
  int px = pix0 + 4 * i;
  const bool px_ok = px < HW;
  if (px > HW - 4) px = HW - 4;
  const uint32_t a_lane = px_ok ? (uint32_t)(px + 16 * h * HW) : kOob;

  const int ksteps = (C + 31) >> 5, whole = C >> 5;
  const uint32_t k_left = (uint32_t)(C - 32 * whole);  // channels of the last, partial step
  // channels 4m .. 4m+3 of the lane's 16 exist or not as a whole (C % 4 == 0): the ones that do not must be exactly
  // zero on both sides (the flip would make them -128, and the 16-byte weight load runs into the next row)
  auto live = [&](int s, int m) { return s < whole || 16u * h + 4u * m < k_left ? 0xffffffffu : 0u; };
  auto load_a = [&](int s, uint32_t (&ab)[16]) {
    const uint32_t so = (uint32_t)(32 * s) * (uint32_t)HW;
    if (s < whole) {  // uniform
#pragma unroll
      for (int d = 0; d < 16; ++d) ab[d] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rin, a_lane, so + (uint32_t)(d * HW), 0);
    } else {  // channels beyond C are not fetched
#pragma unroll
      for (int d = 0; d < 16; ++d)
        ab[d] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
            rin, a_lane != kOob && 16u * h + d < k_left ? a_lane + so + (uint32_t)(d * HW) : kOob, 0, 0);
    }
  };
  auto load_w = [&](int s, int n) {
    return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(
        rw, n < N && 32 * s + 16 * h < C ? (uint32_t)(n * C + 16 * h) + (uint32_t)(32 * s) : kOob, 0, 0));
  };
  auto operand = [&](int s, const uint32_t (&ab)[16], v4i (&af)[4]) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      // rows a..d = channels 4m .. 4m+3, bytes = pixels 0..3  ->  rows = pixels, bytes = channels
      const uint32_t a = ab[4 * m], bq = ab[4 * m + 1], c = ab[4 * m + 2], d = ab[4 * m + 3];
      const uint32_t t0 = __builtin_amdgcn_perm(bq, a, 0x05010400u);  // a0 b0 a1 b1
      const uint32_t t1 = __builtin_amdgcn_perm(bq, a, 0x07030602u);  // a2 b2 a3 b3
      const uint32_t t2 = __builtin_amdgcn_perm(d, c, 0x05010400u);   // c0 d0 c1 d1
      const uint32_t t3 = __builtin_amdgcn_perm(d, c, 0x07030602u);   // c2 d2 c3 d3
      const uint32_t x4 = act_xor4 & live(s, m);  // (bytes that were not fetched are 0 and stay it)
      af[0][m] = (int)(__builtin_amdgcn_perm(t2, t0, 0x05040100u) ^ x4);
      af[1][m] = (int)(__builtin_amdgcn_perm(t2, t0, 0x07060302u) ^ x4);
      af[2][m] = (int)(__builtin_amdgcn_perm(t3, t1, 0x05040100u) ^ x4);
      af[3][m] = (int)(__builtin_amdgcn_perm(t3, t1, 0x07060302u) ^ x4);
    }
  };
  v16i acc[4];
  int32_t wsum;
  auto clear = [&]() {
    wsum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][r] = 0;
  };
  auto multiply = [&](int s, v4i wb, const v4i (&af)[4]) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      wb[m] &= (int)live(s, m);
      wsum = __builtin_amdgcn_sdot4(wb[m], 0x01010101, wsum, false);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[j], wb, acc[j], 0, 0, 0);
  };
  struct Rq { int32_t bias, m, sh; };  // of the lane's output channel
  auto load_rq = [&](int n) {
    Rq r{0, 0, 0};
    if (n < N) {
      if (p.bias) r.bias = p.bias[n];
      if (MODE == 0) {
        r.m = rq_mult(p.mult, per_channel ? n : 0);
        r.sh = rq_shift(p.mult, p.shift, per_channel ? n : 0);
      }
    }
    return r;
  };

  const RequantScalars rs = p.rs;
  constexpr int kEsz = MODE == 0 ? 1 : (MODE == 1 ? 4 : 2);
  // results of output channel n from the accumulators (KS = 4: of register group `wave` only, in the first four registers)
  auto finish = [&](int n0, int n, Rq rq) {
    const int32_t corr = rq.bias + p.corr_coef * wsum;
    const int64_t rnd = (int64_t)1 << (30 + rq.sh);
    uint8_t* const orow = static_cast<uint8_t*>(p.out) + ((int64_t)b * N + n) * HW;  // (8-bit results)
    // FOLD (requantized, 32-bit accumulator, every lane's constants small enough): the correction
    // term, the rounding term and the output zero point go into one 64-bit constant per lane, so
    // an output is clamp((acc * m + k64) >> (31 + sh)) against the absolute bounds:
    // ((acc + corr) * m + rnd) >> s + z == (acc * m + corr * m + rnd + z * 2^s) >> s exactly, and
    // acc + corr cannot wrap when |corr| <= 2^30 and |acc| <= 2^30 (|acc| <= C * 2^15 < 2^30 for
    // C < 2^15).  With sh <= 19 and an 8-bit z nothing leaves 63 bits.
    // SAT (the same, sh >= 1 and a clip to the container's whole range): two results' shift, clip and pack are one
    // instruction, 9 cycles per output in all instead of 16 (24 -> 144 channels on 32 x 56 x 56: 0.6 us less).
    enum { kGeneral, kFold, kSat };
    const int32_t away = rs.half_away ? -1 : 0;  // mask of the sign-bit correction
    auto store_all = [&]<int FORM>() {
      constexpr bool FOLD = FORM != kGeneral;
      const int32_t lo = rs.lo_rel + (FOLD ? rs.z_out : 0), hi = rs.hi_rel + (FOLD ? rs.z_out : 0);
      const int32_t zc = rs.z_out + (FORM == kSat ? sat_bias(rs) : 0);
      const int64_t k64 = FOLD ? (int64_t)corr * rq.m + rnd + ((int64_t)zc << (31 + rq.sh)) : rnd;
      const uint32_t flip = sat_flip(rs);
      const int32_t add = FOLD ? 0 : corr;
      constexpr int kGroups = 4 / KS;
      uint32_t dw[kGroups][4];
#pragma unroll
      for (int g = 0; g < kGroups; ++g) {
        uint32_t raw[4][MODE == 1 ? 4 : 2];
        const int32_t mult = opaque(rq.m);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          int32_t v[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            v[j] = acc[j][4 * g + e] + add;
            if (ACC16) v[j] = (int32_t)(int16_t)v[j];
          }
          if constexpr (MODE == 0 && FORM == kSat) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = (int32_t)(((int64_t)v[j] * (int64_t)mult + k64) >> 32);
            ashr_sat_pair<0>(dw[g][e], v[0], v[1], rq.sh - 1);
            ashr_sat_pair<1>(dw[g][e], v[2], v[3], rq.sh - 1);
            dw[g][e] ^= flip;
          } else if constexpr (MODE == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              // (general form only: halves away from zero add the accumulator's sign bit)
              const int64_t pr = (int64_t)v[j] * (int64_t)mult + k64 + (FOLD ? 0 : (int64_t)((v[j] >> 31) & away));
              v[j] = med3((int32_t)(pr >> (31 + rq.sh)), lo, hi) + (FOLD ? 0 : rs.z_out);
            }
            dw[g][e] = pack4_perm(v[0], v[1], v[2], v[3]);
          } else if constexpr (MODE == 1) {
#pragma unroll
            for (int j = 0; j < 4; ++j) raw[e][j] = (uint32_t)v[j];
          } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) raw[e][j] = ((uint32_t)v[2 * j] & 0xffffu) | ((uint32_t)v[2 * j + 1] << 16);
          }
        }
        if constexpr (MODE == 0 && (KS == 4 || SMALL)) {
          const int pg = pix0 + 32 * (KS == 1 ? g : wave) + 16 * h;
          if (n < N && pg + 16 <= HW) {
            *reinterpret_cast<v4i_u*>(orow + pg) = v4i{(int)dw[g][0], (int)dw[g][1], (int)dw[g][2], (int)dw[g][3]};
          } else if (n < N) {  // (an image of less than 128 pixels)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (pg + 4 * e < HW) *reinterpret_cast<u32_u*>(orow + (pg + 4 * e > HW - 4 ? HW - 4 : pg + 4 * e)) = dw[g][e];
          }
        } else if constexpr (MODE != 0) {
          // four pixels a piece: four lanes write 64 (32) consecutive bytes
          if constexpr (!SMALL) quad_transpose(raw, lane);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const int nn = SMALL ? n : (n & ~3) + t;
            int pq = pix0 + 32 * (KS == 1 ? g : wave) + 16 * h + 4 * (SMALL ? t : lane & 3);
            const bool ok = nn < N && pq < HW;
            if (pq > HW - 4) pq = HW - 4;
            uint8_t* const dst = static_cast<uint8_t*>(p.out) + (((int64_t)b * N + nn) * HW + pq) * kEsz;
            if constexpr (MODE == 1) {
              if (ok) store16(!SMALL && through, dst, raw[t][0], raw[t][1], raw[t][2], raw[t][3]);
            } else {
              if (ok) *reinterpret_cast<v2i_u*>(dst) = v2i_u{(int)raw[t][0], (int)raw[t][1]};
            }
          }
        }
      }
      if constexpr (MODE == 0 && KS == 1 && !SMALL) {
        // pieces 2g + h of 16 pixels: the upper ones to the upper half of the wavefront, then to the lanes of a quad
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            const auto sw = __builtin_amdgcn_permlane32_swap(dw[g][e], dw[g + 2][e], false, false);
            dw[g][e] = sw[0], dw[g + 2][e] = sw[1];
          }
          const uint32_t x = dw[1][e];
          dw[1][e] = dw[2][e], dw[2][e] = x;
        }
        quad_transpose(dw, lane);
        uint8_t* const first_row = static_cast<uint8_t*>(p.out) + ((int64_t)b * N + n0) * HW;
        auto row = [&](int nn) { return first_row + (uint64_t)(uint32_t)(nn - n0) * (uint32_t)HW; };
        const int pg = pix0 + 64 * h + 16 * (lane & 3);
#pragma unroll
        for (int t = 0; t < kGroups; ++t) {
          const int nn = (n & ~3) + t;
          if (nn < N) store16(through, row(nn) + pg, dw[t][0], dw[t][1], dw[t][2], dw[t][3]);
        }
      }
    };
    const bool lane_ok = rq.sh >= 0 && rq.sh <= 19 && corr >= -(1 << 30) && corr <= (1 << 30);
    const bool fold = MODE == 0 && !ACC16 && C < (1 << 15) && rs.z_out >= -256 && rs.z_out <= 255 &&
                      !rs.half_away && __builtin_amdgcn_ballot_w64(!lane_ok) == 0;  // wavefront-uniform
    if constexpr (RANGE) {
      if (fold && __builtin_amdgcn_ballot_w64(n < N && rq.sh < 1) == 0) store_all.template operator()<kSat>();
      else if (fold) store_all.template operator()<kFold>();
      else store_all.template operator()<kGeneral>();
    } else {
      if (fold) store_all.template operator()<kFold>();
      else store_all.template operator()<kGeneral>();
    }
  };

  if constexpr (KS == 1 && CH <= 3) {
    uint32_t ab[CH][16];
#pragma unroll
    for (int s = 0; s < CH; ++s) load_a(s, ab[s]);
    v4i wb[CH], wn[CH];
    auto load_block = [&](int blk, v4i (&w)[CH]) {
#pragma unroll
      for (int s = 0; s < CH; ++s) w[s] = load_w(s, blk * 32 + i);
      return load_rq(blk * 32 + i);
    };
    Rq rq = load_block(blk0, wb);
    v4i af[CH][4];
#pragma unroll
    for (int s = 0; s < CH; ++s) operand(s, ab[s], af[s]);
    const int blocks = (N + 31) >> 5, last = blk0 + p.per_wave < blocks ? blk0 + p.per_wave : blocks;
    for (int blk = blk0; blk < last; ++blk) {
      clear();
#pragma unroll
      for (int s = 0; s < CH; ++s) multiply(s, wb[s], af[s]);
      Rq rn{0, 0, 0};
      if (blk + 1 < last) rn = load_block(blk + 1, wn);  // under way during this block's results
      wsum += __shfl_xor(wsum, 32);                      // the two k-halves of the row sums
      finish(blk * 32, blk * 32 + i, rq);
      rq = rn;
#pragma unroll
      for (int s = 0; s < CH; ++s) wb[s] = wn[s];
    }
  } else {
    const int n = blk0 * 32 + i;
    clear();
    // FULL: all CH steps exist and are whole, so the code has no branches and the compiler waits for each
    // step's loads separately (the first MFMAs run while later steps are still arriving)
    auto chunk = [&]<bool FULL>(int s0) {
      uint32_t ab[CH][16];
      v4i wb[CH];
      if constexpr (FULL) __builtin_assume(s0 + (CH - 1) * KS < whole);
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int s = s0 + u * KS;
        if (FULL || s < ksteps) {  // uniform
          if constexpr (FULL) {
            const uint32_t so = (uint32_t)(32 * s) * (uint32_t)HW;
#pragma unroll
            for (int d = 0; d < 16; ++d) ab[u][d] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rin, a_lane, so + (uint32_t)(d * HW), 0);
          } else {
            load_a(s, ab[u]);
          }
          wb[u] = load_w(s, n);
        }
      }
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int s = FULL ? 0 : s0 + u * KS;  // (step 0 is a whole one wherever FULL is)
        if (FULL || s < ksteps) {  // uniform
          v4i af[4];
          operand(s, ab[u], af);
          multiply(s, wb[u], af);
        }
      }
    };
    const Rq rq = load_rq(n);
    for (int s0 = wave; s0 < ksteps; s0 += CH * KS) {
      if (s0 + (CH - 1) * KS < whole)
        chunk.template operator()<true>(s0);
      else
        chunk.template operator()<false>(s0);
    }
    wsum += __shfl_xor(wsum, 32);  // the two k-halves of the row sums
    if constexpr (KS > 1) {
      // each wavefront takes one group g of registers of all four tiles
      int32_t* part = lds + (wave * 64 + lane) * kPart;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) part[(r >> 2) * 16 + j * 4 + (r & 3)] = acc[j][r];
      part[64] = wsum;
      __syncthreads();
      const int32_t* mine = lds + lane * kPart;
      wsum = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j][e] = 0;
#pragma unroll
      for (int w = 0; w < KS; ++w) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[j][e] += mine[w * 64 * kPart + wave * 16 + j * 4 + e];
        wsum += mine[w * 64 * kPart + 64];
      }
    }
    finish(blk0 * 32, n, rq);
  }
}

// Wavefronts of the variant for CH = 2 and 3 (33 to 64 and 65 to 96 channels) that a SIMD has registers for, of 512: up to 128
// registers a wavefront four, up to 168 three, up to 256 two.
constexpr int waves_per_simd(int mode, bool acc16, int ch, bool small) {
  const bool wide = mode == 0 && !acc16;  // (64-bit requantize of four values at a time)
  if (ch == 3) return wide || small ? 2 : 3;
  return small ? (wide ? 2 : 3) : (mode == 2 ? 4 : 3);
}

template <int MODE, bool ACC16>
hipError_t launch(PwArgs q, int64_t tiles, hipStream_t st) {
  const int32_t blocks = (q.N + 31) / 32;
  // C <= 96: several blocks per wavefront.  Above 32 channels as few as bring all wavefronts into one round, by the registers of the
  // variant (us with 1, 2 and 3 blocks: 72 -> 432 on 42 x 28 x 28, 4116 blocks, two wavefronts per SIMD, 13.5, 12.8,
  // 11.3; 96 -> 576 on 2 x 112 x 112, 3528, two, 11.1, 9.7, 11.1; 56 -> 336 on 4 x 98 x 98, 3344, three, 9.2, 8.2, 9.4; 64 -> 384 on 8 x
  // 56 x 56, 2400, three, 6.8, 7.4; with 16-bit accumulators 88 -> 44 on 285 x 20 x 20, 2280, three, 9.8, 10.8).  Over 416 layers of all
  // variants such a count is 1.5 % from the best of five, with two wavefronts above 64 channels and three below for all of them 2.1.
  // Where one round cannot hold them, and up to 32 channels, so many blocks that 1.5 wavefronts per SIMD are left (24 -> 144
  // -> 24 with its depthwise layer on 32 x 56 x 56, 4000 blocks of the first, 24.2, 23.3).
  const int64_t all = tiles * blocks, slots = 1024 * waves_per_simd(MODE, ACC16, q.C > 64 ? 3 : 2, q.HW < 128);
  int64_t per = 1;
  if (q.C <= 32 || tiles > slots) per = q.C <= 96 && all >= 1536 ? all / 1536 : 1;
  else if (q.C <= 96) per = (blocks + slots / tiles - 1) / (slots / tiles);
  q.per_wave = (int32_t)(per < blocks ? per : blocks);
  q.nblocks = (blocks + q.per_wave - 1) / q.per_wave;
  q.per_wave = (blocks + q.nblocks - 1) / q.nblocks;
  const int64_t ids = tiles * q.nblocks;
  q.ids = (uint32_t)ids;
  auto inverse = [&](int32_t d, int64_t n) { return d > 1 && n * d < (1ll << 32) ? (uint32_t)(((1ull << 32) + d - 1) / d) : 0u; };
  q.inv_tpi = inverse(q.tiles_per_img, tiles);
  q.inv_nb = inverse(q.nblocks, ids);
  // Four wavefronts per tile and block up to where one each fills half of the SIMDs (us with four and with one: 384 -> 64
  // on 8 x 56 x 56, 400 of them, 6.0, 7.9; 480 -> 80 on 2 x 112 x 112, 588, 10.5, 8.3).
  auto run = [&]<int KS, int CH>() {
    auto go = [&]<bool RANGE>() {
      const auto kern = KS == 1 && q.HW < 128 ? pw_nchw_kernel<MODE, ACC16, KS, CH, KS == 1, RANGE> : pw_nchw_kernel<MODE, ACC16, KS, CH, false, RANGE>;
      return launch_kernel(kern, dim3((unsigned)ids), dim3(64 * KS), 0, st, q);
    };
    if constexpr (MODE == 0 && !ACC16) {
      if (sat_range(q.rs) && !q.rs.half_away && q.rs.z_out >= -256 && q.rs.z_out <= 255) return go.template operator()<true>();
    }
    return go.template operator()<false>();
  };
  if (q.C > 64 && ids <= 512) return run.template operator()<4, 5>();
  if (q.C <= 32) return run.template operator()<1, 1>();
  if (q.C <= 64) return run.template operator()<1, 2>();
  if (q.C <= 96) return run.template operator()<1, 3>();
  return run.template operator()<1, 5>();
}

}  // namespace

bool is_qconv_pointwise_nchw(const ConvGeom& cg) {
  return !cg.nhwc && cg.KH == 1 && cg.KW == 1 && cg.stride_h == 1 && cg.stride_w == 1 && cg.pad_h == 0 && cg.pad_w == 0 &&
         cg.C % 4 == 0 && (int64_t)cg.H * cg.W >= 4;
}

// Returns false (and launches nothing) when the geometry is not this kernel's.
bool try_qconv_pointwise_nchw(const GemmArgs& a, const ConvGeom& cg, hipStream_t st, hipError_t* err) {
  const int64_t HW = (int64_t)cg.H * cg.W;
  if (a.acc_wrap_shift != 0 && a.acc_wrap_shift != 16) return false;  // 24-bit accumulators: the general path
  if (!is_qconv_pointwise_nchw(cg) || (int64_t)cg.C * HW >= (1ll << 31) || (int64_t)cg.O * cg.C >= (1ll << 31) ||
      cg.B * ((HW + 127) / 128) * ((cg.O + 31) / 32) > max_blocks(64))
    return false;
  PwArgs p{};
  p.act = static_cast<const uint8_t*>(a.act);
  p.wgt = a.wgt;
  p.bias = a.bias;
  p.out = a.out;
  p.mult = a.rq.multiplier;
  p.shift = a.rq.shift;
  p.C = cg.C; p.HW = (int32_t)HW; p.N = cg.O;
  p.tiles_per_img = (int32_t)((HW + 127) / 128);
  const int64_t tiles = (int64_t)cg.B * p.tiles_per_img;
  p.corr_coef = (a.act_unsigned ? 128 : 0) - a.act_zero_point;
  p.rs = RequantScalars{a.rq.z_out, a.rq.clip_lo - a.rq.z_out, a.rq.clip_hi - a.rq.z_out, a.rq.half_away};
  // 64 bytes of a row at a time, 128 where they are one-byte results, go through the L2 unless they begin off 16 bytes: one-byte results
  // of a row of 900 and more do there too (24 -> 144 on 32 x 56 x 56, us through it and not: 6.4, 7.7; 32 -> 192 on 4 x 112 x 112 4.55, 5.69; 12 x 55 x 55 4.83, 5.05; 24 x 35 x 35
  // 4.53, 4.71; 32 x 23 x 23 4.10, 4.00; 64 x 13 x 13 3.87, 3.72; raw on 16 x 28 x 28 3.82, 4.64; on 8 x 57 x 57 7.35, 7.06).
  const bool through = a.has_rq ? (HW % 16 == 0 && ptr_aligned(a.out, 16)) || HW >= 900 : !a.acc16 && HW % 4 == 0 && ptr_aligned(a.out, 16);
  p.flags = (a.act_unsigned ? kFlip : 0u) | (a.rq.per_channel ? kPerChannel : 0u) | (through ? kThrough : 0u);
  if (tiles == 0) return false;
  if (a.has_rq) *err = a.acc16 ? launch<0, true>(p, tiles, st) : launch<0, false>(p, tiles, st);
  else *err = a.acc16 ? launch<2, true>(p, tiles, st) : launch<1, false>(p, tiles, st);
  return true;
}

}  // namespace hago
