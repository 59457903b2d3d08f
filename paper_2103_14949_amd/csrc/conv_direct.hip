// The plan of the any-geometry convolution in one launch, which calls it takes and their tiles, and its kernels for codes clipped to their container's whole
// range; the other kinds' are in conv_direct_any.hip and conv_direct_sums.hip.
#include "conv_direct_kernel.h"

namespace hago {

template hipError_t launch_conv_direct<kFullCodes>(const CdParams&, bool, int, int, size_t, int64_t, hipStream_t);
extern template hipError_t launch_conv_direct<kAnyCodes>(const CdParams&, bool, int, int, size_t, int64_t, hipStream_t);
extern template hipError_t launch_conv_direct<kSums>(const CdParams&, bool, int, int, size_t, int64_t, hipStream_t);

namespace {

inline uint32_t recip(int64_t d) { return d <= 1 ? 0xffffffffu : (uint32_t)((1ull << 32) / (uint64_t)d); }

}  // namespace

// Plans the launch; false (nothing launched) when the geometry is not this kernel's: images narrower than four pixels
// (NCHW), tensors of 2^31 bytes or fewer than 16, or tiles whose rows do not fit the LDS.
bool try_qconv_direct(const GemmArgs& a, const ConvGeom& cg, int forced_shape, hipStream_t st, hipError_t* err) {
  const int64_t act_bytes = (int64_t)cg.B * cg.C * cg.H * cg.W;
  if ((!cg.nhwc && cg.W < 4) || act_bytes < 16 || act_bytes >= (1ll << 31) || (int64_t)cg.O * a.K >= (1ll << 31)) return false;
  CdParams p{};
  p.act = static_cast<const uint8_t*>(a.act);
  p.wgt = a.wgt;
  p.bias = a.bias;
  p.out = a.out;
  p.mult = a.rq.multiplier;
  p.shift = a.rq.shift;
  p.B = cg.B; p.C = cg.C; p.H = cg.H; p.W = cg.W; p.O = cg.O; p.OH = cg.OH; p.OW = cg.OW;
  p.KH = cg.KH; p.KW = cg.KW; p.sh = cg.stride_h; p.sw = cg.stride_w; p.ph = cg.pad_h; p.pw = cg.pad_w;
  p.per_channel = a.rq.per_channel;
  p.acc_wrap_shift = a.acc_wrap_shift;
  p.out_mode = a.has_rq ? 0 : (a.acc16 ? 2 : 1);
  p.act_xor4 = a.act_unsigned ? 0x80808080u : 0u;
  p.pad4 = ((((uint32_t)a.act_zero_point) ^ (a.act_unsigned ? 0x80u : 0u)) & 0xffu) * 0x01010101u;
  p.corr_coef = (a.act_unsigned ? 128 : 0) - a.act_zero_point;
  p.act_bytes = act_bytes;
  p.rs = RequantScalars{a.rq.z_out, a.rq.clip_lo - a.rq.z_out, a.rq.clip_hi - a.rq.z_out, a.rq.half_away};
  p.sr = cg.KH < cg.stride_h ? cg.KH : cg.stride_h;
  p.HV = (cg.OH - 1) * p.sr + cg.KH;
  if ((int64_t)p.HV * (cg.B + 1) >= (1ll << 31)) return false;

  // Wavefront shapes: pixels x output channels of a workgroup.
  struct Shape { int px, ch, af; };
  // (four wavefronts, two workgroups per CU, were slower throughout: the weights are staged twice as often)
  static const Shape shapes[] = {{512, 64, 2}, {256, 64, 1}, {128, 128, 1}};
  double best_cost = 1e300;
  CdParams best{};
  int best_shape = -1;
  size_t best_lds = 0;
  int64_t best_grid = 0;
  for (int s = 0; s < 3; ++s) {
    if (forced_shape >= 0 && s != forced_shape) continue;
    const Shape& sp = shapes[s];
    const int nu = cg.nhwc ? 8 : (sp.af == 2 ? 2 : 3);
    p.nblk = (cg.O + sp.ch - 1) / sp.ch;
    for (int nch = 1; nch <= 64; nch = nch < 4 ? nch + 1 : nch * 2) {
      // few channels: 4, 8 or 16 bytes per pixel, runs of taps per group; else chunks of a multiple of 32 channels
      if (cg.C <= 16) {
        if (nch > 1) break;
        p.small_c = cg.C <= 4 ? 4 : (cg.C <= 8 ? 8 : 16);
        p.CC = p.small_c; p.PS = p.small_c; p.nchunk = 1;
        p.NX = (cg.KW * p.small_c + 31) / 32; p.xB = 32; p.CK = 1;
      } else {
        p.small_c = 0;
        p.CC = ((cg.C + nch - 1) / nch + 31) / 32 * 32;
        p.nchunk = (cg.C + p.CC - 1) / p.CC;
        if (p.nchunk != nch && nch > 1 && p.CC == 32 && (cg.C + 31) / 32 < nch) break;  // no smaller chunk exists
        p.PS = p.CC + 16;
        p.NX = cg.KW; p.xB = p.PS; p.CK = p.CC / 32;
      }
      if (p.nchunk > 1 && s == 0) continue;
      p.groups = cg.KH * p.NX * p.CK;
      const int64_t wbytes = (int64_t)sp.ch * (p.groups * 32 + 16);
      if (wbytes > 150 * 1024) continue;
      for (int seg = 1; seg <= 16; ++seg) {
        int tw = (cg.OW + seg - 1) / seg;
        if (seg > 1) tw = (tw + 15) / 16 * 16;
        if (tw > sp.px) continue;
        p.nseg = (cg.OW + tw - 1) / tw;
        if (p.nseg != seg) continue;
        p.TW = tw;
        const int64_t stack = (int64_t)cg.B * cg.OH;
        int tr_max = sp.px / tw;
        if (tr_max > stack) tr_max = (int)stack;
        for (int tr = tr_max; tr >= 1; tr = tr > 8 ? tr - tr / 4 : tr - 1) {
          p.TR = tr;
          const int cross = cg.OH == 1 ? tr - 1 : (tr - 1 + cg.OH - 1) / cg.OH;  // image boundaries inside a tile, at most
          p.rows = (tr - 1) * p.sr + cg.KH + (stack > cg.OH ? cross : 0) * (cg.KH - p.sr);
          // aligned quads: the staged columns start at a multiple of four of the image row
          p.aligned = !cg.nhwc && cg.W % 4 == 0 && (p.nseg == 1 || (tw * cg.stride_w) % 4 == 0);
          p.off_x = p.aligned ? (4 - cg.pad_w % 4) % 4 : 0;
          p.Wq = ((tw - 1) * cg.stride_w + cg.KW + p.off_x + 3) / 4;
          const int64_t in_bytes = (int64_t)p.rows * p.Wq * 4 * p.PS + 64;
          const int64_t raw = (int64_t)sp.ch * a.K;  // (few channels: the weights pass through the input's place)
          int64_t room = in_bytes;
          if (p.small_c && raw + 4 > room) room = raw + 4;
          room = (room + 15) / 16 * 16;
          p.in_room = (int32_t)room;
          const int64_t lds = wbytes + room + 8ll * sp.ch * 4 + 16;
          const int64_t cgroups = p.small_c ? 1 : p.CC / 16;
          const int64_t units = cg.nhwc ? (int64_t)p.rows * p.Wq * 4 * cgroups : cgroups * p.rows * p.Wq;
          if (lds > 160 * 1024 || units > 512 * nu) continue;
          const int64_t ntiles = (stack + tr - 1) / tr * p.nseg;
          if (ntiles >= (1ll << 30)) continue;
          int64_t per_blk = 256 / p.nblk;  // (eight wavefronts of up to 256 registers: one workgroup per CU)
          if (per_blk < 1) per_blk = 1;
          if (per_blk > ntiles) per_blk = ntiles;
          const int64_t grid = per_blk * p.nblk;
          const double rounds = (double)((ntiles + per_blk - 1) / per_blk) * (double)((grid + 255) / 256);
          // Cycles, from phase timestamps: weights (once, or with every chunk), staging, matrix instructions (two wavefronts
          // per SIMD, or the LDS reads that feed them), epilogue with its partial groups of 16 pixels.
          const double wst = (double)wbytes / 512 * 8.0 + 800;
          // (NCHW: a row of every channel is a run of its own, short runs fetch mostly other lines' bytes)
          const double lines = cg.nhwc ? 0 : (double)(p.small_c ? cg.C : p.CC) * p.rows * (p.Wq * 4 / 128.0 + 1);
          const double stage = (double)units / 512 * (cg.nhwc ? 150 : 600) + lines * 2 + 1500;
          const double mm = (double)p.groups * (sp.af == 2 ? 256 : 192) + 500;
          const double ohw = (double)cg.OH * cg.OW, pt = (double)tr * tw;
          double slow = 0;
          if (!cg.nhwc) slow = p.nseg > 1 ? (cg.OW % 16 ? 0.3 : 0.0) : ((int64_t)ohw % 16 ? 16.0 / ohw : 0.0) + ((int64_t)pt % 16 ? 16.0 / pt : 0.0);
          const double epi = sp.af * (2400.0 + (slow < 1 ? slow : 1) * 3000.0);
          const double cost = 3000 + (p.nchunk == 1 ? wst : 0) + rounds * (p.nchunk * (stage + mm + (p.nchunk > 1 ? wst + 3000 : 0)) + epi);
          if (cost < best_cost) {
            best_cost = cost; best = p; best.ntiles = (int32_t)ntiles; best_shape = s; best_lds = (size_t)lds; best_grid = grid;
          }
        }
      }
    }
  }
  if (best_shape < 0) return false;
  // results that a lane's store takes: of one image (or row) and at 16 bytes; channel-last: of one pixel, one-byte ones a whole line's
  const int64_t run = a.has_rq ? 16 : (a.acc16 ? 8 : 4);
  best.through = cg.nhwc ? (a.has_rq ? a.N % 64 == 0 && ptr_aligned(a.out, 64) : a.N % run == 0 && ptr_aligned(a.out, 16))
                         : ptr_aligned(a.out, 16) && (best.nseg == 1 ? (int64_t)cg.OH * cg.OW % run == 0 && (int64_t)best.TR * best.TW % run == 0
                                                                     : cg.OW % run == 0);
  const int best_cg = best.small_c ? 1 : best.CC / 16;
  best.inv_unit1 = recip(cg.nhwc ? (int64_t)best.Wq * 4 * best_cg : (int64_t)best.rows * best.Wq);
  best.inv_unit2 = recip(cg.nhwc ? best_cg : best.Wq);
  best.inv_hv = recip(best.HV); best.inv_oh = recip(best.OH); best.inv_tw = recip(best.TW); best.inv_nseg = recip(best.nseg);
  const int taps = cg.KH * cg.KW;
  const bool contiguous = !best.small_c && (cg.nhwc || taps == 1), taps9 = !best.small_c && !cg.nhwc && taps == 9;
  best.inv_wper = recip(taps9 ? best.CC / 4 : (contiguous ? (int64_t)taps * (best.CC / 16) : (int64_t)best.groups * 8));
  best.inv_line = recip(best.small_c ? best.NX * 32 : best.CC);
  best.inv_bpp = recip(best.small_c ? best.small_c : best.CC);
  best.inv_c16 = recip(best.CC / 16);
  const bool full = sat_range(p.rs) && !p.rs.half_away && p.acc_wrap_shift == 0 && p.rs.z_out >= -256 && p.rs.z_out <= 255 && a.K <= 65536;
  const auto launch = !a.has_rq ? launch_conv_direct<kSums> : full ? launch_conv_direct<kFullCodes> : launch_conv_direct<kAnyCodes>;
  *err = launch(best, cg.nhwc, contiguous ? 2 : taps9 ? 9 : 0, best_shape, best_lds, best_grid, st);
  return true;
}

}  // namespace hago
