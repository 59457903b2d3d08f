// The plan of the one-launch 3x3 convolution on NCHW tensors, which calls it takes and their tiles, and its kernels for codes clipped to their container's
// whole range; the other kinds' are in conv3x3_clipped.hip, conv3x3_words.hip and conv3x3_halves.hip.
#include "conv3x3_kernel.h"

namespace hago {

template hipError_t launch_conv3x3<kFull>(const C3Params&, int, int, int, int, size_t, int64_t, hipStream_t);

extern template hipError_t launch_conv3x3<kClipped>(const C3Params&, int, int, int, int, size_t, int64_t, hipStream_t);
extern template hipError_t launch_conv3x3<kWords>(const C3Params&, int, int, int, int, size_t, int64_t, hipStream_t);
extern template hipError_t launch_conv3x3<kHalves>(const C3Params&, int, int, int, int, size_t, int64_t, hipStream_t);

bool is_qconv3x3_nchw(const ConvGeom& cg) {
  return !cg.nhwc && cg.KH == 3 && cg.KW == 3 && cg.stride_h == 1 && cg.stride_w == 1 && cg.pad_h == 1 && cg.pad_w == 1 &&
         cg.C % 32 == 0 && cg.C <= 128 && cg.W % 4 == 0 && cg.W <= 128;
}

// Takes NCHW 3x3 stride-1 pad-1 convolutions with C a multiple of 32 up to 128, W a multiple of 4
// up to 128 and 4-byte aligned activations; returns false (nothing launched) for anything else.
bool try_qconv3x3_nchw(const GemmArgs& a, const ConvGeom& cg, hipStream_t st, hipError_t* err) {
  if (!is_qconv3x3_nchw(cg) || (reinterpret_cast<uintptr_t>(a.act) & 3u) != 0 || (int64_t)cg.B * cg.C * cg.H * cg.W >= (1ll << 31) ||
      (int64_t)cg.B * cg.O * cg.H * cg.W >= (1ll << 31))
    return false;
  C3Params p{};
  p.act = static_cast<const uint8_t*>(a.act);
  p.wgt = a.wgt;
  p.bias = a.bias;
  p.out = a.out;
  p.mult = a.rq.multiplier;
  p.shift = a.rq.shift;
  p.B = cg.B; p.C = cg.C; p.H = cg.H; p.W = cg.W; p.O = cg.O;
  p.per_channel = a.rq.per_channel;
  p.acc_wrap_shift = a.acc_wrap_shift;
  p.out_mode = a.has_rq ? 0 : (a.acc16 ? 2 : 1);
  // 64 bytes of a channel at a time go through the L2: 32-bit results up to 32 MB, one-byte results of images that begin at 16 bytes, 16-bit
  // ones of images that begin with a line.  Us through it and not: raw 64 -> 64 on 16 x 56 x 56 6.7, 8.1; 64 -> 64 on 64 x 56 x 56 14.6, 16.2;
  // 128 -> 128 on 64 x 28 x 28 13.1, 13.5; 32 -> 200 on 8 x 113 x 100 16.7, 15.7; 16 bits: 128 -> 128 on 64 x 28 x 28 14.45, 14.0; 64 -> 40 on 64
  // x 19 x 20 6.8, 5.0.  32-bit results through it and with the nontemporal hint, from the last-level cache and on buffers beyond it: 64 -> 64 on 64 x 56 x 56,
  // 51 MB, 17.0, 17.7 and 29.1, 18.1; 128 -> 128 on 64 x 28 x 28, 26 MB, 12.3, 13.3 and 13.8, 12.7.
  const int HW = cg.H * cg.W;
  p.through = p.out_mode == 0   ? HW % 16 == 0 && ptr_aligned(a.out, 16)
              : p.out_mode == 1 ? ptr_aligned(a.out, 16) && (int64_t)cg.B * cg.O * HW <= 8000000 : HW % 32 == 0 && ptr_aligned(a.out, 64);
  p.act_xor4 = a.act_unsigned ? 0x80808080u : 0u;
  p.pad4 = ((((uint32_t)a.act_zero_point) ^ (a.act_unsigned ? 0x80u : 0u)) & 0xffu) * 0x01010101u;
  p.corr_coef = (a.act_unsigned ? 128 : 0) - a.act_zero_point;
  p.rs = RequantScalars{a.rq.z_out, a.rq.clip_lo - a.rq.z_out, a.rq.clip_hi - a.rq.z_out, a.rq.half_away};
  // Tile shapes (wavefronts x 32-pixel row blocks per wavefront) and blocks of 32 or 64 output channels: those with the
  // least time on the busiest CU, in microseconds: the weights once; per tile the matrix instructions, and staging and
  // epilogue, which two workgroups on a CU do in each other's shadow.  Blocks of 32 leave less of a last block empty, make
  // twice the workgroups and need half the weights, 64 and wide tiles read fewer LDS bytes per matrix instruction (us with
  // 32 and 64, by loads of 64-bit addresses: 64 -> 64 on one 56 x 56 image 5.1, 6.9; 32 -> 72 on 28 x 49 x 48 7.9, 13.6; 128 -> 184 on 6 x 74 x 72 17.5,
  // 21.9; 128 -> 256 on 16 x 56 x 56 26.9, 23.9).
  struct Shape { int nw, af; };
  static const Shape shapes[] = {{8, 2}, {8, 1}, {4, 1}};
  size_t lds = 0;
  int nu = 0, pick = -1, tn = 0, per_cu = 1;
  int64_t ntiles = 0;
  double best = 1e300;
  for (int i = 0; i < 3; ++i)
    for (int n = 1; n <= 2; ++n) {
      const int pixels = 32 * shapes[i].nw * shapes[i].af, threads = 64 * shapes[i].nw, ob = 32 * n;
      if (i == 2 && pick >= 0) continue;  // (four wavefronts: where the wider tiles' rows do not fit the LDS)
      int tr = pixels / cg.W < cg.H ? pixels / cg.W : cg.H;
      // whole 16-pixel groups per tile where that is possible: 16-byte stores
      int gran = 16;
      for (int wv = cg.W; (wv & 1) == 0 && gran > 1; wv >>= 1) gran >>= 1;   // 16 / gcd(W, 16)
      if (tr >= gran) tr -= tr % gran;
      if (tr < 1) continue;
      const int tiles_per_img = (cg.H + tr - 1) / tr, nblk = (cg.O + ob - 1) / ob;
      const int64_t nt = (int64_t)cg.B * tiles_per_img;
      const size_t need = (size_t)ob * (9 * cg.C + 16) + (size_t)(tr + 2) * (cg.W + 2) * (cg.C + 16) + ob * sizeof(int32_t);
      const int units = ((cg.C / 16) * (tr + 2) * (cg.W / 4) + threads - 1) / threads;
      if (need > 160 * 1024 || units > 3 || nt >= (1ll << 31)) continue;
      // two workgroups on a CU, if the LDS and the registers (as compiled) of both fit it
      const int regs = 66 + 20 * units + (shapes[i].af == 2 ? (n == 2 ? 68 : 20) : (n == 2 ? 32 : 0));
      const int together = 2 * need <= 160 * 1024 && (shapes[i].nw == 4 || regs <= 128) ? 2 : 1;
      const double per = (double)((nt * nblk + 255) / 256);
      // (fewer row blocks or channels share a fragment: the LDS reads take longer than the matrix instructions)
      const int mine = shapes[i].af * n;
      const double lds_bound = mine >= 4 ? 1.0 : mine == 2 ? 1.5 : 2.0;
      const double matrix = shapes[i].nw * mine * lds_bound * 9.0 * (cg.C / 32) * 8.0 / 2100;
      const double other = 0.6 + 0.5 * units + 0.2 * mine;
      const double cost = ob * 9.0 * cg.C / 51200 + per * matrix + (per > together ? per / together : 1.0) * other;
      if (cost < best) {
        best = cost;
        pick = i; tn = n; lds = need; nu = units; ntiles = nt; per_cu = together;
        p.TR = tr; p.tiles_per_img = tiles_per_img; p.nblk = nblk;
      }
    }
  if (pick < 0) return false;
  p.ntiles = (int32_t)ntiles;
  // persistent workgroups, as many as fit the chip, shared out evenly among the blocks of output channels
  int64_t per_blk = (256ll * per_cu) / p.nblk;
  if (per_blk < 1) per_blk = 1;
  if (per_blk > ntiles) per_blk = ntiles;
  const int64_t grid = per_blk * p.nblk;
  auto inverse = [](int64_t d, int64_t n) { return d > 1 && n * d < (1ll << 32) ? (uint32_t)(((1ull << 32) + (uint64_t)d - 1) / (uint64_t)d) : 0u; };
  p.inv_tpi = inverse(p.tiles_per_img, ntiles);
  p.inv_nblk = inverse(p.nblk, grid);
  p.inv_w4 = inverse(cg.W / 4, (p.TR + 2) * (cg.W / 4));
  p.inv_run4 = inverse((p.TR + 2) * (cg.W / 4), 3 * 512);
  p.inv_w = inverse(cg.W, 512);
  const int out = p.out_mode == 1 ? kWords : p.out_mode == 2 ? kHalves : sat_range(p.rs) && !p.rs.half_away && p.acc_wrap_shift == 0 ? kFull : kClipped;
  const auto launch = out == kFull ? launch_conv3x3<kFull> : out == kClipped ? launch_conv3x3<kClipped> : out == kWords ? launch_conv3x3<kWords> : launch_conv3x3<kHalves>;
  *err = launch(p, shapes[pick].nw, shapes[pick].af, nu, tn, lds, grid, st);
  return true;
}

}  // namespace hago
