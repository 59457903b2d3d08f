// What the any-geometry convolution's plan (conv_direct.hip) and its kernels (conv_direct_kernel.h) share.
#pragma once

#include "qgemm_common.h"

namespace hago {

struct CdParams {
  const uint8_t* act;
  const int8_t* wgt;
  const int32_t* bias;
  void* out;
  const int32_t* mult;
  const int32_t* shift;
  int32_t B, C, H, W, O, OH, OW, KH, KW, sh, sw, ph, pw;
  int32_t TR, TW, nseg;       // tile: stacked output rows x columns; column segments per row
  int32_t ntiles, nblk;       // pixel tiles, blocks of output channels
  int32_t sr, HV;             // staged rows per output row, per image
  int32_t Wq, rows;           // staged quads of columns per row, most staged rows of a tile
  int32_t in_room;            // LDS bytes of the staged input (few channels: a group may run 31 bytes past the last row)
  int32_t CC, PS, nchunk;     // channels per chunk, bytes per staged pixel
  int32_t small_c;            // 0, or bytes per pixel (4, 8, 16) of the form for few channels
  int32_t NX, xB, CK, groups; // reduction groups: KH rows x NX steps of xB bytes x CK groups of 32
  int32_t off_x;              // staged columns before the padding's first (aligned form: quads of the image row)
  int32_t aligned;            // NCHW: every quad lies inside the image row or outside it
  uint32_t inv_hv, inv_oh, inv_tw, inv_nseg, inv_unit1, inv_unit2, inv_wper, inv_line, inv_bpp, inv_c16;  // floor(2^32 / d)
  int32_t per_channel, acc_wrap_shift, out_mode;
  uint32_t act_xor4, pad4;
  int32_t corr_coef;
  int32_t through;            // 16 bytes of results, from a multiple of as many pixels (channel-last: channels) on, lie in one image (or row, pixel) and at 16 bytes
  int64_t act_bytes;
  RequantScalars rs;
};

// Kinds of results, each with kernels of its own (conv_direct_kernel.h).
enum { kSums, kFullCodes, kAnyCodes };

// wt as the kernel's WT.  Each kind is compiled in a file of its own (conv_direct.hip, conv_direct_any.hip and conv_direct_sums.hip): a process that calls one
// loads a file's kernels, 26, and in one file with all others they were 78 (the first call of a process 3.5 ms, 1.8 so).
template <int OUT>
hipError_t launch_conv_direct(const CdParams& p, bool nhwc, int wt, int shape, size_t lds, int64_t grid, hipStream_t st);

}  // namespace hago
