// What the one-launch 3x3 convolution's plan (conv3x3.hip) and its kernels (conv3x3_kernel.h) share.
#pragma once

#include "hago_device.h"
#include "launch.h"

namespace hago {

struct C3Params {
  const uint8_t* act;
  const int8_t* wgt;
  const int32_t* bias;
  void* out;
  const int32_t* mult;
  const int32_t* shift;
  int32_t B, C, H, W, O;
  int32_t TR;            // output rows per tile
  int32_t tiles_per_img; // ceil(H / TR)
  int32_t ntiles;        // B * tiles_per_img
  int32_t nblk;          // blocks of 32 TN output channels
  int32_t per_channel, acc_wrap_shift;
  int32_t out_mode;      // 0: requantized 8-bit, 1: raw int32, 2: raw int16
  int32_t through;       // results go through the L2
  uint32_t act_xor4;     // 0x80808080 for uint8 activations
  uint32_t pad4;         // staged value of a pixel outside the image, in every byte
  int32_t corr_coef;     // off - z_a
  uint32_t inv_tpi, inv_nblk, inv_run4, inv_w4, inv_w;  // ceil(2^32 / d) of tiles_per_img, nblk, the dwords of a run and of a row, W
  RequantScalars rs;
};

// Kinds of results, each with kernels of its own (conv3x3_kernel.h).
enum { kFull, kClipped, kWords, kHalves };

// nw, af, nu, tn as the kernel's NW, AF, NU and TN.  Each kind is compiled in a file of its own (conv3x3.hip, conv3x3_clipped.hip and so on): a process that calls one
// loads a file's kernels, 72, and in one file with all others they were 288 (the first call of a process 9.9 ms, 3.2 so).
template <int OUT>
hipError_t launch_conv3x3(const C3Params& p, int nw, int af, int nu, int tn, size_t lds, int64_t grid, hipStream_t st);

}  // namespace hago
