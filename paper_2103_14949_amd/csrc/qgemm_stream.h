// Pieces shared by the GEMM kernels whose operands stream from global memory straight into LDS (qgemm_dma.hip,
// qgemm_line.hip): the DMA instruction, its descriptors, the LDS layout and the numbering of the tiles.
#pragma once

#include "qgemm_common.h"
#include "stream_offset.h"

#include <type_traits>
#include <utility>

namespace hago {

// Chunk permutation of an LDS row of BK bytes.  With these a fragment read (lane -> row lane % 32,
// chunk 2 h + lane / 32 for 32-k group h) runs at the full LDS rate (measured; other XOR patterns
// of the row bits run at half rate or less).  It depends on the row inside a 16-row block only.
template <int BK>
__device__ __forceinline__ int swz(int row) {
  return BK == 64 ? (row >> 2) & 3 : (row >> 1) & 7;
}

__device__ __forceinline__ void dma16(v4i rsrc, uint32_t lds_addr, uint32_t voff) {
  // m0 = LDS byte address of the wavefront's 1 KB window; lane l lands at m0 + 16 * l.  A write of m0 and an LDS load
  // need a wait state between them, which the compiler does not see to inside inline assembly (the four encoder layers of
  // 4096 rows take 55.5 us with it, 55.6 without).
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :
               : "s"(lds_addr), "v"(voff), "s"(rsrc)
               : "memory", "m0");
}

// Same with a scalar byte offset added to every lane's address.  The range check does not see it: what is not to be fetched
// needs a lane offset beyond the tensor.
__device__ __forceinline__ void dma16s(v4i rsrc, uint32_t lds_addr, uint32_t voff, uint32_t soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :
               : "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff)
               : "memory", "m0");
}

__device__ __forceinline__ v4i make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  v4i r;
  r.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r.y = __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));  // stride 0, no swizzle
  r.z = __builtin_amdgcn_readfirstlane((int)bytes);
  r.w = 0x00020000;  // raw buffer, 32-bit data format
  return r;
}

// The descriptor of a tensor that is loaded in runs (stream_offset.h).
__device__ __forceinline__ v4i make_run_rsrc(const uint8_t* base, uint32_t bytes) { return make_rsrc(base - kRunBack, bytes + kRunBack); }

template <int N>
using template_int = std::integral_constant<int, N>;

// Tiles are numbered panel by panel (kPanel tiles wide along P, all of Q), row by row inside
// a panel: the tiles that run on an XCD at the same time then form a compact block and share
// both operands' rows in its L2.
__device__ __forceinline__ void panel_tile(int tile, int tiles_p, int tiles_q, int& tile_p, int& tile_q) {
  constexpr int kPanel = 8;
  const int full = tiles_p / kPanel;
  const int per_panel = kPanel * tiles_q;
  int r = tile, w = kPanel, base = 0;
  if (tile >= full * per_panel) {
    r = tile - full * per_panel;
    w = tiles_p - full * kPanel;
    base = full * kPanel;
  } else {
    const int pn = tile / per_panel;
    r = tile - pn * per_panel;
    base = pn * kPanel;
  }
  tile_q = r / w;
  tile_p = base + (r - tile_q * w);
}

}  // namespace hago
