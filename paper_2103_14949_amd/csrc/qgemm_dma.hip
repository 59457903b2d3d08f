// Which streaming kernel a dense layer or an implicit convolution takes, by its results and tile; and the kernels for codes clipped to their container's
// whole range, of small and middling tiles and of implicit convolutions (the other kinds': qgemm_dma_clipped.hip and qgemm_dma_other.hip).
#include "qgemm_common.h"

namespace hago {
namespace {
constexpr int kOut = kOutFull;
}  // namespace
}  // namespace hago

#include "qgemm_dma_kernel.h"

namespace hago {

hipError_t launch_qdense_dma(const QgemmParams& p, int shape, hipStream_t st) {
  const int out = qgemm_out(p);
  const bool line = shape != 2 && shape != 3 && shape != 4 && shape != 6;  // (192 x 256, 128 x 256 and 256 x 256)
  if (out == kOutFull) return line ? qdense_line<kOutFull>(p, shape, st) : qdense_dma<kOutFull>(p, shape, st);
  if (out == kOutClipped) return line ? qdense_line<kOutClipped>(p, shape, st) : qdense_dma<kOutClipped>(p, shape, st);
  return line ? qdense_line<kOutOther>(p, shape, st) : qdense_dma<kOutOther>(p, shape, st);
}

hipError_t launch_qconv_dma_direct(const QgemmParams& p, int shape, hipStream_t st) {
  const int out = qgemm_out(p);
  return out == kOutFull ? qconv_dma_direct<kOutFull>(p, shape, st) : out == kOutClipped ? qconv_dma_direct<kOutClipped>(p, shape, st)
                                                                                        : qconv_dma_direct<kOutOther>(p, shape, st);
}

hipError_t launch_qconv_dma(const QgemmParams& p, bool nchw_out, hipStream_t st) {
  const int out = nchw_out ? kOutOther : qgemm_out(p);
  return out == kOutFull ? qconv_dma<kOutFull>(p, nchw_out, st) : out == kOutClipped ? qconv_dma<kOutClipped>(p, nchw_out, st)
                                                                                 : qconv_dma<kOutOther>(p, nchw_out, st);
}

}  // namespace hago
