// Codes of other clips and zero points, of small and middling tiles and of implicit convolutions.
#include "qgemm_common.h"

namespace hago {
namespace {
constexpr int kOut = kOutClipped;
}  // namespace
}  // namespace hago

#include "qgemm_dma_kernel.h"
