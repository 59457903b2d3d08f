// Sums, and codes of narrow accumulators or of the other tie rule, of small and middling tiles and of implicit convolutions.
#include "qgemm_common.h"

namespace hago {
namespace {
constexpr int kOut = kOutOther;
}  // namespace
}  // namespace hago

#include "qgemm_dma_kernel.h"
