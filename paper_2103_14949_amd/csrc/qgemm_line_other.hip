// Sums, and codes of narrow accumulators or of the other tie rule, of large dense tiles.
#include "qgemm_common.h"

namespace hago {
namespace {
constexpr int kOut = kOutOther;
}  // namespace
}  // namespace hago

#include "qgemm_line_kernel.h"
