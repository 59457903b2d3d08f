// Codes clipped to their container's whole range, of large dense tiles.
#include "qgemm_common.h"

namespace hago {
namespace {
constexpr int kOut = kOutFull;
}  // namespace
}  // namespace hago

#include "qgemm_line_kernel.h"
