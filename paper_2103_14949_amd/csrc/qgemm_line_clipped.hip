// Codes of other clips and zero points, of large dense tiles.
#include "qgemm_common.h"

namespace hago {
namespace {
constexpr int kOut = kOutClipped;
}  // namespace
}  // namespace hago

#include "qgemm_line_kernel.h"
