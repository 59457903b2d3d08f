// Codes of any other clip, accumulator or tie rule of the one-launch 3x3 convolution.
#include "conv3x3_kernel.h"

namespace hago {

template hipError_t launch_conv3x3<kClipped>(const C3Params&, int, int, int, int, size_t, int64_t, hipStream_t);

}  // namespace hago
