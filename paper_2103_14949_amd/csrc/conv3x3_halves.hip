// 16-bit sums of the one-launch 3x3 convolution.
#include "conv3x3_kernel.h"

namespace hago {

template hipError_t launch_conv3x3<kHalves>(const C3Params&, int, int, int, int, size_t, int64_t, hipStream_t);

}  // namespace hago
