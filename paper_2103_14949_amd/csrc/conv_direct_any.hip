// Codes of any other clip, accumulator or tie rule of the any-geometry convolution in one launch.
#include "conv_direct_kernel.h"

namespace hago {

template hipError_t launch_conv_direct<kAnyCodes>(const CdParams&, bool, int, int, size_t, int64_t, hipStream_t);

}  // namespace hago
