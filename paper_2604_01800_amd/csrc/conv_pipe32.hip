// The pipelined 3x3 convolution, 32 output channels per workgroup.
#include "conv_pipe.hpp"

namespace ppe {

void convp_launch32(const ConvpLaunch& L, hipStream_t s) { convp_launch<32, 32>(L, s); }

}  // namespace ppe
