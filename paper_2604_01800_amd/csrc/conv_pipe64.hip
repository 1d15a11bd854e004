// The pipelined 3x3 convolution, 64 output channels per workgroup.
#include "conv_pipe.hpp"

namespace ppe {

void convp_launch64(const ConvpLaunch& L, hipStream_t s) { convp_launch<64, 32>(L, s); }

}  // namespace ppe
