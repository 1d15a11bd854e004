// The pipelined 3x3 convolution, 32 output channels per workgroup and 16-row tiles.
#include "conv_pipe.hpp"

namespace ppe {

void convp_launch16(const ConvpLaunch& L, hipStream_t s) { convp_launch<32, 16>(L, s); }

}  // namespace ppe
