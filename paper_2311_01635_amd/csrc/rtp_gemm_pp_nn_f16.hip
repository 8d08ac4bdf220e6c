// Instantiation of the ping-pong GEMM for fp16 inputs, NN operand layout (see rtp_gemm_pp.h).
#include "rtp_gemm_pp.h"

namespace rtp {
hipError_t launch_gemm_pp_nn_f16(const PpGroup &g, hipStream_t s, hipEvent_t done)
{
    return launch_gemm_pp_layout<LAY_NN, _Float16>(g, s, done);
}
} // namespace rtp
