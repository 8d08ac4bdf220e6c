// Instantiation of the ping-pong GEMM for fp16 inputs, NN and TN operand layouts in one launch (see rtp_gemm_pp.h).
#include "rtp_gemm_pp.h"

namespace rtp {
hipError_t launch_gemm_pp_nn_tn_f16(const PpGroup &g, hipStream_t s, hipEvent_t done)
{
    return launch_gemm_pp_layout<LAY_NN_TN, _Float16>(g, s, done);
}
} // namespace rtp
