// Instantiation of the ping-pong GEMM for bf16 inputs, TN operand layout (see rtp_gemm_pp.h).
#include "rtp_gemm_pp.h"

namespace rtp {
hipError_t launch_gemm_pp_tn_bf16(const PpGroup &g, hipStream_t s, hipEvent_t done)
{
    return launch_gemm_pp_layout<LAY_TN, __bf16>(g, s, done);
}
} // namespace rtp
