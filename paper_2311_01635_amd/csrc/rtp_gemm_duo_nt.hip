// Instantiation of the GEMM of two workgroups a compute unit for bf16 inputs, NT operand layout (see rtp_gemm_duo.h).
#include "rtp_gemm_duo.h"

namespace rtp {
hipError_t launch_gemm_duo_nt_bf16(const PpGroup &g, hipStream_t s) { return launch_gemm_duo_layout<LAY_NT, __bf16>(g, s); }
} // namespace rtp
