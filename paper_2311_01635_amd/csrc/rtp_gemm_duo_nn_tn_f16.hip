// Instantiation of the GEMM of two workgroups a compute unit for fp16 inputs, NN and TN problems (see rtp_gemm_duo.h).
#include "rtp_gemm_duo.h"

namespace rtp {
hipError_t launch_gemm_duo_nn_tn_f16(const PpGroup &g, hipStream_t s) { return launch_gemm_duo_layout<LAY_NN_TN, _Float16>(g, s); }
} // namespace rtp
