// MFMA GEMM kernels for one operand layout (see gemm_mfma_impl.h).
#include "gemm_mfma_impl.h"

namespace tmk {
TM_GEMM_INSTANTIATE(true, true, 0)
template __global__ void gemm_pipe_kernel<128, 128, GEMM_BK, 2, 2, true, true, 0, 2, 2, true>(const MfmaGemmParams);
int gemm_mfma_nt(const GemmArgs &g, int config, hipStream_t s) { return launch_layout<true, true, 0>(g, config, s); }
}  // namespace tmk
