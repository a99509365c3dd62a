// The 16-bit GEMM for bf16 operands.
#include "gemm16.h"

namespace fd {

hipError_t gemm_mfma_bf16(const GemmArgs& g, hipStream_t s) { return dispatch_epi<__hip_bfloat16>(g, s); }

}  // namespace fd
