// The 16-bit GEMM for fp16 operands.
#include "gemm16.h"

namespace fd {

hipError_t gemm_mfma_f16(const GemmArgs& g, hipStream_t s) { return dispatch_epi<_Float16>(g, s); }

}  // namespace fd
