// Entry of the 16-bit GEMM: argument checks, then the operand type's kernels.
#include "fd_kernels.h"

namespace fd {

constexpr int BKD = 32;  // K-columns per stage

hipError_t gemm_mfma(Act16 t, const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (g.K <= 0 || g.K % BKD || !g.a_packed || g.lda != g.K || g.ldw != g.K) return hipErrorInvalidValue;
  if (g.ep.out_packed &&
      (g.ep.ld_out % 32 || !(g.epi == EPI_SWIGLU || g.epi == EPI_STORE_SILU || g.epi == EPI_STORE_GELU)))
    return hipErrorInvalidValue;
  if ((g.epi == EPI_SWIGLU || g.epi == EPI_QKV) && g.N % 64) return hipErrorInvalidValue;
  if (g.epi == EPI_QKV && g.ep.qkv.Dh != 64) return hipErrorInvalidValue;
  return t == Act16::F16 ? gemm_mfma_f16(g, s) : gemm_mfma_bf16(g, s);
}

}  // namespace fd
