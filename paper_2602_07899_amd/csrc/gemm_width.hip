// Tiles of 256 output rows x 192 and x 320 tokens (see gemm_tile for what they are for).
#include "contraction.h"

namespace tlq {

// 256 output rows x 64 JB tokens, JB = 3 or 5
template <typename T, int EPI, bool SYMK, bool TAIL, int JB>
__global__ __launch_bounds__(512) void gemm_width_kernel(GemmDev a) {
  gemm_dma_body<T, 2, EPI, SYMK, TAIL, 2, JB>(a);
}

template <typename T, int EPI, int JB>
static hipError_t launch(const GemmDev& d, unsigned blocks, hipStream_t stream) {
  constexpr bool SYMK = EPI == EPI_DOT;
  if (d.c_in % kDmaBK == 0) gemm_width_kernel<T, EPI, SYMK, false, JB><<<blocks, 512, 0, stream>>>(d);
  else gemm_width_kernel<T, EPI, SYMK, true, JB><<<blocks, 512, 0, stream>>>(d);
  return hipGetLastError();
}

hipError_t launch_dma_width(const GemmDev& d, int epi, bool bf16, int tok_blocks, unsigned blocks, hipStream_t stream) {
  if (epi == EPI_STORE && tok_blocks == 3) return bf16 ? launch<BF16, EPI_STORE, 3>(d, blocks, stream) : launch<F16, EPI_STORE, 3>(d, blocks, stream);
  if (epi == EPI_STORE) return bf16 ? launch<BF16, EPI_STORE, 5>(d, blocks, stream) : launch<F16, EPI_STORE, 5>(d, blocks, stream);
  if (bf16) return hipErrorInvalidValue;
  if (epi == EPI_LOSS) return tok_blocks == 3 ? launch<F16, EPI_LOSS, 3>(d, blocks, stream) : launch<F16, EPI_LOSS, 5>(d, blocks, stream);
  if (tok_blocks == 3) return hipErrorInvalidValue;
  return epi == EPI_LOSS_TOK ? launch<F16, EPI_LOSS_TOK, 5>(d, blocks, stream) : launch<F16, EPI_DOT, 5>(d, blocks, stream);
}

}  // namespace tlq
