// Tiles of 128 output rows x 64 tokens, one a CU: for launches whose 128 x 128 tiles would leave half of the CUs idle.  Such a
// launch is one chain of k-tiles (64 channels) in every block, with one wave a SIMD; what bounds a k-tile is the LDS reads of
// its fragments (48 KB instead of 64, at 128 bytes a cycle) and the waits between its two phases, 0.27 us instead of 0.40.
// Stores, us, tiles of 128 x 128 -> these, tokens x channels x outputs: 128 x 64 x 1024 4.8 -> 4.0, 512 x 1000 x 1024
// 11.0 -> 8.3, 216 x 512 x 256 9.5 -> 6.6, 64 x 2048 x 8192 19.6 -> 13.1, 512 x 8192 x 512 56.5 -> 39.0, at 256 tiles
// 1000 x 2048 x 2000 20.5 -> 15.0.  Just beyond, a second round: 288 tiles of 1100 x 1000 x 2000
// 13.8 with 128 x 128, 18.4 with these.
#include "contraction.h"

namespace tlq {

template <typename T, int EPI, bool TAIL>
__global__ __launch_bounds__(256) void gemm_half_kernel(GemmDev a) {
  gemm_dma_body<T, 4, EPI, false, TAIL, 1, 2>(a);
}

template <typename T, int EPI>
static hipError_t launch(const GemmDev& d, unsigned blocks, hipStream_t stream) {
  if (d.c_in % kDmaBK == 0) gemm_half_kernel<T, EPI, false><<<blocks, 256, 0, stream>>>(d);
  else gemm_half_kernel<T, EPI, true><<<blocks, 256, 0, stream>>>(d);
  return hipGetLastError();
}

hipError_t launch_dma_half(const GemmDev& d, int epi, bool bf16, unsigned blocks, hipStream_t stream) {
  if (epi == EPI_STORE) return bf16 ? launch<BF16, EPI_STORE>(d, blocks, stream) : launch<F16, EPI_STORE>(d, blocks, stream);
  if (bf16 || epi == EPI_DOT) return hipErrorInvalidValue;
  return epi == EPI_LOSS ? launch<F16, EPI_LOSS>(d, blocks, stream) : launch<F16, EPI_LOSS_TOK>(d, blocks, stream);
}

}  // namespace tlq
