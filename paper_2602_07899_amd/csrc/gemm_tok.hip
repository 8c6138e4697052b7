// Losses with per-token errors in tiles of 128 x 128, where tiles of 256 rows would leave most CUs idle (gemm_small_tiles says
// where).  Bound by the chain of k-tiles of a block: 0.4 us each, against 1.1 of a 256 x 256 tile.  Weights quantised, then
// the loss with errors, us 256 rows -> 128, tokens x channels x outputs: 142 x 256 x 5685 30 -> 24, 493 x 11648 x 337 242 ->
// 111, 763 x 7936 x 3366 198 -> 108, 1781 x 2944 x 2810 114 -> 80, 3190 x 7424 x 983 172 -> 87.
#include "contraction.h"

namespace tlq {

template <int NSTAGE, bool TAIL>
__global__ __launch_bounds__(256) void gemm_small_tok_kernel(GemmDev a) {
  gemm_dma_body<F16, NSTAGE, EPI_LOSS_TOK, false, TAIL, 1, 4>(a);
}

hipError_t launch_dma_small_tok(const GemmDev& d, bool deep, unsigned blocks, hipStream_t stream) {
  const bool tail = d.c_in % kDmaBK != 0;
  if (deep) tail ? gemm_small_tok_kernel<4, true><<<blocks, 256, 0, stream>>>(d) : gemm_small_tok_kernel<4, false><<<blocks, 256, 0, stream>>>(d);
  else tail ? gemm_small_tok_kernel<2, true><<<blocks, 256, 0, stream>>>(d) : gemm_small_tok_kernel<2, false><<<blocks, 256, 0, stream>>>(d);
  return hipGetLastError();
}

}  // namespace tlq
