// The contraction of activation codes with weight codes on int8 MFMA.
#include "contraction.h"

namespace tlq {

// Integer codes on both sides (per-token activation codes, per-row weight codes): twice the multiplications per
// MFMA cycle and per byte moved of the fp16 form of the same codes, exact sums, one rounding less (the dequantised
// weight's).  The rows of both operands are padded with zeros to whole k-tiles.  20 candidates of 3678 x 4096 x 4096,
// W4A8: contraction 2.1 -> 1.2 ms, the whole search 2.19 -> 1.31 ms; relative error of the losses against 64
// bits 5e-6 -> 3e-8.
template <int NSTAGE, int EPI, int HALVES, int JB>
__global__ __launch_bounds__(HALVES * 256) void gemm_i8_kernel(GemmDev a) {
  gemm_dma_body<Int8, NSTAGE, EPI, false, false, HALVES, JB>(a);
}

template <int EPI>
static hipError_t launch(const GemmDev& d, GemmTile tile, unsigned blocks, hipStream_t stream) {
  if (!tile.small && tile.tok_blocks == 3) gemm_i8_kernel<2, EPI, 2, 3><<<blocks, 512, 0, stream>>>(d);
  else if (!tile.small && tile.tok_blocks == 5) gemm_i8_kernel<2, EPI, 2, 5><<<blocks, 512, 0, stream>>>(d);
  else if (!tile.small) gemm_i8_kernel<2, EPI, 2, 4><<<blocks, 512, 0, stream>>>(d);
  else if ((int64_t)d.tiles_o * d.tiles_t * d.n_cand <= 256) gemm_i8_kernel<4, EPI, 1, 4><<<blocks, 256, 0, stream>>>(d);
  else gemm_i8_kernel<2, EPI, 1, 4><<<blocks, 256, 0, stream>>>(d);
  return hipGetLastError();
}

hipError_t launch_dma_i8(const GemmDev& d, int epi, GemmTile tile, unsigned blocks, hipStream_t stream) {
  if (epi == EPI_LOSS) return launch<EPI_LOSS>(d, tile, blocks, stream);
  return epi == EPI_STORE ? launch<EPI_STORE>(d, tile, blocks, stream) : hipErrorInvalidValue;
}

}  // namespace tlq
