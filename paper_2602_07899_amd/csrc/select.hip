// Gradient-guided token selection (Sec. 3.1.2): the per-position gradient
// statistic sum_n = sum_b ||g_{b,n}||, the Top-K position set I, and (in
// stats.hip) the channel maximum over the selected positions.  Small,
// HBM-bound kernels; all reductions run in double in a fixed order.
#include "common.h"

namespace tlq {

// One wave per gradient row: mean_c |g| (the reading of the text) or the Euclidean norm.  VEC: 16-byte
// loads (c % 8 == 0, 16-byte aligned rows of 256 channels and more), four in flight; HBM-bound, 128 x 1200 rows of 5120 channels
// 805 -> 267 us against 2-byte loads, 235 past the caches (NT, 6.7 TB/s).
template <typename T, bool VEC, bool NT>
__global__ __launch_bounds__(256) void row_norm_kernel(const uint16_t* __restrict__ G, int64_t rows, int64_t c,
                                                       int64_t ldg, int l2, double* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  double acc = 0.0;
  if constexpr (VEC) {
    const uint16_t* g = G + row * ldg;
#pragma unroll 4
    for (int64_t j = lane * 8; j < c; j += 512) {
      const uint4 v = load16<NT>(g + j);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const double x = (double)T::to_float((uint16_t)((w[e >> 1] >> ((e & 1) * 16)) & 0x7fffu));
        acc += l2 ? x * x : x;
      }
    }
  } else {
    for (int64_t j = lane; j < c; j += 64) {
      const double v = (double)T::to_float(G[row * ldg + j]);
      acc += l2 ? v * v : fabs(v);
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (lane == 0) out[row] = l2 ? sqrt(acc) : acc / (double)c;
}

// Sum over the samples in sample order.  STAGED: 64 positions per block; 16 waves bring 128 samples at a time into
// LDS, one adds them (one thread per position that walked its loads alone: 48 us for 128 x 1200).  Otherwise a
// thread per position, for samples that are few enough to be loaded together and for positions that are enough
// threads (2 samples x 262,144 positions: 11 us staged, 5 this way; 8 x 65,536: 4.7 both).
constexpr int kPosWaves = 16, kPosBatch = 128, kPosFew = 8, kPosMany = 131072;
template <bool STAGED>
__global__ __launch_bounds__(STAGED ? kPosWaves * 64 : 256) void position_sum_kernel(const double* __restrict__ row_norm,
                                                                                     int64_t n_samples, int64_t n_pos,
                                                                                     double* __restrict__ sum_n) {
  if constexpr (!STAGED) {
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= n_pos) return;
    double s = 0.0;
#pragma unroll 8
    for (int64_t b = 0; b < n_samples; ++b) s += row_norm[b * n_pos + n];
    sum_n[n] = s;
  } else {
    __shared__ double part[kPosBatch][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t n = (int64_t)blockIdx.x * 64 + lane;
    double s = 0.0;
    for (int64_t b0 = 0; b0 < n_samples; b0 += kPosBatch) {
#pragma unroll
      for (int i = 0; i < kPosBatch / kPosWaves; ++i) {
        const int64_t b = b0 + wave + i * kPosWaves;
        part[wave + i * kPosWaves][lane] = (n < n_pos && b < n_samples) ? row_norm[b * n_pos + n] : 0.0;
      }
      __syncthreads();
      if (wave == 0) {
        const int m = n_samples - b0 < kPosBatch ? (int)(n_samples - b0) : kPosBatch;
#pragma unroll 8
        for (int i = 0; i < m; ++i) s += part[i][lane];
      }
      __syncthreads();
    }
    if (wave == 0 && n < n_pos) sum_n[n] = s;
  }
}

hipError_t launch_token_importance(const void* G, int64_t n_samples, int64_t n_pos, int64_t c, int64_t ldg,
                                   bool bf16, bool l2, double* row_norm, double* sum_n, hipStream_t stream) {
  ProfScope ps("token_importance", stream, 2.0 * (double)n_samples * (double)n_pos * (double)c);
  const int64_t rows = n_samples * n_pos;
  const unsigned grid = (unsigned)ceil_div(rows, 4);
  // (below 256 channels most lanes of the wide form have nothing to do and the others add eight values in a
  // row: 524,288 rows of 8 channels 76 us element-wise, 122 wide; of 128 98 and 130; of 256 155 and 138)
  const bool vec = c >= 256 && (c % 8) == 0 && (ldg % 8) == 0 && ((uintptr_t)G % 16) == 0;
  auto go = [&](auto kern) { kern<<<grid, 256, 0, stream>>>((const uint16_t*)G, rows, c, ldg, l2 ? 1 : 0, row_norm); };
  const bool nt = streams_past(2.0 * (double)rows * (double)c);
  auto pick = [&](auto t) {
    using T = decltype(t);
    if (!vec) go(row_norm_kernel<T, false, false>);
    else if (nt) go(row_norm_kernel<T, true, true>);
    else go(row_norm_kernel<T, true, false>);
  };
  bf16 ? pick(BF16{}) : pick(F16{});
  if (n_samples < kPosFew || n_pos >= kPosMany)
    position_sum_kernel<false><<<(unsigned)ceil_div(n_pos, 256), 256, 0, stream>>>(row_norm, n_samples, n_pos, sum_n);
  else
    position_sum_kernel<true><<<(unsigned)ceil_div(n_pos, 64), kPosWaves * 64, 0, stream>>>(row_norm, n_samples, n_pos,
                                                                                           sum_n);
  return hipGetLastError();
}

// I = Top_k: position i is selected when fewer than k positions rank ahead of it
// (larger value, or equal value and lower index).  Rank by counting: O(n_pos^2), n_pos is
// a sequence length.  A block ranks 64 positions, its 16 waves count over a sixteenth of the rivals each
// (a thread that walked all 1200 rivals alone took 88 us).
constexpr int kTopWaves = 16;
__global__ __launch_bounds__(kTopWaves * 64) void topk_mask_kernel(const double* __restrict__ sum_n, int64_t n_pos,
                                                                   int64_t k, uint8_t* __restrict__ mask) {
  __shared__ int red[kTopWaves][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  const double v = i < n_pos ? sum_n[i] : 0.0;
  const int64_t per = (n_pos + kTopWaves - 1) / kTopWaves;
  const int64_t j1 = (wave + 1) * per < n_pos ? (wave + 1) * per : n_pos;
  int ahead = 0;                               // n_pos <= 65536
#pragma unroll 8
  for (int64_t j = wave * per; j < j1; ++j) {
    const double u = sum_n[j];
    ahead += (u > v || (u == v && j < i)) ? 1 : 0;
  }
  red[wave][lane] = ahead;
  __syncthreads();
  if (wave != 0 || i >= n_pos) return;
#pragma unroll
  for (int w = 1; w < kTopWaves; ++w) ahead += red[w][lane];
  mask[i] = ahead < k ? 1 : 0;
}

hipError_t launch_topk_mask(const double* sum_n, int64_t n_pos, int64_t k, uint8_t* mask, hipStream_t stream) {
  ProfScope ps("topk_mask", stream, 8.0 * (double)n_pos);
  topk_mask_kernel<<<(unsigned)ceil_div(n_pos, 64), kTopWaves * 64, 0, stream>>>(sum_n, n_pos, k, mask);
  return hipGetLastError();
}

}  // namespace tlq
