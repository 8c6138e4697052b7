// S0 (x_stat), S1 (scale table), the final loss combine and S5 (selection).
// All HBM-bound or tiny; none uses floating-point atomics, so results are
// bit-identical from run to run.
#include <type_traits>

#include "common.h"

namespace tlq {

// ---------------------------------------------------------------- S0 x_stat
// Sec. 3.1.2 x_stat (mean variant of the ablation table, or max over all
// tokens).  Each lane owns 8 consecutive channels (one 16-byte load per row);
// the waves of a block walk interleaved rows of the block's row chunk and
// are combined through LDS; chunks are combined by a second kernel.  Sums are
// carried in double, in an order that the shape fixes, so a result is
// reproducible.  |fp16| values are multiples of 2^-24: a channel's sum is exact
// in any order while it stays below 2^29; beyond that, and for bf16 channels of
// wide range, the order shows in the last bits of the double.
constexpr int kXsCols = 64 * 8;  // channels per block
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t wave_max(uint32_t m) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const uint32_t o = __shfl_xor(m, off, 64);
    m = m > o ? m : o;
  }
  return m;
}

int xstat_chunks(int64_t n_tok) {
  int64_t c = ceil_div(n_tok, 128);
  return (int)(c < 1 ? 1 : (c > 128 ? 128 : c));
}

// NW waves per block: 16 where a chunk has 128 rows at most (8 a wave; with 4 waves the two blocks of a
// 256 x 512 input walked 32 rows each wave, 11 us against 4) and where few channels make few blocks, whose 4 waves with a
// row each in flight leave memory idle: up to 2048 channels, and without a mask up to 5120 on chunks of more than 256 rows (us, 4
// waves -> 16 with four rows each in flight: 24,000 x 312 13.6 -> 9.8, 64,699 x 640 46.6 -> 19.2, 153,600 x 1024 154 -> 52,
// 44,166 x 1536 38 -> 24, 17,000 x 2048 18.8 -> 15.1, 60,000 x 4096 91 -> 79, 33,000 x 5120 62 -> 56, 153,600 x 5120 244 -> 241).
// Elsewhere 4, with as many blocks as it takes (4 and 16: 20,000 x 4096 27.4 and 28.4, masked 153,600 x 5120 129 and 132; 44,000 x
// 5632 78.8 and 82.6, 60,000 x 6144 112.8 and 117.9, 100,000 x 7168 212 and 224, 153,600 x 5632 264 and 269, x 6144 276 and 290, x
// 8192 380 and 390).  The line misses that 16 are ahead again from 10,240 channels on (60,000 x 10,240 215 and 197, 44,000 x
// 13,824 220 and 204) and up to 33,000 rows (x 8192 110 and 94).
// The order of a channel's sums follows the number of waves; where it shows see above.
// NT: rows that come past the caches (153,600 x 5120: 265 -> 244 us, 6.4 TB/s).
// MAXBITS: every block also leaves the largest magnitude (as bits) that it has seen in block_max, for the fp16
// re-expression of bf16 tokens, which would read them all once more for it.
// U: rows of a wave that are loaded together (the masked form takes four).
template <typename T, int KIND, bool MASKED, int NW, bool MAXBITS, bool NT, int U>
__global__ __launch_bounds__(NW * 64) void xstat_partial_kernel(
    const uint16_t* __restrict__ X, int64_t n_tok, int64_t c_in, int64_t ldx, int rows_per_chunk,
    double* __restrict__ partial, const uint8_t* __restrict__ pos_mask, int64_t period, uint32_t* __restrict__ block_max) {
  __shared__ double red[NW][kXsCols];
  __shared__ uint32_t redm[NW];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t c0 = (int64_t)blockIdx.x * kXsCols + lane * 8;
  const int64_t r0 = (int64_t)blockIdx.y * rows_per_chunk;
  int64_t r1 = r0 + rows_per_chunk;
  if (r1 > n_tok) r1 = n_tok;
  double acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = 0.0;
  u16x2 top = {0, 0};
  auto add = [&](const uint4& v) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    if constexpr (MAXBITS) {
#pragma unroll
      for (int j = 0; j < 4; ++j) top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, w[j] & 0x7fff7fffu));
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint16_t b = (uint16_t)((w[j >> 1] >> ((j & 1) * 16)) & 0x7fffu);  // |x|
      const double a = (double)T::to_float(b);
      if (KIND == 0) acc[j] += a; else acc[j] = a > acc[j] ? a : acc[j];
    }
  };
  if (MASKED || c0 < c_in) {
    if constexpr (!MASKED) {
      int64_t r = r0 + wave;
      for (; r + (U - 1) * NW < r1; r += U * NW) {
        uint4 v[U];
#pragma unroll
        for (int i = 0; i < U; ++i) v[i] = load16<NT>(X + (r + i * NW) * ldx + c0);
#pragma unroll
        for (int i = 0; i < U; ++i) add(v[i]);
      }
      if constexpr (U > 1)
        for (; r < r1; r += NW) add(load16<NT>(X + r * ldx + c0));
    } else {
      const int64_t cr = c0 < c_in ? c0 : 0;     // (every lane takes part in the look-up)
      // rows that are not selected are not read: the lanes look 64 of the wave's rows up at once, the set
      // bits are then walked four loads at a time (a mask load and a division per row kept the loads apart)
      for (int64_t rb = r0 + wave; rb < r1; rb += NW * 64) {
        const int64_t row = rb + NW * (int64_t)lane;
        uint64_t sel = __builtin_amdgcn_ballot_w64(row < r1 && pos_mask[row % period] != 0);
        while (sel) {
          uint4 v[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            v[i] = make_uint4(0, 0, 0, 0);       // a zero changes neither the sum nor the maximum
            if (sel) {
              v[i] = load16<NT>(X + (rb + NW * (int64_t)__builtin_ctzll(sel)) * ldx + cr);
              sel &= sel - 1;
            }
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) add(v[i]);
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) red[wave][lane * 8 + j] = acc[j];
  if constexpr (MAXBITS) {
    const uint32_t m = wave_max(top[0] > top[1] ? top[0] : top[1]);
    if (lane == 0) redm[wave] = m;
  }
  __syncthreads();
  if (MAXBITS && threadIdx.x == 0) {
    uint32_t m = redm[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) m = m > redm[w] ? m : redm[w];
    block_max[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = m;
  }
  for (int i = threadIdx.x; i < kXsCols; i += NW * 64) {
    const int64_t c = (int64_t)blockIdx.x * kXsCols + i;
    if (c < c_in) {
      double s = red[0][i];
#pragma unroll
      for (int w = 1; w < NW; ++w) s = KIND == 0 ? s + red[w][i] : fmax(s, red[w][i]);
      partial[(int64_t)blockIdx.y * c_in + c] = s;
    }
  }
}

// 64 channels per block, the chunks in 16 contiguous stretches (one a wave) that are combined in order: one
// thread per channel walked 128 dependent loads (32 us at 5120 channels; 5 us this way).  Wave 0 returns the
// statistic of its lane's channel.
constexpr int kXfWaves = 16;
template <int KIND>
__device__ __forceinline__ float xstat_combine(const double* __restrict__ partial, int n_chunks, int64_t c_in,
                                               int64_t n_tok, double (&red)[kXfWaves][64]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t c = (int64_t)blockIdx.x * 64 + lane;
  const int per = (n_chunks + kXfWaves - 1) / kXfWaves;
  const int i1 = (wave + 1) * per < n_chunks ? (wave + 1) * per : n_chunks;
  double s = 0.0;
  if (c < c_in) {
#pragma unroll 8
    for (int i = wave * per; i < i1; ++i) {
      const double v = partial[(int64_t)i * c_in + c];
      if (KIND == 0) s += v; else s = v > s ? v : s;
    }
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave != 0) return 0.0f;
#pragma unroll
  for (int i = 1; i < kXfWaves; ++i) {
    const double v = red[i][lane];
    if (KIND == 0) s += v; else s = v > s ? v : s;
  }
  return (float)(KIND == 0 ? s / (double)n_tok : s);
}

template <int KIND>
__global__ __launch_bounds__(kXfWaves * 64) void xstat_final_kernel(const double* __restrict__ partial, int n_chunks,
                                                                    int64_t c_in, int64_t n_tok,
                                                                    float* __restrict__ x_stat) {
  __shared__ double red[kXfWaves][64];
  const float xs = xstat_combine<KIND>(partial, n_chunks, c_in, n_tok, red);
  const int64_t c = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (threadIdx.x < 64 && c < c_in) x_stat[c] = xs;
}

// Partial sums of every chunk, and with block_max the largest magnitude of every block of the grid.
static hipError_t launch_xstat_partial(const void* X, int64_t n_tok, int64_t c_in, int64_t ldx, bool bf16, int kind,
                                       double* partial, hipStream_t stream, const uint8_t* pos_mask, int64_t period,
                                       uint32_t* block_max) {
  const int chunks = xstat_chunks(n_tok);
  const int rows = (int)ceil_div(n_tok, chunks);
  const dim3 grid((unsigned)ceil_div(c_in, kXsCols), (unsigned)chunks);
  const uint16_t* x = (const uint16_t*)X;
  ProfScope ps("xstat_partial", stream, 2.0 * (double)n_tok * (double)c_in);
  const bool wide = rows <= 128 || grid.x <= 4 || (!pos_mask && grid.x <= 10 && rows > 256);
  // Chunks of 128 rows at most: a row a wave at a time, but the mean of many chunks of many channels four (us, one -> four, mean: 6000 x 4096
  // 13.6 -> 13.1, 12,000 x 8192 43.4 -> 39.1, 16,384 x 8192 56.5 -> 50.5, but 6000 x 3072 11.1 -> 11.7, 12,000 x 2048 14.5 -> 15.4, 3000 x 8192
  // 13.9 -> 14.4; maximum: 3000 x 8192 14.1 -> 16.0, 6000 x 4096 13.7 -> 15.2, 16,384 x 5120 30.2 -> 32.9, but 6000 x 8192 27.0 -> 25.2)
  const bool shallow = rows <= 128 && (kind != 0 || chunks <= 32 || grid.x < 8);
  const bool nt = streams_past(2.0 * (double)n_tok * (double)c_in);
  auto go = [&](auto kern, int waves) {
    kern<<<grid, waves * 64, 0, stream>>>(x, n_tok, c_in, ldx, rows, partial, pos_mask, period, block_max);
  };
  auto pick = [&](auto t, auto kind_c, auto masked_c, auto max_c) {
    using T = decltype(t);
    constexpr int KIND = decltype(kind_c)::value;
    constexpr bool MASKED = decltype(masked_c)::value, MAXBITS = decltype(max_c)::value;
    constexpr int FOUR = MASKED ? 1 : 4;
    if (shallow) go(xstat_partial_kernel<T, KIND, MASKED, 16, MAXBITS, false, 1>, 16);
    else if (wide && nt) go(xstat_partial_kernel<T, KIND, MASKED, 16, MAXBITS, true, FOUR>, 16);
    else if (wide) go(xstat_partial_kernel<T, KIND, MASKED, 16, MAXBITS, false, FOUR>, 16);
    else if (nt) go(xstat_partial_kernel<T, KIND, MASKED, 4, MAXBITS, true, 1>, 4);
    else go(xstat_partial_kernel<T, KIND, MASKED, 4, MAXBITS, false, 1>, 4);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using Yes = std::true_type;
  using No = std::false_type;
  if (pos_mask) bf16 ? pick(BF16{}, I1{}, Yes{}, No{}) : pick(F16{}, I1{}, Yes{}, No{});   // (only the maximum has a masked form)
  else if (!bf16) kind == 0 ? pick(F16{}, I0{}, No{}, No{}) : pick(F16{}, I1{}, No{}, No{});
  else if (block_max) kind == 0 ? pick(BF16{}, I0{}, No{}, Yes{}) : pick(BF16{}, I1{}, No{}, Yes{});
  else kind == 0 ? pick(BF16{}, I0{}, No{}, No{}) : pick(BF16{}, I1{}, No{}, No{});
  return hipGetLastError();
}

template <typename T, int KIND>
__device__ __forceinline__ float xstat_direct(const uint16_t* __restrict__ X, int64_t n_tok, int64_t c_in, int64_t ldx,
                                              double (&red)[kXfWaves][64]);
template <typename T, int KIND>
__global__ __launch_bounds__(kXfWaves * 64) void xstat_direct_kernel(const uint16_t* __restrict__ X, int64_t n_tok, int64_t c_in,
                                                                     int64_t ldx, float* __restrict__ x_stat) {
  __shared__ double red[kXfWaves][64];
  const float xs = xstat_direct<T, KIND>(X, n_tok, c_in, ldx, red);
  const int64_t c = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (threadIdx.x < 64 && c < c_in) x_stat[c] = xs;
}

hipError_t launch_xstat(const void* X, int64_t n_tok, int64_t c_in, int64_t ldx, bool bf16,
                        int kind, double* partial, float* x_stat, hipStream_t stream,
                        const uint8_t* pos_mask, int64_t period) {
  if (!pos_mask && n_tok <= kDirectRows && c_in <= kDirectCols) {
    ProfScope ps("xstat_partial", stream, 2.0 * (double)n_tok * (double)c_in);
    auto go = [&](auto kern) {
      kern<<<(unsigned)ceil_div(c_in, 64), kXfWaves * 64, 0, stream>>>((const uint16_t*)X, n_tok, c_in, ldx, x_stat);
    };
    if (!bf16) kind == 0 ? go(xstat_direct_kernel<F16, 0>) : go(xstat_direct_kernel<F16, 1>);
    else kind == 0 ? go(xstat_direct_kernel<BF16, 0>) : go(xstat_direct_kernel<BF16, 1>);
    return hipGetLastError();
  }
  const hipError_t e = launch_xstat_partial(X, n_tok, c_in, ldx, bf16, kind, partial, stream, pos_mask, period, nullptr);
  if (e != hipSuccess) return e;
  const int chunks = xstat_chunks(n_tok);
  {
    ProfScope ps("xstat_final", stream, 8.0 * (double)chunks * (double)c_in);
    const unsigned g2 = (unsigned)ceil_div(c_in, 64);
    if (kind == 0) xstat_final_kernel<0><<<g2, kXfWaves * 64, 0, stream>>>(partial, chunks, c_in, n_tok, x_stat);
    else xstat_final_kernel<1><<<g2, kXfWaves * 64, 0, stream>>>(partial, chunks, c_in, n_tok, x_stat);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------ S1 scale table
// Sec. 3.1.2 scale equation: s = x_stat^alpha, evaluated in double and rounded
// once; the reciprocal table feeds the folded GEMM operand deq / s.
__device__ __forceinline__ double pow2(int k) { return (double)__builtin_bit_cast(float, (uint32_t)(127 + k) << 23); }
__device__ __forceinline__ double pow2_shift(const uint32_t* xmax_bits) {
  return pow2(xmax_bits ? shift_from_bf16_bits(*xmax_bits) : 0);
}

// one entry of the table; s_copy and inv_table may be NULL
__device__ __forceinline__ void table_entry(float xs, float alpha, double up, int64_t at, float* __restrict__ s_table,
                                            float* __restrict__ s_copy, float* __restrict__ inv_table) {
  xs = xs > kXstatFloor ? xs : kXstatFloor;  // also maps NaN to the floor
  const float s = (float)pow((double)xs, (double)alpha);
  s_table[at] = s;
  if (s_copy) s_copy[at] = s;
  if (inv_table) inv_table[at] = (float)(up / (double)s);
}

__global__ void scale_table_kernel(const float* __restrict__ x_stat, int64_t c_in,
                                   const float* __restrict__ alpha, int n_alpha,
                                   float* __restrict__ s_table, float* __restrict__ s_copy, float* __restrict__ inv_table,
                                   const uint32_t* __restrict__ xmax_bits) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int k = blockIdx.y;
  if (c >= c_in || k >= n_alpha) return;
  table_entry(x_stat[c], alpha[k], pow2_shift(xmax_bits), (int64_t)k * c_in + c, s_table, s_copy, inv_table);
}

hipError_t launch_scale_table(const float* x_stat, int64_t c_in, const float* alpha, int n_alpha,
                              float* s_table, float* s_copy, float* inv_table, const uint32_t* xmax_bits,
                              hipStream_t stream) {
  ProfScope ps("scale_table", stream, 8.0 * (double)n_alpha * (double)c_in);
  dim3 grid((unsigned)ceil_div(c_in, 256), (unsigned)n_alpha);
  scale_table_kernel<<<grid, 256, 0, stream>>>(x_stat, c_in, alpha, n_alpha, s_table, s_copy, inv_table, xmax_bits);
  return hipGetLastError();
}

// The statistic of 64 channels over all rows, straight from the tokens: eight lanes read the 128 bytes of a row, a wave
// eight rows at a time.  The value of its lane's channel arrives in wave 0.
template <typename T, int KIND>
__device__ __forceinline__ float xstat_direct(const uint16_t* __restrict__ X, int64_t n_tok, int64_t c_in, int64_t ldx,
                                              double (&red)[kXfWaves][64]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t c0 = (int64_t)blockIdx.x * 64 + (lane & 7) * 8;
  double acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = 0.0;
  if (c0 < c_in) {
#pragma unroll 4
    for (int64_t r = wave * 8 + (lane >> 3); r < n_tok; r += kXfWaves * 8) {
      const uint4 v = *reinterpret_cast<const uint4*>(X + r * ldx + c0);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const double a = (double)T::to_float((uint16_t)((w[j >> 1] >> ((j & 1) * 16)) & 0x7fffu));
        if (KIND == 0) acc[j] += a; else acc[j] = a > acc[j] ? a : acc[j];
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
#pragma unroll
    for (int off = 8; off <= 32; off <<= 1) {
      const double o = __shfl_xor(acc[j], off, 64);
      if (KIND == 0) acc[j] += o; else acc[j] = o > acc[j] ? o : acc[j];
    }
    if (lane < 8) red[wave][lane * 8 + j] = acc[j];
  }
  __syncthreads();
  if (wave != 0) return 0.0f;
  double s = red[0][lane];
#pragma unroll
  for (int i = 1; i < kXfWaves; ++i) {
    const double v = red[i][lane];
    if (KIND == 0) s += v; else s = v > s ? v : s;
  }
  return (float)(KIND == 0 ? s / (double)n_tok : s);
}

struct TableDev {
  const float* alpha; int n_alpha; int64_t c_in;
  float* s_table; float* s_copy; float* inv_table;
  const uint32_t* xmax_bits;                                   // sets the shift of the reciprocals unless block_max does
  const uint32_t* block_max; int n_max; uint32_t* xmax_out;
};

// xstat_final_kernel and scale_table_kernel in one launch for a search that computes its own statistic: wave 0
// hands the 64 channels' statistics to the 16 waves, which take the candidates in turn.  With block_max, the largest
// magnitude over its n_max words is taken first (by every block: it is part of the reciprocals) and stored in *xmax_out.
// Latency-bound: two launches of 3 - 5 us each became one of 5.
template <int KIND>
__global__ __launch_bounds__(kXfWaves * 64) void xstat_table_kernel(const double* __restrict__ partial, int n_chunks,
                                                                    int64_t n_tok, TableDev t) {
  __shared__ double red[kXfWaves][64];
  __shared__ float stat[64];
  __shared__ uint32_t redm[kXfWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (t.block_max) {
    uint32_t m = 0;
    for (int i = threadIdx.x; i < t.n_max; i += kXfWaves * 64) m = m > t.block_max[i] ? m : t.block_max[i];
    m = wave_max(m);
    if (lane == 0) redm[wave] = m;       // (read behind the barriers below)
  }
  const float xs = xstat_combine<KIND>(partial, n_chunks, t.c_in, n_tok, red);
  if (wave == 0) stat[lane] = xs;
  __syncthreads();
  uint32_t top = 0;
  if (t.block_max) {
#pragma unroll
    for (int w = 0; w < kXfWaves; ++w) top = top > redm[w] ? top : redm[w];
    if (blockIdx.x == 0 && threadIdx.x == 0) *t.xmax_out = top;
  }
  const int64_t c = (int64_t)blockIdx.x * 64 + lane;
  if (c >= t.c_in) return;
  const double up = t.block_max ? pow2(shift_from_bf16_bits(top)) : pow2_shift(t.xmax_bits);
  for (int k = wave; k < t.n_alpha; k += kXfWaves)
    table_entry(stat[lane], t.alpha[k], up, (int64_t)k * t.c_in + c, t.s_table, t.s_copy, t.inv_table);
}

// The same for few rows, without partial sums: one launch instead of two.
template <typename T, int KIND>
__global__ __launch_bounds__(kXfWaves * 64) void xstat_table_direct_kernel(const uint16_t* __restrict__ X, int64_t n_tok,
                                                                           int64_t ldx, TableDev t) {
  __shared__ double red[kXfWaves][64];
  __shared__ float stat[64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float xs = xstat_direct<T, KIND>(X, n_tok, t.c_in, ldx, red);
  if (wave == 0) stat[lane] = xs;
  __syncthreads();
  const int64_t c = (int64_t)blockIdx.x * 64 + lane;
  if (c >= t.c_in) return;
  const double up = pow2_shift(t.xmax_bits);
  for (int k = wave; k < t.n_alpha; k += kXfWaves)
    table_entry(stat[lane], t.alpha[k], up, (int64_t)k * t.c_in + c, t.s_table, t.s_copy, t.inv_table);
}

size_t xstat_block_max_words(int64_t n_tok, int64_t c_in) { return (size_t)xstat_chunks(n_tok) * (size_t)ceil_div(c_in, kXsCols); }

hipError_t launch_xstat_table(const void* X, int64_t n_tok, int64_t c_in, int64_t ldx, bool bf16, int kind, double* partial,
                              const float* alpha, int n_alpha, float* s_table, float* s_copy, float* inv_table,
                              const uint32_t* xmax_bits, uint32_t* block_max, uint32_t* xmax_out, hipStream_t stream) {
  TableDev t{alpha, n_alpha, c_in, s_table, s_copy, inv_table, xmax_bits, block_max, 0, xmax_out};
  const double table_bytes = 8.0 * (double)n_alpha * (double)c_in;
  if (!block_max && n_tok <= kDirectRows) {
    ProfScope ps("xstat_table", stream, 2.0 * (double)n_tok * (double)c_in + table_bytes);
    auto go = [&](auto kern) {
      kern<<<(unsigned)ceil_div(c_in, 64), kXfWaves * 64, 0, stream>>>((const uint16_t*)X, n_tok, ldx, t);
    };
    if (!bf16) kind == 0 ? go(xstat_table_direct_kernel<F16, 0>) : go(xstat_table_direct_kernel<F16, 1>);
    else kind == 0 ? go(xstat_table_direct_kernel<BF16, 0>) : go(xstat_table_direct_kernel<BF16, 1>);
    return hipGetLastError();
  }
  const hipError_t e = launch_xstat_partial(X, n_tok, c_in, ldx, bf16, kind, partial, stream, nullptr, 1, block_max);
  if (e != hipSuccess) return e;
  const int chunks = xstat_chunks(n_tok);
  t.n_max = (int)xstat_block_max_words(n_tok, c_in);
  ProfScope ps("xstat_table", stream, 8.0 * (double)chunks * (double)c_in + table_bytes);
  auto go = [&](auto kern) { kern<<<(unsigned)ceil_div(c_in, 64), kXfWaves * 64, 0, stream>>>(partial, chunks, n_tok, t); };
  kind == 0 ? go(xstat_table_kernel<0>) : go(xstat_table_kernel<1>);
  return hipGetLastError();
}

__global__ void recip_kernel(const float* __restrict__ s, int64_t n, const uint32_t* __restrict__ xmax_bits,
                             float* __restrict__ inv) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) inv[i] = (float)(pow2_shift(xmax_bits) / (double)s[i]);
}

hipError_t launch_recip(const float* s, int64_t c_in, const uint32_t* xmax_bits, float* inv,
                        hipStream_t stream) {
  recip_kernel<<<(unsigned)ceil_div(c_in, 256), 256, 0, stream>>>(s, c_in, xmax_bits, inv);
  return hipGetLastError();
}

// ------------------------------------------------ bf16 activations -> fp16 operand
__global__ void zero_u32_kernel(uint32_t* p) { *p = 0u; }

// max over the tensor of the magnitude bits; for bf16 the integer order of the
// magnitude bits is the order of the magnitudes, so an integer atomic max is exact
// and order independent.  A wave walks whole rows (no index division) and a block ends in ONE atomic on
// the single result word: with one per wave and four times the blocks the atomics alone took 130 us.
// blockIdx.y picks the stretch of `per` chunks of a row: the whole row unless the rows are too few for the chip.
// (The tokens stay in the caches here, whatever their size: the conversion reads them once more.  Both passes over
// 40,960 x 4096 bf16, conversion past the caches: 152 us, with this one past them too 164; 65,536 x 4096 240 and 262.)
constexpr int kPrepBlocks = 1024;   // 4 per CU
__global__ __launch_bounds__(256) void absmax_bits_kernel(const uint16_t* __restrict__ X, int64_t n_tok,
                                                          int64_t c_in, int64_t ldx, int64_t per,
                                                          uint32_t* __restrict__ out, bool words) {
  __shared__ uint32_t red[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t chunks = c_in / 8, i0 = blockIdx.y * per, i1 = i0 + per < chunks ? i0 + per : chunks;
  uint32_t m = 0;
  for (int64_t r = (int64_t)blockIdx.x * 4 + wave; r < n_tok; r += (int64_t)gridDim.x * 4) {
    const uint16_t* row = X + r * ldx;
#pragma unroll 4
    for (int64_t i = i0 + lane; i < i1; i += 64) {
      const uint4 v = *reinterpret_cast<const uint4*>(row + i * 8);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t lo = w[j] & 0x7fffu, hi = (w[j] >> 16) & 0x7fffu;
        m = m > lo ? m : lo;
        m = m > hi ? m : hi;
      }
    }
  }
  m = wave_max(m);
  if (lane == 0) red[wave] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < 4; ++i) m = m > red[i] ? m : red[i];
    if (words) out[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = m;
    else atomicMax(out, m);
  }
}

__device__ __forceinline__ float down_scale(uint32_t top) {
  return __builtin_bit_cast(float, (uint32_t)(127 - shift_from_bf16_bits(top)) << 23);
}
__device__ __forceinline__ uint4 bf16x8_to_f16(const uint4& v, float scale) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  uint32_t o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float lo = BF16::to_float((uint16_t)w[j]) * scale, hi = BF16::to_float((uint16_t)(w[j] >> 16)) * scale;
    o[j] = (uint32_t)F16::from_float(lo) | ((uint32_t)F16::from_float(hi) << 16);
  }
  return make_uint4(o[0], o[1], o[2], o[3]);
}
// the reciprocals of a scale vector for the tokens' shift, dealt over the blocks of a launch
__device__ __forceinline__ void recip_share(const float* __restrict__ s, int64_t n, uint32_t top, float* __restrict__ inv) {
  const double up = pow2(shift_from_bf16_bits(top));
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    inv[i] = (float)(up / (double)s[i]);
}

// All of it in one launch for few tokens: every block reads them all for the maximum (from L2 but for the first time) and
// converts its share.  Latency-bound, see xprep_whole.
__global__ __launch_bounds__(1024) void xprep_whole_kernel(const uint16_t* __restrict__ X, uint32_t pieces, uint32_t chunks,
                                                           int64_t ldx, uint32_t* __restrict__ xmax, uint16_t* __restrict__ Xh,
                                                           const float* __restrict__ s, float* __restrict__ inv) {
  __shared__ uint32_t red[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t row = threadIdx.x / chunks, col = threadIdx.x - row * chunks;
  const uint32_t drow = 1024 / chunks, dcol = 1024 - drow * chunks;
  u16x2 m = {0, 0};
#pragma unroll 8
  for (uint32_t i = threadIdx.x; i < pieces; i += 1024) {
    const uint4 v = *reinterpret_cast<const uint4*>(X + row * ldx + col * 8);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, w[j] & 0x7fff7fffu));
    col += dcol;
    row += drow;
    if (col >= chunks) { col -= chunks; ++row; }
  }
  uint32_t top = wave_max(m[0] > m[1] ? m[0] : m[1]);
  if (lane == 0) red[wave] = top;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 16; ++w) top = top > red[w] ? top : red[w];
  if (blockIdx.x == 0 && threadIdx.x == 0) *xmax = top;
  const uint32_t i = blockIdx.x * 1024 + threadIdx.x;
  if (i < pieces) {
    row = i / chunks;
    col = i - row * chunks;
    const uint4 v = *reinterpret_cast<const uint4*>(X + row * ldx + col * 8);
    *reinterpret_cast<uint4*>(Xh + (int64_t)i * 8) = bf16x8_to_f16(v, down_scale(top));
  }
  if (s) recip_share(s, (int64_t)chunks * 8, top, inv);
}

// NT, NTS: loads and stores past the caches.  n_words: the maximum is that of so many words (then it is stored in *xmax),
// 0: it is the one word, and nothing is stored, so it is a scalar load (20,000 x 4096 85.7 -> 85.2 us).
template <bool NT, bool NTS>
__global__ __launch_bounds__(256) void bf16_to_f16_kernel(const uint16_t* __restrict__ X, int64_t n_tok,
                                                          int64_t c_in, int64_t ldx, int64_t per,
                                                          const uint32_t* __restrict__ words, int n_words,
                                                          uint32_t* __restrict__ xmax, uint16_t* __restrict__ Xh,
                                                          const float* __restrict__ s, float* __restrict__ inv) {
  __shared__ uint32_t red[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t chunks = c_in / 8, i0 = blockIdx.y * per, i1 = i0 + per < chunks ? i0 + per : chunks;
  uint32_t top;
  if (n_words) {
    top = 0;
    for (int i = threadIdx.x; i < n_words; i += 256) top = top > words[i] ? top : words[i];
    top = wave_max(top);
    if (lane == 0) red[wave] = top;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 4; ++w) top = top > red[w] ? top : red[w];
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *xmax = top;
  } else {
    top = *words;
  }
  const float scale = down_scale(top);
  for (int64_t r = (int64_t)blockIdx.x * 4 + wave; r < n_tok; r += (int64_t)gridDim.x * 4) {
#pragma unroll 4
    for (int64_t i = i0 + lane; i < i1; i += 64)
      store16<NTS>(Xh + r * c_in + i * 8, bf16x8_to_f16(load16<NT>(X + r * ldx + i * 8), scale));
  }
  if (s && blockIdx.y == 0) recip_share(s, c_in, top, inv);
}

hipError_t launch_xprep(const void* X, int64_t n_tok, int64_t c_in, int64_t ldx, uint32_t* xmax_bits,
                        void* Xh, hipStream_t stream, bool have_max, uint32_t* words, size_t room, const float* s, float* inv) {
  ProfScope ps("bf16_to_f16", stream, 6.0 * (double)n_tok * (double)c_in);
  const int64_t pieces = n_tok * (c_in / 8);
  if (!have_max && xprep_whole(n_tok, c_in)) {
    xprep_whole_kernel<<<(unsigned)ceil_div(pieces, 1024), 1024, 0, stream>>>((const uint16_t*)X, (uint32_t)pieces, (uint32_t)(c_in / 8),
                                                                              ldx, xmax_bits, (uint16_t*)Xh, s, inv);
    return hipGetLastError();
  }
  const int64_t rows = ceil_div(n_tok, 4);
  // Few rows: split them into as many stretches (of 512 channels at least) as give every CU a block (us for the
  // three launches, a wave a row -> split: 4 x 131072 45.5 -> 12.6, 1 x 65536 23.7 -> 12.5, 64 x 65536
  // 26.7 -> 12.3).
  const int64_t per = ceil_div(ceil_div(c_in, 512), rows < 256 ? 256 / rows : 1) * 64;   // in chunks of 8 channels
  const unsigned split = (unsigned)ceil_div(c_in / 8, per);
  const dim3 mgrid((unsigned)(rows < kPrepBlocks ? rows : kPrepBlocks), split), cgrid((unsigned)(rows < 8192 ? rows : 8192), split);
  const size_t n_words = (size_t)mgrid.x * mgrid.y;
  const bool by_words = !have_max && words && n_words * sizeof(uint32_t) <= room && n_words <= 4096;
  if (!have_max) {
    if (!by_words) zero_u32_kernel<<<1, 1, 0, stream>>>(xmax_bits);
    absmax_bits_kernel<<<mgrid, 256, 0, stream>>>((const uint16_t*)X, n_tok, c_in, ldx, per, by_words ? words : xmax_bits, by_words);
  }
  auto go = [&](auto kern) {
    kern<<<cgrid, 256, 0, stream>>>((const uint16_t*)X, n_tok, c_in, ldx, per, by_words ? words : xmax_bits, by_words ? (int)n_words : 0, xmax_bits,
                                    (uint16_t*)Xh, s, inv);
  };
  const double bytes = (double)n_tok * (double)c_in;
  if (!streams_past(4.0 * bytes)) go(bf16_to_f16_kernel<false, false>);
  else if (!outgrows_cache(2.0 * bytes)) go(bf16_to_f16_kernel<true, false>);
  else go(bf16_to_f16_kernel<true, true>);
  return hipGetLastError();
}

// ------------------------------------------- final combine (S4) + select (S5)
// Wave k of the block sums candidate k's tile partials in double in a fixed order (lane-strided, then a fixed
// butterfly), scales by 1/c_out, and stores the loss as float (+inf if not finite).  Wave 0 then picks the first
// minimum (Sec. 3.2.1 argmin, in as many exchanges as the candidates need: six for one of them were 0.5 us) and the block copies that row of the table.  The order does not depend on the number of
// waves.  The partials are loaded 16 at a time and added in order (latency-bound, 20 candidates of 12000 tiles 167 -> 25 us, of
// 640 tiles 13 -> 8), up to 64 of them those of eight candidates at a time.  sl: TLQ_MAX_ALPHA floats of LDS and one int.
__device__ __forceinline__ void finalize_block(const FinalDev& f, float* sl) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
  const double scale = f.inv_c_out;
  auto finish = [&](int k, double acc) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) {
      float l = (float)(acc * scale * (f.factor ? *f.factor : 1.0));
      if (!(l == l) || l == __builtin_inff() || l == -__builtin_inff()) l = __builtin_inff();
      sl[k] = l;
      f.losses[k] = l;
    }
  };
  if (f.tiles <= 64) {
    for (int k0 = wave; k0 < f.n_cand; k0 += 8 * nwaves) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int k = k0 + j * nwaves < f.n_cand ? k0 + j * nwaves : k0;
        v[j] = f.partial[(int64_t)k * f.tiles + (lane < f.tiles ? lane : 0)];
      }
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (k0 + j * nwaves < f.n_cand) finish(k0 + j * nwaves, lane < f.tiles ? (double)v[j] : 0.0);
    }
  } else {
    for (int k = wave; k < f.n_cand; k += nwaves) {
      double acc = 0.0;
      const float* p = f.partial + (int64_t)k * f.tiles;
      for (int64_t i = lane; i < f.tiles; i += 16 * 64) {   // 16 loads in flight, added in order
        float v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = p[i + j * 64 < f.tiles ? i + j * 64 : lane];   // (no branch)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc += i + j * 64 < f.tiles ? (double)v[j] : 0.0;
      }
      finish(k, acc);
    }
  }
  if (!f.best_idx && !f.best_scales) return;
  int* sbest = reinterpret_cast<int*>(sl + TLQ_MAX_ALPHA);
  __syncthreads();
  if (wave == 0) {
    float bl = lane < f.n_cand ? sl[lane] : __builtin_inff();     // (n_cand <= TLQ_MAX_ALPHA = 64)
    int b = bl < __builtin_inff() ? lane : -1;
    for (int off = 1; off < f.n_cand; off <<= 1) {
      const float ol = __shfl_xor(bl, off, 64);
      const int ob = __shfl_xor(b, off, 64);
      if (ob >= 0 && (b < 0 || ol < bl || (ol == bl && ob < b))) { bl = ol; b = ob; }
    }
    if (lane == 0) {
      *sbest = b;
      if (f.best_idx) *f.best_idx = b;
    }
  }
  __syncthreads();
  if (f.best_scales) {
    const int b = *sbest;
    for (int64_t c = threadIdx.x; c < f.c_in; c += blockDim.x)
      f.best_scales[c] = b >= 0 ? f.s_table[(int64_t)b * f.c_in + c] : __builtin_nanf("");
  }
}

__global__ __launch_bounds__(1024) void finalize_kernel(FinalDev f) {
  __shared__ float sl[TLQ_MAX_ALPHA + 1];
  finalize_block(f, sl);
}

hipError_t launch_finalize(const FinalDev& f, hipStream_t stream) {
  ProfScope ps("finalize", stream, 4.0 * (double)f.n_cand * (double)f.tiles);
  finalize_kernel<<<1, 1024, 0, stream>>>(f);
  return hipGetLastError();
}

// Block 0 combines the loss, the others the errors of 256 tokens each: one launch instead of two of 4 us.
__global__ __launch_bounds__(256) void layer_err_kernel(FinalDev f, const float* __restrict__ tok_partial, int64_t tiles_o,
                                                        int64_t n_tok, float* __restrict__ out) {
  __shared__ float sl[TLQ_MAX_ALPHA + 1];
  if (blockIdx.x == 0) {
    finalize_block(f, sl);
    return;
  }
  const int64_t t = (int64_t)(blockIdx.x - 1) * 256 + threadIdx.x;
  if (t >= n_tok) return;
  double acc = 0.0;
#pragma unroll 8
  for (int64_t i = 0; i < tiles_o; ++i) acc += (double)tok_partial[i * n_tok + t];
  out[t] = (float)(acc * f.inv_c_out);
}

hipError_t launch_layer_err(const FinalDev& f, const float* tok_partial, int64_t tiles_o, int64_t n_tok, float* err, hipStream_t stream) {
  ProfScope ps("token_err_reduce", stream, 4.0 * (double)tiles_o * (double)n_tok);
  layer_err_kernel<<<(unsigned)ceil_div(n_tok, 256) + 1, 256, 0, stream>>>(f, tok_partial, tiles_o, n_tok, err);
  return hipGetLastError();
}

}  // namespace tlq
