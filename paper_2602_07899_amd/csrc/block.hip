// Glue of the synthetic decoder block that the calibrated linears sit in (not
// part of the paper's method; Sec. 3.2.1 only requires that activations are
// propagated through the model between two searches): causal self-attention per
// calibration sample, the SiLU gate and the residual addition.
#include <utility>

#include "common.h"

namespace tlq {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

#if defined(__HIP_DEVICE_COMPILE__)
template <typename T> __device__ __forceinline__ f32x16 mma16(u16x8 a, u16x8 b, f32x16 c);
template <> __device__ __forceinline__ f32x16 mma16<F16>(u16x8 a, u16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x16 mma16<BF16>(u16x8 a, u16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// 16-bit transposing LDS read: 16 lanes address four rows of 16 elements (four lanes x 8 bytes a row) and
// lane i of the sixteen receives column i of those four rows
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u16x4 lds_read_tr(const unsigned char* p) {
  return __builtin_bit_cast(u16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                       (__attribute__((address_space(3))) s16x4*)(uint32_t)(uintptr_t)p));
}
// the value that lane ^ 32 holds
__device__ __forceinline__ float other_half(float v) { return __shfl_xor(v, 32, 64); }
#endif

constexpr int kAttDh = 128;   // head width
constexpr int kAttBq = 128;   // queries per block (32 per wave)
[[maybe_unused]] constexpr int kAttBk = 64;    // keys per step (two 32-key halves)
[[maybe_unused]] constexpr int kAttRow = kAttDh * 2;             // bytes per LDS row of K or V
[[maybe_unused]] constexpr int kAttTile = kAttBk * kAttRow;      // bytes of one K or V tile

// out[t, head] = softmax_j<=t( q_t . k_j / sqrt(128) ) v_j, rows in blocks of seq_len.
// The matrix cores compute the TRANSPOSED products S^T = K Q^T and O^T = V^T P^T, so that a lane
// owns one query column: the running reference and sum of the online softmax are per-lane scalars
// shared only with lane ^ 32.  The accumulator registers of S^T, taken in order, are the keys
// 16 sl + 8 (e / 4) + 4 (lane / 32) + e % 4 of a 16-key step; the transposing LDS read hands a lane
// four keys of one column of V, so V^T is read in that same order and P never moves between lanes.
//
// What bounds it: per 32 queries x 64 keys a wave spends 1024 cycles on its matrix core, about as long
// on the softmax (32 exponentials a lane) and its share of 128 B/cycle of LDS reads; two blocks per CU
// (64 KB of LDS, <= 256 registers) overlap the three (matrix cores busy 30 % of the time, the
// rest is exposed latency of that chain).  Per step: the next 64 keys are fetched into registers while
// this step computes and go to the other LDS stage behind it (one barrier per step).
// The softmax advances 32 keys at a time with the exact running maximum as its reference, so that the
// largest probability is exactly 1 in 16 bits; the 64 output accumulators are rescaled only where some
// query of the wave meets a new maximum.  (One reference per 64 keys, raised only by a rise of 2^8:
// 2.99 ms instead of 3.27, but an error against 64 bits of 2.1e-3 instead of 1.8e-3, not kept.)
// All query blocks of a (sample, head) run on one XCD, so that its keys and values (0.6 MB at 1200
// tokens) are fetched into one L2, not into eight.  Fewer than eight pairs would leave XCDs idle that way:
// their query blocks are dealt over all eight (us, one XCD a pair -> dealt: 32768 tokens, one pair
// 2156 -> 791, two 2395 -> 943; 8192 tokens, four pairs 228 -> 214).
// LDS rows are 256 B; the 16-byte chunks of a K row are XORed with row % 16, the 32-byte pairs of a V
// row with a permutation of row % 8: fragment reads and transposing reads hit each bank once.
// 128 samples x 1200 tokens x 40 heads, bf16: 3.27 ms (578 TFLOP/s) against 8.87 ms with 32-key steps,
// K fragments read from global memory by every wave and V transposed by 2-byte LDS stores.
template <typename T>
__global__ __launch_bounds__(256, 2) void causal_attention_kernel(
    const uint16_t* __restrict__ Q, int64_t ldq, const uint16_t* __restrict__ K, int64_t ldk,
    const uint16_t* __restrict__ V, int64_t ldv, uint16_t* __restrict__ O, int64_t ldo, int seq_len,
    int n_heads, int64_t n_hs, unsigned ways, float scale) {
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ __attribute__((aligned(1024))) unsigned char kv[2][2][kAttTile];   // [stage][K, V]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, h = lane >> 5;
  // blockIdx.x = ways * query block + pair: with 8 ways the 8 XCDs work on 8 different (sample, head) pairs
  unsigned pair = blockIdx.x & 7, qblock = blockIdx.x >> 3, n_qblocks = gridDim.x >> 3;
  if (ways != 8) {
    qblock = blockIdx.x / ways;
    pair = blockIdx.x - qblock * ways;
    n_qblocks = gridDim.x / ways;
  }
  const int64_t hs = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * ways + pair;
  if (hs >= n_hs) return;
  const int qb = (int)(n_qblocks - 1 - qblock);  // longest rows first
  const int64_t row0 = (hs / n_heads) * seq_len;
  const int64_t col0 = (hs % n_heads) * kAttDh;
  const int q0 = qb * kAttBq + wave * 32;
  const int q = q0 + l32;                      // may lie past the end of the sample: computed, never stored
  const int qc = q < seq_len ? q : seq_len - 1;

  u16x8 qf[8];
  {
    const uint16_t* qp = Q + (row0 + qc) * ldq + col0 + 8 * h;
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[s] = *reinterpret_cast<const u16x8*>(qp + 16 * s);
  }
  f32x16 acc[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[dt][v] = 0.0f;
  float m_run = -INFINITY, l_run = 0.0f;

  int last_q = qb * kAttBq + kAttBq - 1;
  if (last_q > seq_len - 1) last_q = seq_len - 1;
  const int n_kt = last_q / kAttBk + 1;
  int wave_last_q = q0 + 31;
  if (wave_last_q > seq_len - 1) wave_last_q = seq_len - 1;
  if (q0 > wave_last_q) wave_last_q = -1;      // the whole wave lies past the end: it only helps to load

  // global -> registers -> LDS: 64 rows x 16 chunks each of K and V, four 16-byte chunks a thread
  const int srow = tid >> 4, sch = tid & 15;     // rows srow + 16 i
  const uint16_t* kp0 = K + (row0 + srow) * ldk + col0 + sch * 8;
  const uint16_t* vp0 = V + (row0 + srow) * ldv + col0 + sch * 8;
  u16x8 gk[4], gv[4];
  auto fetch = [&](int kt) {
    const int first = kt * kAttBk;
    if (first + kAttBk <= seq_len) {   // block-uniform; the row products are scalar here
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        gk[i] = *reinterpret_cast<const u16x8*>(kp0 + (int64_t)(first + i * 16) * ldk);
        gv[i] = *reinterpret_cast<const u16x8*>(vp0 + (int64_t)(first + i * 16) * ldv);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        int key = first + i * 16 + srow;
        if (key > seq_len - 1) key = seq_len - 1;  // masked below
        gk[i] = *reinterpret_cast<const u16x8*>(kp0 + (int64_t)(key - srow) * ldk);
        gv[i] = *reinterpret_cast<const u16x8*>(vp0 + (int64_t)(key - srow) * ldv);
      }
    }
  };
  // (row + 16 i) has the same row % 16, so the swizzled position inside the row is the same for all i
  const int kpos = srow * kAttRow + ((sch ^ srow) << 4);
  const int vpos = srow * kAttRow + (((((sch >> 1) ^ (((srow & 3) << 1) | ((srow >> 2) & 1))) << 1) | (sch & 1)) << 4);
  auto stash = [&](int stage) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      *reinterpret_cast<u16x8*>(&kv[stage][0][kpos + i * 16 * kAttRow]) = gk[i];
      *reinterpret_cast<u16x8*>(&kv[stage][1][vpos + i * 16 * kAttRow]) = gv[i];
    }
  };
  const int kbase = l32 * kAttRow + ((h ^ (l32 & 15)) << 4);
  const int r4 = (lane & 15) >> 2, vg = (lane >> 4) & 1;
  const int vbase = (h * 4 + r4) * kAttRow + (((vg ^ h) << 1 | ((lane >> 1) & 1)) << 4) + (lane & 1) * 8;

  // one step of NSUB 32-key halves; MASK: the last half holds keys beyond some query of the wave
  auto step = [&](auto nsub_c, auto mask_c, int kt, int stage) {
    constexpr int NSUB = decltype(nsub_c)::value;
    constexpr bool MASK = decltype(mask_c)::value != 0;
    f32x16 s[NSUB];
#pragma unroll
    for (int u = 0; u < NSUB; ++u)
#pragma unroll
      for (int v = 0; v < 16; ++v) s[u][v] = 0.0f;
    const unsigned char* kt_lds = kv[stage][0];
#pragma unroll
    for (int st = 0; st < 8; ++st)
#pragma unroll
      for (int u = 0; u < NSUB; ++u)
        s[u] = mma16<T>(*reinterpret_cast<const u16x8*>(kt_lds + u * 32 * kAttRow + (kbase ^ (st << 5))), qf[st], s[u]);
    const unsigned char* vt_lds = kv[stage][1];
#pragma unroll
    for (int u = 0; u < NSUB; ++u) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[u][v] *= scale;
        if (MASK && u == NSUB - 1) {
          const int key = kt * kAttBk + u * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
          s[u][v] = key <= q ? s[u][v] : -INFINITY;
        }
      }
      float mx = s[u][0];
#pragma unroll
      for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[u][v]);
      // wave-uniform: while no query meets a new maximum every factor is exactly 1
      float alpha = 1.0f;
      if (__builtin_amdgcn_ballot_w64(mx > m_run) != 0) {
        // key 0 is visible to every query and is part of the first step, so m_run becomes finite there
        const float m_new = fmaxf(m_run, fmaxf(mx, other_half(mx)));
        alpha = __expf(m_run - m_new);
        m_run = m_new;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[dt][v] *= alpha;
      }
      float ps = 0.0f;
      u16x8 pf[2];
#pragma unroll
      for (int sl = 0; sl < 2; ++sl)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float pv = __expf(s[u][8 * sl + e] - m_run);
          ps += pv;
          pf[sl][e] = T::from_float(pv);
        }
      l_run = __builtin_fmaf(l_run, alpha, ps);
#pragma unroll
      for (int sl = 0; sl < 2; ++sl)
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) {
          const unsigned char* p = vt_lds + (2 * u + sl) * 16 * kAttRow + (vbase ^ ((dt ^ r4) << 6));
          const u16x4 lo = lds_read_tr(p), hi = lds_read_tr(p + 8 * kAttRow);
          const u16x8 a = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          acc[dt] = mma16<T>(a, pf[sl], acc[dt]);
        }
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;

  fetch(0);
  stash(0);
  __syncthreads();
  for (int kt = 0; kt < n_kt; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < n_kt) fetch(kt + 1);
    // wave-uniform: a wave's queries start at a multiple of 32, so only its last 32 visible keys are masked
    if (kt * kAttBk + 63 < q0 && wave_last_q >= 0) step(I2{}, I0{}, kt, cur);
    else if (kt * kAttBk + 32 <= wave_last_q) step(I2{}, I1{}, kt, cur);
    else if (kt * kAttBk <= wave_last_q) step(I1{}, I1{}, kt, cur);
    if (kt + 1 < n_kt) stash(cur ^ 1);
    __syncthreads();
  }
  l_run += other_half(l_run);
  // the wave's 32 x 128 outputs leave as whole rows through its own quarter of the (now free) stages
  const float inv = 1.0f / l_run;
  unsigned char* ol = &kv[0][0][0] + wave * 32 * kAttRow;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      u16x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = T::from_float(acc[dt][4 * j + i] * inv);
      *reinterpret_cast<u16x4*>(ol + l32 * kAttRow + (((dt * 4 + j) ^ (l32 & 15)) << 4) + h * 8) = o;
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = i * 4 + (lane >> 4), c = lane & 15;
    const u16x8 o = *reinterpret_cast<const u16x8*>(ol + r * kAttRow + ((c ^ (r & 15)) << 4));
    if (q0 + r < seq_len) *reinterpret_cast<u16x8*>(O + (row0 + q0 + r) * ldo + col0 + c * 8) = o;
  }
#endif
}

hipError_t launch_causal_attention(const void* Q, int64_t ldq, const void* K, int64_t ldk, const void* V,
                                   int64_t ldv, int64_t n_tok, int n_heads, int seq_len, bool bf16, void* O,
                                   int64_t ldo, hipStream_t stream) {
  const int64_t n_samples = n_tok / seq_len;
  // causal: half of the seq_len^2 score matrix; 2 products of 2*128 flop per score
  ProfScope ps("causal_attention", stream, 2.0 * (double)n_samples * n_heads * (double)seq_len * seq_len * kAttDh);
  const int64_t n_hs = n_samples * n_heads;
  const unsigned ways = n_hs < 8 ? (unsigned)n_hs : 8u;    // pairs side by side (see the kernel)
  const int64_t groups = ceil_div(n_hs, ways);
  const int64_t gy = groups < 32768 ? groups : 32768;
  const dim3 grid(ways * (unsigned)ceil_div(seq_len, kAttBq), (unsigned)gy, (unsigned)ceil_div(groups, gy));
  const float scale = 0.08838834764831845f;  // 1 / sqrt(128)
  if (!bf16)
    causal_attention_kernel<F16><<<grid, 256, 0, stream>>>((const uint16_t*)Q, ldq, (const uint16_t*)K, ldk,
                                                           (const uint16_t*)V, ldv, (uint16_t*)O, ldo, seq_len, n_heads,
                                                           n_hs, ways, scale);
  else
    causal_attention_kernel<BF16><<<grid, 256, 0, stream>>>((const uint16_t*)Q, ldq, (const uint16_t*)K, ldk,
                                                            (const uint16_t*)V, ldv, (uint16_t*)O, ldo, seq_len, n_heads,
                                                            n_hs, ways, scale);
  return hipGetLastError();
}

// MODE 0: out = SiLU(a) * b;  MODE 1: out = a + b.  8 elements per thread; c % 8 == 0.
template <typename T, int MODE>
__global__ __launch_bounds__(256) void pairwise_kernel(const uint16_t* __restrict__ A, int64_t lda,
                                                       const uint16_t* __restrict__ B, int64_t ldb, int64_t n_tok,
                                                       int64_t c8, uint16_t* __restrict__ out, int64_t ldo) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n_tok * c8) return;
  const int64_t row = i / c8, col = (i % c8) * 8;
  const u16x8 a = *reinterpret_cast<const u16x8*>(A + row * lda + col);
  const u16x8 b = *reinterpret_cast<const u16x8*>(B + row * ldb + col);
  u16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float x = T::to_float(a[e]), y = T::to_float(b[e]);
    o[e] = T::from_float(MODE == 0 ? x / (1.0f + __expf(-x)) * y : x + y);
  }
  *reinterpret_cast<u16x8*>(out + row * ldo + col) = o;
}

hipError_t launch_pairwise(int mode, const void* A, int64_t lda, const void* B, int64_t ldb, int64_t n_tok,
                           int64_t c, bool bf16, void* out, int64_t ldo, hipStream_t stream) {
  ProfScope ps(mode == 0 ? "silu_mul" : "residual_add", stream, 6.0 * (double)n_tok * (double)c);
  const int64_t c8 = c / 8;
  const unsigned grid = (unsigned)ceil_div(n_tok * c8, 256);
#define TLQ_PW(TT, M)                                                                                          \
  pairwise_kernel<TT, M><<<grid, 256, 0, stream>>>((const uint16_t*)A, lda, (const uint16_t*)B, ldb, n_tok, c8, \
                                                   (uint16_t*)out, ldo)
  if (mode == 0) { if (bf16) TLQ_PW(BF16, 0); else TLQ_PW(F16, 0); }
  else           { if (bf16) TLQ_PW(BF16, 1); else TLQ_PW(F16, 1); }
#undef TLQ_PW
  return hipGetLastError();
}

}  // namespace tlq
