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
                                       (__attribute__((address_space(3))) s16x4*)p));
}
// the value that lane ^ 32 holds
__device__ __forceinline__ float other_half(float v) { return __shfl_xor(v, 32, 64); }
// the larger of a lane's value and lane ^ 32's.  In assembly because the builtin's two results come out as one; the two
// wait states are what the swap needs behind the write of its operand.
__device__ __forceinline__ float pair_max(float v) {
  float a = v, b = v;
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
  return fmaxf(a, b);
}
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __attribute__((address_space(1))) const void* glb_ptr_t;
#endif

constexpr int kAttDh = 128;   // head width
constexpr int kAttBq = 128;   // queries per block (32 per wave)
[[maybe_unused]] constexpr int kAttBk = 32;    // keys per step
[[maybe_unused]] constexpr int kAttRow = kAttDh * 2;             // bytes per LDS row of K or V
[[maybe_unused]] constexpr int kAttTile = kAttBk * kAttRow;      // bytes of one K or V tile
constexpr int64_t kAttWide = 1LL << 27;   // row strides from which eight rows no longer fit 32-bit byte offsets

// out[t, head] = softmax_j<=t( q_t . k_j / sqrt(128) ) v_j, rows in blocks of seq_len.
// The matrix cores compute the TRANSPOSED products S^T = K Q^T and O^T = V^T P^T, so that a lane
// owns one query column: the running reference and sum of the online softmax are per-lane scalars
// shared only with lane ^ 32.  The accumulator registers of S^T, taken in order, are the keys
// 16 sl + 8 (e / 4) + 4 (lane / 32) + e % 4 of a 16-key step; the transposing LDS read hands a lane
// four keys of one column of V, so V^T is read in that same order and P never moves between lanes.
//
// What bounds it: the issue of vector instructions and, behind that, power.  Per 32 queries x 32 keys a wave issues
// about 170 vector instructions of four cycles and 16 exponentials of eight beside 16 MFMAs of 32 cycles; three
// waves per SIMD (<= 168 registers, 32 KB of LDS a block) overlap the two.  The next 32 keys go from global memory
// to the other LDS stage without registers (the 32 registers of a staged tile were what held it to two waves),
// four K fragments are read ahead of the score product and the first V fragments before the softmax.
// 128 samples x 1200 tokens x 40 heads, bf16: 3.35 -> 2.73 ms, 7.0 -> 5.0 million cycles; the clock falls from 2.14 to
// 1.90 GHz as the chip gets busier, so further overlap pays less than it saves.  (Two waves per SIMD with the
// score product of the next half beside the softmax of this one: no faster than before, or spilled.)
// The softmax advances 32 keys at a time with the exact running maximum as its reference, so that the
// largest probability is exactly 1 in 16 bits; the output accumulators of a query are rescaled only where it meets a
// new maximum.  (One reference per 64 keys, raised only by a rise of 2^8: an error against 64 bits of 2.1e-3
// instead of 1.8e-3, not kept.  64 keys a step on 16x16x32 products, us 2685 -> 2470, 8 x 1024 x 32 94.9 -> 86.9: the
// error is 0.03 - 0.7 % larger in all of twenty shapes in bf16, because fewer keys are the maximum of their step, whose probability
// is exact; with the reference of every 32 keys again it is the same, but 2834 -> 2746, 16 x 512 x 32 63.4 -> 65.8.  With the
// sum over the rounded probabilities it is the same within 0.1 % or up to 1.2 % less, but then the denominator has 16-bit terms.
// Not kept.)
// All query blocks of a (sample, head) pair run on one XCD, so that its keys and values (0.6 MB at 1200
// tokens) are fetched into one L2, not into eight.  Fewer than eight pairs would leave XCDs idle that way:
// their query blocks are dealt over all eight (us, one XCD a pair -> dealt: 32768 tokens, one pair
// 2156 -> 791, two 2395 -> 943; 8192 tokens, four pairs 228 -> 214).  Up to kAttMembers pairs of an XCD are taken together,
// the longest query blocks of all of them first: pair by pair, a launch that fits the chip at once puts blocks of
// equal length on each CU (1 x 2048 tokens x 40 heads: 93 us pair by pair, 85 with four together, 62 with eight or
// sixteen; 128 x 1200 x 40 is the same with all of them).
// LDS rows are 256 B; the 16-byte chunks of a K row are XORed with row % 16, the 32-byte pairs of a V
// row with a permutation of row % 8: fragment reads and transposing reads hit each bank once.
// WIDE: rows too far apart for the 32-bit offsets inside a wave's eight rows go through registers.
constexpr int kAttMembers = 8;
template <typename T, bool WIDE>
__global__ __launch_bounds__(256, 3) void causal_attention_kernel(
    const uint16_t* __restrict__ Q, int64_t ldq, const uint16_t* __restrict__ K, int64_t ldk,
    const uint16_t* __restrict__ V, int64_t ldv, uint16_t* __restrict__ O, int64_t ldo, int seq_len,
    int n_heads, int64_t n_hs, unsigned ways, unsigned members, int n_qblocks, float scale) {
#if defined(__HIP_DEVICE_COMPILE__)
  // two stages of one step's K and V, apart from each other so that the compiler sees that the loads into one do not
  // touch what is read from the other
  __shared__ __attribute__((aligned(1024))) unsigned char stage0[2 * kAttTile], stage1[2 * kAttTile];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  // blockIdx.x = ways * (members * query block + member) + pair
  unsigned pair = blockIdx.x & 7, rest = blockIdx.x >> 3;
  if (ways != 8) {
    rest = blockIdx.x / ways;
    pair = blockIdx.x - rest * ways;
  }
  const unsigned qblock = rest / members, member = rest - qblock * members;
  const int64_t hs = (((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * members + member) * ways + pair;
  if (hs >= n_hs) return;
  const int qb = n_qblocks - 1 - (int)qblock;    // longest rows first
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
  // steps of this wave; none if it lies past the end: then it only helps to load
  const int n_mine = q0 <= wave_last_q ? wave_last_q / kAttBk + 1 : 0;

  // global -> LDS without registers: a wave-wide load fills four rows of 256 bytes, so the swizzle is on the global
  // side; a wave loads rows 8 wave + 4 i + lane / 16, i < 2, of K and of V.  Its descriptors begin at the first of
  // the eight rows and end with the sample: rows past it arrive as zeros (masked below).
  const int drow = lane >> 4, dch = lane & 15;
  const uint16_t* kn = K + (row0 + 8 * wave) * ldk + col0;     // of the next tile
  const uint16_t* vn = V + (row0 + 8 * wave) * ldv + col0;
  int left = seq_len - 8 * wave;                               // rows of the sample from there on
  auto fetch = [&](unsigned char* at) __attribute__((always_inline)) {
    unsigned char *ak = at + 2 * wave * 1024, *av = ak + kAttTile;
    if constexpr (WIDE) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int64_t r = 4 * i + drow < left ? 4 * i + drow : left - 1;     // (left - 1 may lie before kn, not the sample)
        const int kc = (dch ^ ((8 * wave + 4 * i + drow) & 15)) * 8;
        const int vc = ((((dch >> 1) ^ ((drow << 1) | (i & 1))) << 1) | (dch & 1)) * 8;
        *reinterpret_cast<u16x8*>(ak + i * 1024 + lane * 16) = *reinterpret_cast<const u16x8*>(kn + r * ldk + kc);
        *reinterpret_cast<u16x8*>(av + i * 1024 + lane * 16) = *reinterpret_cast<const u16x8*>(vn + r * ldv + vc);
      }
    } else {
      const int rows = left < 8 ? left : 8;
      const int kbytes = rows > 0 ? ((rows - 1) * (int)ldk + kAttDh) * 2 : 0;
      const int vbytes = rows > 0 ? ((rows - 1) * (int)ldv + kAttDh) * 2 : 0;
      const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)kn, 0, kbytes, 0x00020000);
      const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void*)vn, 0, vbytes, 0x00020000);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int r = 4 * i + drow;
        const int kvo = r * (int)ldk * 2 + (dch ^ ((8 * wave + r) & 15)) * 16;
        const int vvo = r * (int)ldv * 2 + ((((dch >> 1) ^ ((drow << 1) | (i & 1))) << 1) | (dch & 1)) * 16;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (lds_ptr_t)(ak + i * 1024), 16, kvo, 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lds_ptr_t)(av + i * 1024), 16, vvo, 0, 0, 0);
      }
    }
    kn += kAttBk * ldk;
    vn += kAttBk * ldv;
    left -= kAttBk;
  };
  const int kbase = l32 * kAttRow + ((h ^ (l32 & 15)) << 4);
  const int r4 = (lane & 15) >> 2, vg = (lane >> 4) & 1;
  const int vbase = (h * 4 + r4) * kAttRow + (((vg ^ h) << 1 | ((lane >> 1) & 1)) << 4) + (lane & 1) * 8;
  int ka[8], va[4];
#pragma unroll
  for (int st = 0; st < 8; ++st) ka[st] = kbase ^ (st << 5);
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) va[dt] = kAttTile + (vbase ^ ((dt ^ r4) << 6));

  // 32 keys; mask: some of them lie beyond some query of the wave
  auto step = [&](const unsigned char* kv, bool mask, int kt) __attribute__((always_inline)) {
    f32x16 s;
    u16x8 kf[4];
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.0f;
#pragma unroll
    for (int st = 0; st < 4; ++st) kf[st] = *reinterpret_cast<const u16x8*>(kv + ka[st]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      s = mma16<T>(kf[st & 3], qf[st], s);
      if (st < 4) kf[st] = *reinterpret_cast<const u16x8*>(kv + ka[st + 4]);
      __builtin_amdgcn_sched_barrier(0);
    }
    u16x8 vf[4];
    auto read_v = [&](int sl) __attribute__((always_inline)) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const unsigned char* p = kv + va[dt] + sl * 16 * kAttRow;
        const u16x4 lo = lds_read_tr(p), hi = lds_read_tr(p + 8 * kAttRow);
        vf[dt] = u16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      }
    };
    read_v(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] *= scale;
    if (mask) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int key = kt * kAttBk + 8 * (v >> 2) + 4 * h + (v & 3);
        s[v] = key <= q ? s[v] : -INFINITY;
      }
    }
    float mx = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
    // key 0 is visible to every query and is part of the first step, so m_run becomes finite there; only the lanes
    // whose query meets a new maximum take part in the rescaling, elsewhere the factor is exactly 1
    float alpha = 1.0f;
    const float m_new = fmaxf(m_run, pair_max(mx));
    if (m_new > m_run) {
      alpha = __expf(m_run - m_new);
      m_run = m_new;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[dt][v] *= alpha;
    }
    float ps = 0.0f;
#pragma unroll
    for (int sl = 0; sl < 2; ++sl) {
      u16x8 pf;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float pv = __expf(s[8 * sl + e] - m_run);
        ps += pv;
        pf[e] = T::from_float(pv);
      }
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) acc[dt] = mma16<T>(vf[dt], pf, acc[dt]);
      if (sl == 0) read_v(1);
    }
    l_run = __builtin_fmaf(l_run, alpha, ps);
  };
  // one barrier a step: behind it the next tile has landed (each wave has waited for its own loads) and the stage
  // read last may be refilled
  auto turn = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  auto walk = [&](unsigned char* here, unsigned char* next, int kt) __attribute__((always_inline)) {
    turn();
    if (kt + 1 < n_kt) fetch(next);
    // a wave's queries start at a multiple of 32, so only its last 32 visible keys are masked
    if (kt < n_mine) step(here, kt == n_mine - 1, kt);
  };
  fetch(stage0);
  for (int kt = 0; kt < n_kt; kt += 2) {
    walk(stage0, stage1, kt);
    if (kt + 1 < n_kt) walk(stage1, stage0, kt + 1);
  }
  __syncthreads();
  l_run += other_half(l_run);
  // the wave's 32 x 128 outputs leave as whole rows through its own quarter of the (now free) stages
  const float inv = 1.0f / l_run;
  unsigned char* ol = (wave < 2 ? stage0 : stage1) + (wave & 1) * 32 * kAttRow;
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
  const unsigned members = (unsigned)(groups < kAttMembers ? groups : kAttMembers);
  const int n_qblocks = (int)ceil_div(seq_len, kAttBq);
  const int64_t chunks = ceil_div(groups, members), gy = chunks < 32768 ? chunks : 32768;
  const dim3 grid(ways * members * (unsigned)n_qblocks, (unsigned)gy, (unsigned)ceil_div(chunks, gy));
  const float scale = 0.08838834764831845f;  // 1 / sqrt(128)
  const bool wide = ldk >= kAttWide || ldv >= kAttWide;
  auto go = [&](auto kern) {
    kern<<<grid, 256, 0, stream>>>((const uint16_t*)Q, ldq, (const uint16_t*)K, ldk, (const uint16_t*)V, ldv, (uint16_t*)O,
                                   ldo, seq_len, n_heads, n_hs, ways, members, n_qblocks, scale);
  };
  if (!bf16) wide ? go(causal_attention_kernel<F16, true>) : go(causal_attention_kernel<F16, false>);
  else wide ? go(causal_attention_kernel<BF16, true>) : go(causal_attention_kernel<BF16, false>);
  return hipGetLastError();
}

// MODE 0: out = SiLU(a) * b;  MODE 1: out = a + b.  8 elements per thread; c % 8 == 0.  HBM-bound; NT, NTS: loads and stores past
// the caches: gate of 40960 x 11008 477 -> 426 us (6.3 TB/s), sum of 40960 x 4096 171 -> 154 (6.5 TB/s).
template <typename T, int MODE, bool NT, bool NTS>
__global__ __launch_bounds__(256) void pairwise_kernel(const uint16_t* __restrict__ A, int64_t lda,
                                                       const uint16_t* __restrict__ B, int64_t ldb, int64_t n_tok,
                                                       int64_t c8, uint16_t* __restrict__ out, int64_t ldo) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n_tok * c8) return;
  const int64_t row = i / c8, col = (i % c8) * 8;
  const u16x8 a = __builtin_bit_cast(u16x8, load16<NT>(A + row * lda + col));
  const u16x8 b = __builtin_bit_cast(u16x8, load16<NT>(B + row * ldb + col));
  u16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float x = T::to_float(a[e]), y = T::to_float(b[e]);
    o[e] = T::from_float(MODE == 0 ? x / (1.0f + __expf(-x)) * y : x + y);
  }
  store16<NTS>(out + row * ldo + col, __builtin_bit_cast(uint4, o));
}

hipError_t launch_pairwise(int mode, const void* A, int64_t lda, const void* B, int64_t ldb, int64_t n_tok,
                           int64_t c, bool bf16, void* out, int64_t ldo, hipStream_t stream) {
  ProfScope ps(mode == 0 ? "silu_mul" : "residual_add", stream, 6.0 * (double)n_tok * (double)c);
  const int64_t c8 = c / 8;
  const unsigned grid = (unsigned)ceil_div(n_tok * c8, 256);
  const double bytes = (double)n_tok * (double)c;
  const bool nt = streams_past(6.0 * bytes), nts = nt && outgrows_cache(2.0 * bytes);
  auto go = [&](auto kern) {
    kern<<<grid, 256, 0, stream>>>((const uint16_t*)A, lda, (const uint16_t*)B, ldb, n_tok, c8, (uint16_t*)out, ldo);
  };
  auto pick = [&](auto t) {
    using T = decltype(t);
    auto of = [&](auto m) {
      constexpr int MODE = decltype(m)::value;
      if (!nt) go(pairwise_kernel<T, MODE, false, false>);
      else if (!nts) go(pairwise_kernel<T, MODE, true, false>);
      else go(pairwise_kernel<T, MODE, true, true>);
    };
    if (mode == 0) of(std::integral_constant<int, 0>{});
    else of(std::integral_constant<int, 1>{});
  };
  bf16 ? pick(BF16{}) : pick(F16{});
  return hipGetLastError();
}

}  // namespace tlq
