// Glue of the synthetic decoder block that the calibrated linears sit in (not
// part of the paper's method; Sec. 3.2.1 only requires that activations are
// propagated through the model between two searches): causal self-attention per
// calibration sample, the SiLU gate and the residual addition.
#include <utility>

#include "common.h"

namespace tlq {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

#if defined(__HIP_DEVICE_COMPILE__)
template <typename T> __device__ __forceinline__ f32x4 mma32(u16x8 a, u16x8 b, f32x4 c);
template <> __device__ __forceinline__ f32x4 mma32<F16>(u16x8 a, u16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x4 mma32<BF16>(u16x8 a, u16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
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
// Rows of 16 lanes: a's odd rows change places with b's even ones (swap16); a's upper half with b's lower one (swap32).  In
// assembly because the builtins' two results come out as one; the two wait states are what a swap needs behind the write of its
// operands.
__device__ __forceinline__ void swap16(float& a, float& b) { asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b)); }
// the larger of the two behind such an exchange (the compiler would first make sure that neither is a signalling NaN)
__device__ __forceinline__ float swap16_max(float a, float b) {
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 0\n\tv_max_f32 %0, %0, %1" : "+v"(a), "+v"(b));
  return a;
}
__device__ __forceinline__ float swap32_max(float a, float b) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 0\n\tv_max_f32 %0, %0, %1" : "+v"(a), "+v"(b));
  return a;
}
// the lane's number, worked out where it is needed instead of held in a register until then
__device__ __forceinline__ int lane_anew() {
  int v;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(v));
  return v;
}
// sum over the four rows; every lane gets it
__device__ __forceinline__ float rows_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}
// two floats rounded to 16 bits, and such a pair added to a sum
template <typename T> __device__ __forceinline__ uint32_t pack2(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef typename T::raw raw2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), raw2));
}
template <typename T> __device__ __forceinline__ float add2(uint32_t v, float sum);
template <> __device__ __forceinline__ float add2<F16>(uint32_t v, float sum) {
  typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
  return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, v), f16x2{(_Float16)1.0f, (_Float16)1.0f}, sum, false);
}
template <> __device__ __forceinline__ float add2<BF16>(uint32_t v, float sum) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v), bf16x2{(__bf16)1.0f, (__bf16)1.0f}, sum, false);
}
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __attribute__((address_space(1))) const void* glb_ptr_t;
#endif

constexpr int kAttDh = 128;   // head width
constexpr int kAttBq = 128;   // queries per block (32 per wave)
[[maybe_unused]] constexpr int kAttBk = 64;    // keys per step
[[maybe_unused]] constexpr int kAttRow = kAttDh * 2;             // bytes per row of V or of the outputs
[[maybe_unused]] constexpr int kAttHalf = kAttBk * kAttRow / 2;  // bytes of the first or second 64 columns of a K tile
[[maybe_unused]] constexpr int kAttTile = kAttBk * kAttRow;      // bytes of one K or V tile
constexpr int64_t kAttWide = 1LL << 27;   // row strides from which eight rows no longer fit 32-bit byte offsets

// out[t, head] = softmax_j<=t( q_t . k_j / sqrt(128) ) v_j, rows in blocks of seq_len.
// The matrix cores compute the TRANSPOSED products S^T = K Q^T and O^T = V^T P^T, so that a lane owns one query column of
// each of the wave's two tiles of 16 queries: the running reference and sum of the online softmax are per-lane scalars
// shared only with the lanes 16, 32 and 48 away.  A lane's scores of a 32-key block are the keys 4 g + i and 16 + 4 g + i
// (g = lane / 16); the transposing LDS read hands a lane four keys of one column of V, so V^T is read in that same order
// and P never moves between lanes.
//
// What bounds it: power, and behind it the issue of vector instructions.  128 samples x 1200 tokens x 40 heads, bf16:
// 2.68 -> 2.42 ms at 1.6 - 1.8 GHz (0.78 PFLOP/s); 8 x 1024 x 32 93.5 -> 83.1 us, 16 x 512 x 32 59.8 -> 54.8, 32 x 256 x 32
// 45.7 -> 44.5, 30 x 100 x 30 18.7 -> 18.8, against 32 keys a step with 32x32x16 products.  What it took:
// - 64 keys a step: the accumulators of a query are rescaled where it meets a new maximum, and some query of a wave
//   does so in most steps, so half the steps need little more than half of those 64 multiplications.  The two query tiles
//   are rescaled apart, and in the first step there is nothing to rescale.
// - A score less the maximum, times the factor of the exponential (before: two multiplications and a subtraction); the sum of
//   the probabilities is taken over their 16-bit values, two in an instruction (error against 64 bits before the output is
//   rounded, bf16: 8.1e-4 -> 7.9e-4).  Fewer vector instructions, 2.68 -> 2.45 ms with the steps above.  (One FMA of the score
//   with the factor and the rounded product of maximum and factor takes 1.4 % off the whole, but the largest score's exponent is
//   then the rounding of that product and not 0: at scores of 2^30 finite inputs gave infinities and NaN.)
// - 16x16x32 products: half the accumulator traffic of the 32x32x16 shape for the same operands (2.45 -> 2.38 ms).
// - A wave in its products goes first (s_setprio): the others of its SIMD fill in the softmax (2.38 -> 2.33 ms).
// - One K and one V tile in LDS, three waves per SIMD (<= 168 registers, 32 KB of LDS a block).  The next K tile is on its
//   way while the scores are turned into outputs, the V tile while they are formed.  (Two K tiles, so that both loads have
//   the whole step: no faster.)
// - Keys ascend.  (From the diagonal down the steps with a mask come first and need no rescaling, 2.36 ms; but then the
//   query blocks of a head ask for all its tiles within two steps, and where memory counts that is slower: 16 x 512 x 32
//   63.6 us, 32 x 256 x 32 50.6.)
// The softmax has the exact running maximum as its reference, so that the largest probability is exactly 1 in 16
// bits.  (A reference that is raised only by a rise of 2^8 or 2^4 makes errors of 2.0e-3 instead of 1.8e-3, not kept.)
// All query blocks of a (sample, head) pair run on one XCD, so that its keys and values (0.6 MB at 1200
// tokens) are fetched into one L2, not into eight.  Fewer than eight pairs would leave XCDs idle that way:
// their query blocks are dealt over all eight (us, one XCD a pair -> dealt: 32768 tokens, one pair
// 2156 -> 791, two 2395 -> 943; 8192 tokens, four pairs 228 -> 214).  Up to kAttMembers pairs of an XCD are taken together,
// the longest query blocks of all of them first: pair by pair, a launch that fits the chip at once puts blocks of
// equal length on each CU (1 x 2048 tokens x 40 heads: 93 us pair by pair, 85 with four together, 62 with eight or
// sixteen; 128 x 1200 x 40 is the same with all of them).
// LDS tiles are two halves of 64 columns, rows of 128 bytes; the 16-byte chunks of a K row are XORed with three bits of
// its number, the 32-byte blocks of a V row with two: fragment reads and transposing reads hit each bank once.
// WIDE: rows too far apart for the 32-bit offsets inside eight rows go through registers.
constexpr int kAttMembers = 8;
template <typename T, bool WIDE>
__global__ __launch_bounds__(256, 3) void causal_attention_kernel(
    const uint16_t* __restrict__ Q, int64_t ldq, const uint16_t* __restrict__ K, int64_t ldk,
    const uint16_t* __restrict__ V, int64_t ldv, uint16_t* __restrict__ O, int64_t ldo, int seq_len,
    int n_heads, int64_t n_hs, unsigned ways, unsigned members, int n_qblocks, float scale) {
#if defined(__HIP_DEVICE_COMPILE__)
  // one tile of K and one of V, apart from each other so that the compiler sees that the loads into one do not
  // touch what is read from the other
  __shared__ __attribute__((aligned(1024))) unsigned char ktile[kAttTile], vtile[kAttTile];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ql = lane & 15, g = lane >> 4;
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
  // query tile u of the wave: queries q0 + 16 u + ql (those past the end of the sample are never stored)
  u16x8 qf[2][4];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int q = q0 + 16 * u + ql;
    const uint16_t* qp = Q + (row0 + (q < seq_len ? q : seq_len - 1)) * ldq + col0 + 8 * g;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) qf[u][kk] = *reinterpret_cast<const u16x8*>(qp + 32 * kk);
  }
  f32x4 acc[8][2];
#pragma unroll
  for (int d = 0; d < 8; ++d)
#pragma unroll
    for (int u = 0; u < 2; ++u) acc[d][u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // the running maximum of q . k (of tile 0 in the even rows of lanes, of tile 1 in the odd ones), the sums of
  // the probabilities as they are rounded
  float mc = -INFINITY, l_run[2] = {0.0f, 0.0f};

  int last_q = qb * kAttBq + kAttBq - 1;
  if (last_q > seq_len - 1) last_q = seq_len - 1;
  const int n_kt = last_q / kAttBk + 1;
  int wave_last_q = q0 + 31;
  if (wave_last_q > seq_len - 1) wave_last_q = seq_len - 1;
  // 32-key blocks of this wave; none if it lies past the end: then it only helps to load
  const int n_mine = q0 <= wave_last_q ? wave_last_q / 32 + 1 : 0;

  // global -> LDS without registers.  Both tiles are kept as two halves of 64 columns, rows of 128 bytes; a wave loads
  // 16 rows, eight half rows (1 KB) at a time, so the swizzle is on the global side.  A tile's key 32 a + 16 b + 8 c + d is
  // its row 32 a + 16 c + 8 b + d: the swizzle of the K chunks, row / 2 % 4 + 4 c, is then one for both of a
  // wave's loads.  The descriptors begin at the first of the eight keys and end with the sample: keys past it arrive as zeros.
  const int lrow = lane >> 3, first = (wave >> 1) * 32 + (wave & 1) * 8;
  const uint16_t* kn = K + (row0 + first) * ldk + col0;    // of the next tile
  const uint16_t* vn = V + (row0 + first) * ldv + col0;
  int kleft = seq_len - first, vleft = kleft;              // rows of the sample from there on
  const int kc = ((lane & 7) ^ (lrow >> 1) ^ (wave & 1) * 4) * 16, vc = ((lane & 7) ^ (lrow & 6)) * 16;
  auto fetch = [&](unsigned char* tile, const uint16_t*& next, int& left, int64_t ld, int c) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      unsigned char* at = tile + wave * 2048 + i * 1024;
      if constexpr (WIDE) {
        const int64_t r = 16 * i + lrow < left ? 16 * i + lrow : left - 1;    // (may lie before `next`, not before the sample)
#pragma unroll
        for (int half = 0; half < 2; ++half)
          *reinterpret_cast<u16x8*>(at + half * kAttHalf + lane * 16) =
              *reinterpret_cast<const u16x8*>(next + r * ld + half * 64 + c / 2);
      } else {
        const int rows = left - 16 * i < 8 ? left - 16 * i : 8;
        const int bytes = rows > 0 ? ((rows - 1) * (int)ld + kAttDh) * 2 : 0;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(next + 16 * i * ld), 0, bytes, 0x00020000);
#pragma unroll
        for (int half = 0; half < 2; ++half)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(at + half * kAttHalf), 16, lrow * (int)ld * 2 + c, half * 128, 0, 0);
      }
    }
    next += kAttBk * ld;
    left -= kAttBk;
  };
  auto fetch_k = [&]() __attribute__((always_inline)) { fetch(ktile, kn, kleft, ldk, kc); };
  auto fetch_v = [&]() __attribute__((always_inline)) { fetch(vtile, vn, vleft, ldv, vc); };
  // fragment addresses in the first half and the first rows; the others are constants away.  K: the row of key ql, the
  // 16-byte chunk 4 (kk % 2) + g, swizzled; V: the row of key 4 g + ql / 4, the 32-byte block d % 4 XOR row / 2 % 4.
  int ka[2], va[4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
    ka[i] = ((ql & 7) | (ql & 8) << 1) * 128 + (((4 * i + g) ^ ((ql >> 1 & 3) | (ql & 8) >> 1)) << 4);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    va[i] = ((g & 1) * 4 + (g >> 1) * 16 + (ql >> 2)) * 128 + ((i ^ (ql >> 3 | (g & 1) << 1)) << 5) + (ql & 3) * 8;
  // bytes from the first key of a tile to key 16 t
  auto key_tile = [](int t) { return (t >> 1) * 4096 + (t & 1) * 1024; };

  // scores of NB blocks of 32 keys
  auto scores = [&](auto nb, f32x4 (&s)[4][2]) __attribute__((always_inline)) {
    constexpr int NT = 2 * decltype(nb)::value, AHEAD = 4;
    u16x8 kf[AHEAD];
    auto read_k = [&](int i) __attribute__((always_inline)) {
      const int kk = i / NT, t = i % NT;
      kf[i % AHEAD] = *reinterpret_cast<const u16x8*>(ktile + ka[kk & 1] + (kk >> 1) * kAttHalf + key_tile(t));
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) read_k(i);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4 * NT; ++i) {
      const int t = i % NT;
#pragma unroll
      for (int u = 0; u < 2; ++u) s[t][u] = mma32<T>(kf[i % AHEAD], qf[u][i / NT], i < NT ? f32x4{0.0f, 0.0f, 0.0f, 0.0f} : s[t][u]);
      __builtin_amdgcn_sched_barrier(0);        // (the next fragment takes this one's registers)
      if (i + AHEAD < 4 * NT) read_k(i + AHEAD);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // the last block reaches beyond some query of the wave
  auto mask = [&](int w, f32x4 (&s)[4][2]) __attribute__((always_inline)) {
    const int el = lane_anew(), last = (el & 15) - 4 * (el >> 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[2 * w][0][i] = i <= last ? s[2 * w][0][i] : -INFINITY;
      s[2 * w + 1][0][i] = -INFINITY;
      s[2 * w + 1][1][i] = i <= last ? s[2 * w + 1][1][i] : -INFINITY;
    }
  };
  // softmax over a tile and its part of the output; `mine` blocks of 32 keys, the last of them masked, or more
  auto weigh = [&](int kt, int mine, f32x4 (&s)[4][2]) __attribute__((always_inline)) {
    constexpr int RING = 4;
    u16x8 vf[RING];
    auto read_v = [&](int i) __attribute__((always_inline)) {     // block i / 8 of 32 keys, channels 16 (i % 8) ..
      const int d = i & 7;
      const unsigned char* p = vtile + va[d & 3] + (d >> 2) * kAttHalf + (i >> 3) * 4096;
      const u16x4 lo = lds_read_tr(p), hi = lds_read_tr(p + 1024);
      vf[i % RING] = u16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    };
    if (mine <= 2) {      // (asked for in this order the steps without a mask keep all their values in registers)
      if (mine == 2) {
        mask(1, s);
      } else {
        mask(0, s);
      }
    }
    float mx[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      mx[u] = s[0][u][0];
#pragma unroll
      for (int v = 1; v < 16; ++v) mx[u] = fmaxf(mx[u], s[v >> 2][u][v & 3]);
    }
    const float both = swap16_max(mx[0], mx[1]);
    // (key 0 is visible to every query; elsewhere than at a new maximum the factor is exactly 1)
    const float top = swap32_max(both, both);
    const uint64_t up = __builtin_amdgcn_ballot_w64(top > mc);
    if (kt == 0) {
      mc = top;
    } else if (up) {
      const float to = top > mc ? top : mc;
      float al[2] = {__builtin_amdgcn_exp2f((mc - to) * scale), 0.0f};
      al[1] = al[0];
      mc = to;
      swap16(al[0], al[1]);
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (up & (u ? 0xffff0000ffff0000ull : 0x0000ffff0000ffffull)) {
          l_run[u] *= al[u];
#pragma unroll
          for (int d = 0; d < 8; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[d][u][i] *= al[u];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < RING; ++i) read_v(i);
    __builtin_amdgcn_sched_barrier(0);
    float ref[2] = {mc, mc};
    swap16(ref[0], ref[1]);
    // probabilities of keys 2 e, 2 e + 1 (of eight) of a lane in block w, tile u.  The difference first: the largest score's is
    // exactly 0, whatever its size
    auto pair_of = [&](int w, int u, int e) __attribute__((always_inline)) {
      const f32x4& x = s[2 * w + (e >> 1)][u];
      const uint32_t v = pack2<T>(__builtin_amdgcn_exp2f((x[2 * (e & 1)] - ref[u]) * scale),
                                  __builtin_amdgcn_exp2f((x[2 * (e & 1) + 1] - ref[u]) * scale));
      l_run[u] = add2<T>(v, l_run[u]);
      asm volatile("" : "+v"(l_run[u]));     // (now, not when its operands have been held to the end)
      return v;
    };
    uint32_t pf[2][2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) pf[0][u][e] = pair_of(0, u, e);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    // a block's products beside the exponentials of the next one
    auto products = [&](int w) __attribute__((always_inline)) {
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        const int i = 8 * w + d;
#pragma unroll
        for (int u = 0; u < 2; ++u) acc[d][u] = mma32<T>(vf[i % RING], __builtin_bit_cast(u16x8, pf[w][u]), acc[d][u]);
        __builtin_amdgcn_sched_barrier(0);      // (the next fragment takes this one's registers)
        if (i + RING < 16) read_v(i + RING);
        if (w == 0) pf[1][d & 1][d >> 1] = pair_of(1, d & 1, d >> 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    products(0);
    if (mine >= 2) products(1);
    __builtin_amdgcn_s_setprio(0);
  };
  // a barrier behind which the tile that was on its way has landed (each wave has waited for its own loads) and the one
  // read last may be refilled
  auto turn = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  fetch_k();
  for (int kt = 0; kt < n_kt; ++kt) {
    const int mine = n_mine - 2 * kt;       // blocks of 32 keys from here on; a wave's last one is masked
    turn();
    fetch_v();
    if (mine > 0) {
      f32x4 s[4][2];                        // s[t][u]: keys 16 t + 4 g + i of the tile, query tile u
      if (mine > 1) {
        scores(std::integral_constant<int, 2>{}, s);
      } else {
        scores(std::integral_constant<int, 1>{}, s);
#pragma unroll
        for (int t = 2; t < 4; ++t)
#pragma unroll
          for (int u = 0; u < 2; ++u) s[t][u] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      }
      turn();
      if (kt + 1 < n_kt) fetch_k();
      weigh(kt, mine, s);
    } else {
      turn();
      if (kt + 1 < n_kt) fetch_k();
    }
  }
  __syncthreads();
  // the wave's 32 x 128 outputs leave as whole rows through its own quarter of the (now free) tiles
  const int el = lane_anew(), eq = el & 15, eg = el >> 4;
  unsigned char* ol = (wave < 2 ? ktile : vtile) + (wave & 1) * 32 * kAttRow;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const float inv = 1.0f / rows_sum(l_run[u]);
#pragma unroll
    for (int d = 0; d < 8; ++d) {
      u16x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = T::from_float(acc[d][u][i] * inv);
      *reinterpret_cast<u16x4*>(ol + (16 * u + eq) * kAttRow + (((2 * d + (eg >> 1)) ^ eq) << 4) + (eg & 1) * 8) = o;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = i * 4 + eg, c = eq;
    const u16x8 o = *reinterpret_cast<const u16x8*>(ol + r * kAttRow + ((c ^ (r & 15)) << 4));
    if (q0 + r < seq_len) *reinterpret_cast<u16x8*>(O + (row0 + q0 + r) * ldo + col0 + c * 8) = o;
  }
#endif
}

[[maybe_unused]] constexpr int kShortBk = 32;                         // keys per step
[[maybe_unused]] constexpr int kShortTile = kShortBk * kAttRow;       // bytes of one K or V tile

// The same for short sequences and for launches that leave CUs without a block (short_attention): 32 keys a step, S^T = K Q^T
// and O^T = V^T P^T in 32x32x16 products, a lane owns one query column, its running reference and sum are shared only with
// lane ^ 32.  The accumulator registers of S^T, taken in order, are the keys 16 sl + 8 (e / 4) + 4 (lane / 32) + e % 4 of a
// 16-key step, and V^T is read in that order.  Two stages of K and V: the next 32 keys are on their way for a whole step.
// Latency-bound in such launches: 4.7 us for one step, 0.8 us for every further 64 keys.
// LDS rows are 256 B; the 16-byte chunks of a K row are XORed with row % 16, the 32-byte pairs of a V
// row with a permutation of row % 8: fragment reads and transposing reads hit each bank once.
template <typename T, bool WIDE>
__global__ __launch_bounds__(256, 3) void short_attention_kernel(
    const uint16_t* __restrict__ Q, int64_t ldq, const uint16_t* __restrict__ K, int64_t ldk,
    const uint16_t* __restrict__ V, int64_t ldv, uint16_t* __restrict__ O, int64_t ldo, int seq_len,
    int n_heads, int64_t n_hs, unsigned ways, unsigned members, int n_qblocks, float scale) {
#if defined(__HIP_DEVICE_COMPILE__)
  // two stages of one step's K and V, apart from each other so that the compiler sees that the loads into one do not
  // touch what is read from the other
  __shared__ __attribute__((aligned(1024))) unsigned char stage0[2 * kShortTile], stage1[2 * kShortTile];
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
  const int n_kt = last_q / kShortBk + 1;
  int wave_last_q = q0 + 31;
  if (wave_last_q > seq_len - 1) wave_last_q = seq_len - 1;
  // steps of this wave; none if it lies past the end: then it only helps to load
  const int n_mine = q0 <= wave_last_q ? wave_last_q / kShortBk + 1 : 0;

  // global -> LDS without registers: a wave-wide load fills four rows of 256 bytes, so the swizzle is on the global
  // side; a wave loads rows 8 wave + 4 i + lane / 16, i < 2, of K and of V.  Its descriptors begin at the first of
  // the eight rows and end with the sample: rows past it arrive as zeros (masked below).
  const int drow = lane >> 4, dch = lane & 15;
  const uint16_t* kn = K + (row0 + 8 * wave) * ldk + col0;     // of the next tile
  const uint16_t* vn = V + (row0 + 8 * wave) * ldv + col0;
  int left = seq_len - 8 * wave;                               // rows of the sample from there on
  auto fetch = [&](unsigned char* at) __attribute__((always_inline)) {
    unsigned char *ak = at + 2 * wave * 1024, *av = ak + kShortTile;
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
    kn += kShortBk * ldk;
    vn += kShortBk * ldv;
    left -= kShortBk;
  };
  const int kbase = l32 * kAttRow + ((h ^ (l32 & 15)) << 4);
  const int r4 = (lane & 15) >> 2, vg = (lane >> 4) & 1;
  const int vbase = (h * 4 + r4) * kAttRow + (((vg ^ h) << 1 | ((lane >> 1) & 1)) << 4) + (lane & 1) * 8;
  int ka[8], va[4];
#pragma unroll
  for (int st = 0; st < 8; ++st) ka[st] = kbase ^ (st << 5);
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) va[dt] = kShortTile + (vbase ^ ((dt ^ r4) << 6));

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
        const int key = kt * kShortBk + 8 * (v >> 2) + 4 * h + (v & 3);
        s[v] = key <= q ? s[v] : -INFINITY;
      }
    }
    float mx = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
    // key 0 is visible to every query and is part of the first step, so m_run becomes finite there; only the lanes
    // whose query meets a new maximum take part in the rescaling, elsewhere the factor is exactly 1
    float alpha = 1.0f;
    const float m_new = fmaxf(m_run, swap32_max(mx, mx));
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
  l_run += __shfl_xor(l_run, 32, 64);
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

// Where the 32-key form stays.  Up to two query blocks a sequence neither form is ahead (us, 32 keys a step -> 64: 32 x 100 x 16
// 12.1 -> 11.5, 32 x 100 x 32 19.7 -> 20.7, 32 x 200 x 16 22.5 -> 23.0).  A launch of at most one block a CU waits for latencies
// in both (4 x 300 x 6 10.8 -> 10.1, 8 x 512 x 8 17.0 -> 15.9): searches of a short chain of blocks decide near ties by the last
// bits of these outputs, and less than a microsecond does not pay for other ones.  Beyond, 3 - 13 %: 16 x 300 x 8 14.8 -> 13.1,
// 16 x 512 x 8 23.5 -> 20.5, 16 x 1024 x 8 50.8 -> 45.2.
static bool short_attention(int64_t n_hs, int n_qblocks) { return n_qblocks <= 2 || n_hs * n_qblocks <= 256; }

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
  const bool wide = ldk >= kAttWide || ldv >= kAttWide;
  auto go = [&](auto kern, double scale) {
    kern<<<grid, 256, 0, stream>>>((const uint16_t*)Q, ldq, (const uint16_t*)K, ldk, (const uint16_t*)V, ldv, (uint16_t*)O,
                                   ldo, seq_len, n_heads, n_hs, ways, members, n_qblocks, (float)scale);
  };
  auto pick = [&](auto t) {
    using T = decltype(t);
    const double scale = 0.08838834764831845, log2e = 1.4426950408889634;  // 1 / sqrt(128); the longer form takes powers of two
    if (short_attention(n_hs, n_qblocks)) wide ? go(short_attention_kernel<T, true>, scale) : go(short_attention_kernel<T, false>, scale);
    else wide ? go(causal_attention_kernel<T, true>, scale * log2e) : go(causal_attention_kernel<T, false>, scale * log2e);
  };
  bf16 ? pick(BF16{}) : pick(F16{});
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
