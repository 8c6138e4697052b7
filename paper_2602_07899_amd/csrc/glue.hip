// Glue of the synthetic sequential-calibration chain (not part of the paper's
// method): turns the quantised output of one linear into the exposed input of
// the next one (Sec. 3.2.1 PassAct2 feeds each layer the previous quantised
// layer's output; what sits between two linears of the synthetic stack is a
// row-wise RMS normalisation, an optional elementwise product of two branches
// and a fixed per-channel multiplier that re-imposes the outlier channels).
// HBM-bound, one wave per row.
#include <type_traits>

#include "common.h"

namespace tlq {

// out[t,c] = round16( v[t,c] / sqrt(mean_c v[t,:]^2 + 1e-6) * m(t)[c] ),
// v = Z (or Z * Zb elementwise); m(t) = m_a when (t % period) < split, else m_b.
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_mul_kernel(const uint16_t* __restrict__ Z, int64_t ldz,
                                                          const uint16_t* __restrict__ Zb, int64_t ldzb,
                                                          int64_t n_tok, int64_t c, const float* __restrict__ m_a,
                                                          const float* __restrict__ m_b, int period, int split,
                                                          uint16_t* __restrict__ out, int64_t ldo) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_tok) return;
  float ss = 0.0f;
  for (int64_t j = lane; j < c; j += 64) {
    float v = T::to_float(Z[row * ldz + j]);
    if (Zb) v *= T::to_float(Zb[row * ldzb + j]);
    ss += v * v;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off, 64);
  const float inv = 1.0f / sqrtf(ss / (float)c + 1e-6f);
  const float* m = (period > 0 && (int)(row % period) >= split) ? m_b : m_a;
  for (int64_t j = lane; j < c; j += 64) {
    float v = T::to_float(Z[row * ldz + j]);
    if (Zb) v *= T::to_float(Zb[row * ldzb + j]);
    out[row * ldo + j] = T::from_float(v * inv * (m ? m[j] : 1.0f));
  }
}

// The same for rows that can be read 16 bytes at a time (c % 8 == 0, aligned rows and factors, kVecWidth
// channels at least).  The sum of
// squares keeps the order of the kernel above - lane l adds elements l, l + 64, l + 128, ... - so that the
// results are bit-equal: each 512-element stretch goes through 1 KB of LDS and is picked up two bytes a
// lane.  Rows of up to 512 * HOLD elements stay in registers between the sum and the scaling (HOLD = 0: read
// again, from L2).  40960 x 4096 bf16: 454 -> 146 us (2-byte loads and stores, two passes before),
// 138 past the caches (NT loads, NTS stores).
constexpr int64_t kVecWidth = 72;
template <typename T, int HOLD, bool NT, bool NTS>
__global__ __launch_bounds__(256) void rmsnorm_mul_vec_kernel(const uint16_t* __restrict__ Z, int64_t ldz,
                                                              const uint16_t* __restrict__ Zb, int64_t ldzb,
                                                              int64_t n_tok, int64_t c, const float* __restrict__ m_a,
                                                              const float* __restrict__ m_b, int period, int split,
                                                              uint16_t* __restrict__ out, int64_t ldo) {
  __shared__ __attribute__((aligned(16))) uint16_t stage[4][2][512];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row = (int64_t)blockIdx.x * 4 + wave;
  if (row >= n_tok) return;
  const uint16_t* z = Z + row * ldz;
  const uint16_t* zb = Zb ? Zb + row * ldzb : nullptr;
  uint4 held[HOLD > 0 ? HOLD : 1];
  if constexpr (HOLD > 0) {
#pragma unroll
    for (int i = 0; i < HOLD; ++i) {
      held[i] = make_uint4(0, 0, 0, 0);
      if (i * 512 + lane * 8 < c) held[i] = load16<NT>(z + i * 512 + lane * 8);
    }
  }
  float ss = 0.0f;
  auto stretch = [&](int64_t j0, const uint4& v) {
    *reinterpret_cast<uint4*>(&stage[wave][0][lane * 8]) = v;
    if (zb) {
      uint4 u = make_uint4(0, 0, 0, 0);
      if (j0 + lane * 8 < c) u = *reinterpret_cast<const uint4*>(zb + j0 + lane * 8);
      *reinterpret_cast<uint4*>(&stage[wave][1][lane * 8]) = u;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (j0 + j * 64 + lane < c) {
        float x = T::to_float(stage[wave][0][j * 64 + lane]);
        if (zb) x *= T::to_float(stage[wave][1][j * 64 + lane]);
        ss += x * x;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();      // the next stretch overwrites what other lanes read here
  };
  if constexpr (HOLD > 0) {
#pragma unroll
    for (int i = 0; i < HOLD; ++i)
      if (i * 512 < c) stretch(i * 512, held[i]);
  } else {
    for (int64_t j0 = 0; j0 < c; j0 += 512) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (j0 + lane * 8 < c) v = *reinterpret_cast<const uint4*>(z + j0 + lane * 8);
      stretch(j0, v);
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off, 64);
  const float inv = 1.0f / sqrtf(ss / (float)c + 1e-6f);
  const float* m = (period > 0 && (int)(row % period) >= split) ? m_b : m_a;
  auto emit = [&](int64_t j, const uint4& v) {
    uint32_t u[4] = {v.x, v.y, v.z, v.w}, b[4] = {0, 0, 0, 0}, o[4] = {0, 0, 0, 0};
    if (zb) {
      const uint4 w = *reinterpret_cast<const uint4*>(zb + j);
      b[0] = w.x; b[1] = w.y; b[2] = w.z; b[3] = w.w;
    }
    float f[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = 1.0f;
    if (m) {
      const float4 m0 = *reinterpret_cast<const float4*>(m + j), m1 = *reinterpret_cast<const float4*>(m + j + 4);
      f[0] = m0.x; f[1] = m0.y; f[2] = m0.z; f[3] = m0.w; f[4] = m1.x; f[5] = m1.y; f[6] = m1.z; f[7] = m1.w;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float x = T::to_float((uint16_t)(u[e >> 1] >> ((e & 1) * 16)));
      if (zb) x *= T::to_float((uint16_t)(b[e >> 1] >> ((e & 1) * 16)));
      o[e >> 1] |= (uint32_t)T::from_float(x * inv * f[e]) << ((e & 1) * 16);
    }
    store16<NTS>(out + row * ldo + j, make_uint4(o[0], o[1], o[2], o[3]));
  };
  if constexpr (HOLD > 0) {
#pragma unroll
    for (int i = 0; i < HOLD; ++i)
      if (i * 512 + lane * 8 < c) emit(i * 512 + lane * 8, held[i]);
  } else {
    for (int64_t j = lane * 8; j < c; j += 512) emit(j, *reinterpret_cast<const uint4*>(z + j));
  }
}

hipError_t launch_rmsnorm_mul(const void* Z, int64_t ldz, const void* Zb, int64_t ldzb, int64_t n_tok,
                              int64_t c, bool bf16, const float* m_a, const float* m_b, int period,
                              int split, void* out, int64_t ldo, hipStream_t stream) {
  ProfScope ps("rmsnorm_mul", stream, (Zb ? 6.0 : 4.0) * (double)n_tok * (double)c);
  const unsigned grid = (unsigned)ceil_div(n_tok, 4);
  auto al = [](const void* p) { return ((uintptr_t)p % 16) == 0; };   // (NULL counts as aligned)
  // (up to 64 channels an element-wise lane has one value, and the 16-byte form leaves most lanes idle: us element-wise and
  // 16-byte, 1,000,000 x 8 201 and 262, 300,000 x 64 65 and 81, 250,000 x 72 71 and 69, with Zb 94 and 81)
  const bool vec = c >= kVecWidth && (c % 8) == 0 && (ldz % 8) == 0 && (ldo % 8) == 0 && (!Zb || (ldzb % 8) == 0) && al(Z) && al(Zb) &&
                   al(out) && al(m_a) && al(m_b);
  auto go = [&](auto kern) {
    kern<<<grid, 256, 0, stream>>>((const uint16_t*)Z, ldz, (const uint16_t*)Zb, ldzb, n_tok, c, m_a, m_b, period,
                                   split, (uint16_t*)out, ldo);
  };
  auto pick = [&](auto t) {
    using T = decltype(t);
    auto vec_of = [&](auto nt_c, auto nts_c) {
      constexpr bool NT = decltype(nt_c)::value, NTS = decltype(nts_c)::value;
      if (c <= 1024) go(rmsnorm_mul_vec_kernel<T, 2, NT, NTS>);
      else if (c <= 5120) go(rmsnorm_mul_vec_kernel<T, 10, NT, NTS>);
      else go(rmsnorm_mul_vec_kernel<T, 0, NT, NTS>);
    };
    if (!vec) go(rmsnorm_mul_kernel<T>);
    else if (!streams_past((Zb ? 6.0 : 4.0) * (double)n_tok * (double)c)) vec_of(std::false_type{}, std::false_type{});
    else if (!outgrows_cache(2.0 * (double)n_tok * (double)c)) vec_of(std::true_type{}, std::false_type{});
    else vec_of(std::true_type{}, std::true_type{});
  };
  if (!bf16) pick(F16{}); else pick(BF16{});
  return hipGetLastError();
}

}  // namespace tlq
