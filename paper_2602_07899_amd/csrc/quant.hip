// S2: group-wise fake quantisation of W * diag(s) (Sec. 2.2 quantiser in its
// min/max form; Sec. 3.2.1 Q_w(W * scale)).
//
// This file is compiled with floating-point contraction off: every float
// operation below rounds exactly once, in the order written, so the integer
// codes, zero points and steps are reproducible bit for bit.
//
// One pass reads W once and emits the operands of ALL candidates of the
// search: per candidate k the folded 16-bit matrix  What_k = deq_k / s_k  that
// the contraction kernel multiplies with the *unscaled* tokens (the smoothing
// identity of Sec. 2.2 moves diag(s)^-1 from X onto the dequantised weights).
// HBM traffic per weight element: 2 B read + 2 B written per candidate.
#include <type_traits>

#include "common.h"

namespace tlq {

struct QuantDev {
  const uint16_t* W; int64_t c_out, c_in, ldw;
  float qmax, qlo, qhi; int half;  // asym: codes in [0,qmax]; sym: q in [qlo,qhi], half = 2^(bits-1)
  float rq;                        // fl(1 / qmax) or fl(1 / qhi)
  int64_t group;                   // resolved group size (>= 8)
  const float* s_table; const float* inv_table; int n_cand;
  int cand_step;                   // candidates per block (blockIdx.y picks the stretch)
  uint16_t* what; int64_t what_cand_stride;
  uint8_t* codes; uint8_t* zp; float* delta; uint16_t* wdq; int64_t ld_dq;
  bool diff; const uint32_t* xmax_bits;  // what = deq*inv - W*2^shift
  const float* col_scale;                // [c_in] factor on `what` or NULL
  int shift; bool packed;                // quant_pow2_kernel: log2 of a group's lanes; groups that leave lanes over
  int8_t* w8; int64_t ld8, w8_cand_stride; float* steps; int64_t step_stride;   // Q_INT
  bool nt;                               // the operands of all candidates stream past the caches
};

// What a launch writes: the folded operands of the candidates, their difference form, or the
// single-candidate outputs (codes, zero points, steps, dequantised weights), or the candidates' integer codes less
// their zero points (int8) and steps.
enum { Q_FOLD = 0, Q_DIFF = 1, Q_AUX = 2, Q_INT = 3 };

// Grid of one group: step, an approximate reciprocal, zero point, and how near to a tie the reciprocal may be used.
struct Grid { float delta, rd, zpf, lim; };

// The integer codes need rint(fl(x / delta)).  With rd within one ulp of 1/delta, t = fl(x * rd) lies
// within 2.4e-7 |t| of the rounded quotient, so rint(t) is that integer unless a half-integer sits inside
// the gap; |t - rint(t)| < lim = 0.49999976 - 4.8e-7 max|t| rules that out for a whole group (with a factor of two to
// spare), and the rare rest (one element in 10^5 at 4 bits) is divided, eight elements at a time.
// Outside [1e-5, 1e36) and for NaN lim is negative or NaN: everything is divided.
template <bool SYM>
__device__ __forceinline__ Grid make_grid(float mx, float mn, const QuantDev& a, float& tie) {
  Grid g;
  const float rng = fmaxf(SYM ? mx : mx - mn, kRangeFloor);
  const float dv = SYM ? a.qhi : a.qmax;
  // range / (2^b - 1) by a correction step on range * fl(1 / (2^b - 1)): equal to the division for every significand and
  // all eight divisors (checked exhaustively)
  const float q0 = rng * a.rq;
  g.delta = __builtin_fmaf(__builtin_fmaf(-q0, dv, rng), a.rq, q0);
  g.rd = __builtin_amdgcn_rcpf(g.delta);
  const float top = (SYM ? mx : __builtin_amdgcn_fmed3f(mx, -mn, __builtin_inff())) * g.rd;     // (the larger of the two)
  g.lim = rng < 1e36f ? __builtin_fmaf(top, -4.8e-7f, 0.49999976f) : -1.0f;
  if (SYM) {
    g.zpf = (float)a.half;
    tie = 0.0f;
  } else {
    const float t = -mn * g.rd, z = rintf(t);
    tie = fabsf(t - z);
    g.zpf = __builtin_amdgcn_fmed3f(z, 0.0f, a.qmax);
  }
  return g;
}
// the same with divisions
template <bool SYM>
__device__ __forceinline__ void divide_grid(float mx, float mn, const QuantDev& a, Grid& g) {
  const float rng = fmaxf(SYM ? mx : mx - mn, kRangeFloor);
  if (!(rng < 1e36f)) g.delta = rng / (SYM ? a.qhi : a.qmax);
  if (!SYM) g.zpf = fminf(fmaxf(rintf(-mn / g.delta), 0.0f), a.qmax);
}
template <bool SYM>
__device__ __forceinline__ Grid grid_of(float mx, float mn, const QuantDev& a) {
  float tie;
  Grid g = make_grid<SYM>(mx, mn, a, tie);
  if (!(tie < g.lim)) divide_grid<SYM>(mx, mn, a, g);
  return g;
}

// rint(fl(ws / delta)) of eight values unless the result, or `tie` from before, reaches lim; the larger of the two measures
__device__ __forceinline__ float rint_quotient8(const float (&ws)[8], const Grid& g, float tie, float (&n)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float t = ws[j] * g.rd;
    n[j] = rintf(t);
    tie = fmaxf(tie, fabsf(t - n[j]));
  }
  return tie;
}
__device__ __forceinline__ void divide8(const float (&ws)[8], const Grid& g, float (&n)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    n[j] = rintf(ws[j] / g.delta);
    asm volatile("" : "+v"(n[j]) :: "memory");     // one after the other, and in a branch, not computed and dropped
  }
}

__device__ __forceinline__ void load8(const float* __restrict__ p, float (&v)[8]) {
  const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
template <typename T>
__device__ __forceinline__ void widen8(const uint4& v, float (&w)[8]) {
  const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int j = 0; j < 8; ++j) w[j] = T::to_float((uint16_t)(u[j >> 1] >> ((j & 1) * 16)));
}
__device__ __forceinline__ void times8(const float (&w)[8], const float (&s)[8], float (&ws)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) ws[j] = w[j] * s[j];
}
// what is worked out from v is worked out again, not held in registers from before
__device__ __forceinline__ void anew(uint4& v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w)); }
template <bool SYM>
__device__ __forceinline__ void range8(const float (&ws)[8], float& mx, float& mn) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    mx = fmaxf(mx, SYM ? fabsf(ws[j]) : ws[j]);
    if (!SYM) mn = fminf(mn, ws[j]);
  }
}

// two floats rounded to fp16 (one instruction; bit-equal to two conversions for all 2^32 floats)
__device__ __forceinline__ uint32_t pack_f16(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), f16x2));
}
// four small integers as bytes: beside 1.5 * 2^23 the low byte of the float is the integer's
__device__ __forceinline__ uint32_t pack_i8(float a, float b, float c, float d) {
  auto bits = [](float v) { return __builtin_bit_cast(uint32_t, v + 12582912.0f); };
  return __builtin_amdgcn_perm(bits(b), bits(a), 0x0c0c0400u) | __builtin_amdgcn_perm(bits(d), bits(c), 0x04000c0cu);
}

// Eight quantised values of row `row`, channels c .. c+7 go to memory (`what`: their place in the operand).
template <typename T, bool SYM, int MODE>
__device__ __forceinline__ void emit8(const QuantDev& a, const Grid& g, const float (&w)[8], float (&n)[8],
                                      const float (&inv)[8], const float (&cs)[8], float wsub, uint16_t* what,
                                      int64_t row, int64_t c) {
  uint32_t hw[4] = {0, 0, 0, 0}, cw[2] = {0, 0};
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if constexpr (MODE == Q_AUX) {
      float code, deq;
      if (!SYM) {
        code = fminf(fmaxf(n[j] + g.zpf, 0.0f), a.qmax);
        deq = (code - g.zpf) * g.delta;
      } else {
        const float q = fminf(fmaxf(n[j], a.qlo), a.qhi);
        code = q + g.zpf;
        deq = q * g.delta;
      }
      // deq is rounded to float before it is rounded to 16 bits: keep the product and the conversion from
      // becoming one mixed-precision instruction, which rounds once
      asm("" : "+v"(deq));
      cw[j >> 2] |= ((uint32_t)code & 0xffu) << ((j & 3) * 8);
      hw[j >> 1] |= (uint32_t)T::from_float(deq) << ((j & 1) * 16);
    } else {
      // (clip(n + zp, 0, qmax) - zp) of small integers is clip(n, -zp, qmax - zp)
      const float lo = SYM ? a.qlo : -g.zpf, hi = SYM ? a.qhi : a.qmax - g.zpf;
      // (a NaN weight quantises to `lo` like in the two-step clip)
      if constexpr (MODE == Q_INT) { n[j] = __builtin_amdgcn_fmed3f(n[j], lo, hi); continue; }
      float f = __builtin_amdgcn_fmed3f(n[j], lo, hi) * g.delta * inv[j];
      if constexpr (MODE == Q_DIFF) {
        f -= w[j] * wsub;
        f *= cs[j];
      } else {
        asm("" : "+v"(f));               // rounded to float, then to 16 bits (see above)
      }
      n[j] = f;
    }
  }
  if constexpr (MODE == Q_INT) {
    store8(what, pack_i8(n[0], n[1], n[2], n[3]), pack_i8(n[4], n[5], n[6], n[7]), a.nt);
    return;
  }
  if constexpr (MODE != Q_AUX) {
#pragma unroll
    for (int j = 0; j < 4; ++j) hw[j] = pack_f16(n[2 * j], n[2 * j + 1]);
  }
  const uint4 out = make_uint4(hw[0], hw[1], hw[2], hw[3]);
  if constexpr (MODE == Q_AUX) {
    if (a.codes) *reinterpret_cast<uint2*>(a.codes + row * a.c_in + c) = make_uint2(cw[0], cw[1]);
    if (a.wdq) *reinterpret_cast<uint4*>(a.wdq + row * a.ld_dq + c) = out;
  } else {
    store16(what, out, a.nt);
  }
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
// maximum (MAX) or minimum over aligned runs of `lanes` lanes (a power of two); every lane gets it.  Up to
// 16 lanes stay inside a DPP row: quad permutes, then the mirrors of 8 and 16 lanes.
template <bool MAX>
__device__ __forceinline__ float lanes_reduce(float v, int lanes) {
  auto op = [](float x, float y) { return MAX ? fmaxf(x, y) : fminf(x, y); };
  if (lanes >= 2) v = op(v, dpp<0xB1>(v));
  if (lanes >= 4) v = op(v, dpp<0x4E>(v));
  if (lanes >= 8) v = op(v, dpp<0x141>(v));
  if (lanes >= 16) v = op(v, dpp<0x140>(v));
  if (lanes >= 32) v = op(v, __shfl_xor(v, 16, 64));
  if (lanes >= 64) v = op(v, __shfl_xor(v, 32, 64));
  return v;
}

// mx and mn of R rows over 16 lanes each, every lane gets them.  In assembly: the exchange is part of the maximum
// (the compiler moves first and then makes sure that the moved value is no signalling NaN, three instructions for one);
// a value is read by another lane's instruction two wait states behind its write at the earliest.
template <bool SYM, int R>
__device__ __forceinline__ void row_ranges(float (&mx)[R], float (&mn)[R]) {
#define TLQ_STEP(op, reg, how) "v_" op "_f32_dpp %" reg ", %" reg ", %" reg " " how " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
#define TLQ_FOUR(m) m("quad_perm:[1,0,3,2]") m("quad_perm:[2,3,0,1]") m("row_half_mirror") m("row_mirror")
  if constexpr (R == 2 && !SYM) {
#define TLQ_ALL(how) TLQ_STEP("max", "0", how) TLQ_STEP("min", "1", how) TLQ_STEP("max", "2", how) TLQ_STEP("min", "3", how)
    asm("s_nop 1\n\t" TLQ_FOUR(TLQ_ALL) : "+v"(mx[0]), "+v"(mn[0]), "+v"(mx[1]), "+v"(mn[1]));
#undef TLQ_ALL
  } else if constexpr (R == 2) {
#define TLQ_ALL(how) TLQ_STEP("max", "0", how) TLQ_STEP("max", "1", how) "s_nop 0\n\t"
    asm("s_nop 1\n\t" TLQ_FOUR(TLQ_ALL) : "+v"(mx[0]), "+v"(mx[1]));
#undef TLQ_ALL
  } else if constexpr (!SYM) {
#define TLQ_ALL(how) TLQ_STEP("max", "0", how) TLQ_STEP("min", "1", how) "s_nop 0\n\t"
    asm("s_nop 1\n\t" TLQ_FOUR(TLQ_ALL) : "+v"(mx[0]), "+v"(mn[0]));
#undef TLQ_ALL
  } else {
#define TLQ_ALL(how) TLQ_STEP("max", "0", how) "s_nop 1\n\t"
    asm("s_nop 1\n\t" TLQ_FOUR(TLQ_ALL) : "+v"(mx[0]));
#undef TLQ_ALL
  }
#undef TLQ_FOUR
#undef TLQ_STEP
}

__device__ __forceinline__ float diff_factor(const QuantDev& a) {
  return a.xmax_bits ? __builtin_ldexpf(1.0f, shift_from_bf16_bits(*a.xmax_bits)) : 1.0f;
}

// Groups of a power of two up to 512, and any below 64.  A lane owns 8 consecutive input channels of R rows, a
// group is `group/8` adjacent lanes and a wave covers 512 channels; W stays in registers while the candidates
// are walked, a candidate's scales are loaded once for the R rows.  `packed`: the lanes of a group are rounded up
// to a power of two (the spare ones repeat the group's first channels and store nothing) and the groups of all
// rows fill the waves one after the other.  Bound by vector ALU issue and by what stores reach: 99 vector instructions per
// 512 weights and candidate (135 with a branch and a tie measure with |t| per element, three branches a row, lane exchanges
// apart from the maxima, two conversions and an OR per pair), and five candidates a wave (see launch_quant).  20
// candidates of 4096 x 4096 (0.7 GB written): 171 -> 142 us (4.7 TB/s), of 4096 x 11008 488 -> 398, of 13824 x 5120 757 ->
// 650; difference form of 5120 x 5120 335 -> 256.  LPG > 0 fixes the group at compile time (16 lanes: the usual 128).
// Groups of 24, 40 and 56 of 4096 x 4100 with every output, a wave per group -> this way: 252 -> 22, 153 -> 26, 111 -> 20 us.
template <typename T, bool SYM, int MODE, int R, int LPG>
__global__ __launch_bounds__(256) void quant_pow2_kernel(QuantDev a) {
  // Rows of a wave side by side: both where the lanes of a group are known; elsewhere one after the other, in 64 - 67 registers instead of
  // 83 - 87, difference form 91 and 111 (a search of 4 candidates, us together -> apart: 4096 x 4080 in groups of 40 103.5 -> 97.6, of 256 86.1 -> 81.7; of 20
  // 0.6 - 3.5 % in the mean of five sizes)
  constexpr int B = LPG == 16 ? R : 1;
  const int lane = threadIdx.x & 63;
  // (32 bits: a wave has 512 weights, and no memory holds 2^41)
  const uint32_t wave = blockIdx.x * 4u + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lpg = LPG > 0 ? LPG : 1 << a.shift;
  int64_t row0;                    // the same for the whole wave unless groups are packed
  uint32_t c;
  bool valid, active;              // the lane's channels exist; it also stores them
  if (LPG == 0 && a.packed) {
    const uint32_t groups = (uint32_t)(a.c_in / a.group);
    const uint32_t unit = wave * (64u >> a.shift) + (uint32_t)(lane >> a.shift);   // (row, group), flat
    const int chunk = lane & (lpg - 1);
    const bool spare = chunk * 8 >= a.group;
    row0 = (int64_t)(unit / groups) * R;
    c = unit % groups * (uint32_t)a.group + (spare ? 0 : chunk * 8);
    valid = row0 < a.c_out;
    active = valid && !spare;
  } else {
    const uint32_t cblocks = ((uint32_t)a.c_in + 511) / 512, rb = wave / cblocks;
    row0 = (int64_t)rb * R;
    if (row0 >= a.c_out) return;
    c = (wave - rb * cblocks) * 512 + lane * 8;
    valid = active = c < (uint32_t)a.c_in;
  }
  if (!valid) { row0 = 0; c = 0; }       // (reads what is there, stores nothing)

  float w[R][8];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t row = row0 + r < a.c_out ? row0 + r : row0;
    widen8<T>(*reinterpret_cast<const uint4*>(a.W + row * a.ldw + c), w[r]);
  }
  const float wsub = MODE == Q_DIFF ? diff_factor(a) : 0.0f;
  float s[8], inv[8], cs[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) { s[j] = 1.0f; inv[j] = 1.0f; cs[j] = 1.0f; }
  if (MODE == Q_DIFF && a.col_scale) load8(a.col_scale + c, cs);
  const int k0 = (int)blockIdx.y * a.cand_step;
  const int k1 = k0 + a.cand_step < a.n_cand ? k0 + a.cand_step : a.n_cand;
  const float* ps = a.s_table ? a.s_table + (int64_t)k0 * a.c_in : nullptr;
  const float* pi = MODE != Q_AUX && a.inv_table ? a.inv_table + (int64_t)k0 * a.c_in : nullptr;
  uint16_t* out = MODE != Q_AUX ? a.what + (int64_t)k0 * a.what_cand_stride : nullptr;
#pragma unroll 1
  for (int k = k0; k < k1; ++k) {
    if (ps) { load8(ps + c, s); ps += a.c_in; }
    if (pi) { load8(pi + c, inv); pi += a.c_in; }
    // B rows side by side, with one branch for what has to be divided in any of them
#pragma unroll
    for (int b = 0; b < R; b += B) {
      float n[B][8], mx[B], mn[B];
      Grid g[B];
#pragma unroll
      for (int r = 0; r < B; ++r) {
        mx[r] = SYM ? 0.0f : -__builtin_inff();
        mn[r] = __builtin_inff();
        times8(w[b + r], s, n[r]);
        range8<SYM>(n[r], mx[r], mn[r]);
      }
      if constexpr (LPG == 16) {
        row_ranges<SYM, B>(mx, mn);
      } else {
#pragma unroll
        for (int r = 0; r < B; ++r) {
          mx[r] = lanes_reduce<true>(mx[r], lpg);
          if (!SYM) mn[r] = lanes_reduce<false>(mn[r], lpg);
        }
      }
      bool near = false;
#pragma unroll
      for (int r = 0; r < B; ++r) {
        float tie;
        g[r] = make_grid<SYM>(mx[r], mn[r], a, tie);
        near |= !(rint_quotient8(n[r], g[r], tie, n[r]) < g[r].lim);
      }
      if (near) {
#pragma unroll
        for (int r = 0; r < B; ++r) {
          divide_grid<SYM>(mx[r], mn[r], a, g[r]);
          times8(w[b + r], s, n[r]);
          divide8(n[r], g[r], n[r]);
        }
      }
      if (active) {
#pragma unroll
        for (int r = 0; r < B; ++r) {
          const int64_t row = row0 + b + r;
          if (row >= a.c_out) break;
          emit8<T, SYM, MODE>(a, g[r], w[b + r], n[r], inv, cs, wsub, MODE != Q_AUX ? out + row * a.c_in + c : nullptr, row, c);
          if (MODE == Q_AUX && (lane & (lpg - 1)) == 0) {
            const int64_t gidx = row * (a.c_in / a.group) + c / a.group;
            if (a.zp) a.zp[gidx] = (uint8_t)g[r].zpf;
            if (a.delta) a.delta[gidx] = g[r].delta;
          }
        }
      }
    }
    if (MODE != Q_AUX) out += a.what_cand_stride;
  }
}

// Any other group of up to 16384 channels, whole rows among them: NWG waves (1 or 4) own one group of R
// rows, a lane CH chunks of 8 channels, `64 NWG` chunks apart.  The weights stay packed in registers; times a
// candidate's scales they stay there from the range to the codes where two rows (or one of four chunks) fit, elsewhere they are
// worked out twice.  Bound like the above; the registers decide how many waves there are (widened weights and column factors
// that the compiler held through all candidates took 100 - 200 of them).  us, group = row, 20 candidates: 4096 x 4096 as int8
// 131 -> 107, 5120 x 5120 290 -> 237; 12 candidates' differences of 1400 x 1096 31 -> 25; 16 candidates of 3000 x 13824 412
// -> 383, as int8 of 3000 x 12288 265 -> 245.
template <typename T, bool SYM, int MODE, int NWG, int CH, int R>
__global__ __launch_bounds__(256) void quant_row_kernel(QuantDev a) {
  __shared__ float red[2][4][2 * R];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t G = (uint32_t)(a.c_in / a.group);             // (32 bits: no memory holds 2^32 units of groups)
  const uint32_t unit = NWG == 4 ? blockIdx.x : blockIdx.x * 4u + (uint32_t)wv;
  const int64_t row0 = (int64_t)(unit / G) * R;
  const uint32_t gi = unit % G;
  if (NWG == 1 && row0 >= a.c_out) return;
  const uint32_t group = (uint32_t)a.group, cg = gi * group;
  const uint32_t cl = ((NWG == 4 ? wv * 64 : 0) + lane) * 8;   // channel of chunk 0 inside the group
  constexpr uint32_t STEP = (uint32_t)NWG * 512;
  // the weights times the scales stay in registers between the two sweeps where they fit, and are worked out twice elsewhere
  constexpr bool KEEP = R * CH <= 4;
  constexpr bool ANEW = KEEP || CH > 4 || MODE != Q_FOLD;     // (the widened weights of four chunks and two rows fit beside the rest)
  // chunk i of the lane; past the group's end its first channels again, which change no range and are not stored; a wave
  // of which nothing is left skips the chunk
  auto chunk = [&](int i) { return cl + i * STEP < group ? cl + i * STEP : 0u; };
  auto some = [&](int i) { return (NWG == 4 ? wv * 512u : 0u) + i * STEP < group; };

  uint4 wp[R][CH];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t row = row0 + r < a.c_out ? row0 + r : row0;
#pragma unroll
    for (int i = 0; i < CH; ++i) wp[r][i] = *reinterpret_cast<const uint4*>(a.W + row * a.ldw + cg + chunk(i));
  }
  const float wsub = MODE == Q_DIFF ? diff_factor(a) : 0.0f;
  float s[8], inv[8], cs[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) { s[j] = 1.0f; inv[j] = 1.0f; cs[j] = 1.0f; }
  const int k0 = (int)blockIdx.y * a.cand_step;
  const int k1 = k0 + a.cand_step < a.n_cand ? k0 + a.cand_step : a.n_cand;
#pragma unroll 1
  for (int k = k0; k < k1; ++k) {
    const float* ps = a.s_table ? a.s_table + (int64_t)k * a.c_in + cg : nullptr;
    const float* pi = MODE < Q_AUX && a.inv_table ? a.inv_table + (int64_t)k * a.c_in + cg : nullptr;
    float n[KEEP ? R : 1][KEEP ? CH : 1][8], mx[R], mn[R];
#pragma unroll
    for (int r = 0; r < R; ++r) { mx[r] = SYM ? 0.0f : -__builtin_inff(); mn[r] = __builtin_inff(); }
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      __builtin_amdgcn_sched_barrier(0);     // (not all chunks' scales at once)
      if (!some(i)) continue;
      if (ps) load8(ps + chunk(i), s);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        float w[8], (&ws)[8] = n[KEEP ? r : 0][KEEP ? i : 0];
        if (ANEW) anew(wp[r][i]);
        widen8<T>(wp[r][i], w);
        times8(w, s, ws);
        range8<SYM>(ws, mx[r], mn[r]);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      mx[r] = lanes_reduce<true>(mx[r], 64);
      if (!SYM) mn[r] = lanes_reduce<false>(mn[r], 64);
    }
    if constexpr (NWG == 4) {
      // two buffers: the next candidate's writes cannot overtake this one's reads past one barrier
      float* rb = &red[k & 1][0][0];
      if (lane == 0)
#pragma unroll
        for (int r = 0; r < R; ++r) { rb[wv * 2 * R + 2 * r] = mx[r]; rb[wv * 2 * R + 2 * r + 1] = mn[r]; }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          mx[r] = fmaxf(mx[r], rb[v * 2 * R + 2 * r]);
          if (!SYM) mn[r] = fminf(mn[r], rb[v * 2 * R + 2 * r + 1]);
        }
    }
    Grid g[R];
#pragma unroll
    for (int r = 0; r < R; ++r) g[r] = grid_of<SYM>(mx[r], mn[r], a);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      const bool in = cl + i * STEP < group;
      const uint32_t c = cg + chunk(i);
      if (MODE != Q_INT && !some(i)) continue;     // (the integer rows have zeros behind the last channel)
      if (!KEEP && ps) load8(ps + chunk(i), s);
      if (pi) load8(pi + chunk(i), inv);
      if (MODE == Q_DIFF && a.col_scale) load8(a.col_scale + c, cs);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        float w[8], (&q)[8] = n[KEEP ? r : 0][KEEP ? i : 0];
        if (MODE != Q_INT || some(i)) {
          if (!KEEP) {
            if (ANEW) anew(wp[r][i]);
            widen8<T>(wp[r][i], w);
            times8(w, s, q);
          }
          if (!(rint_quotient8(q, g[r], 0.0f, q) < g[r].lim)) {
            if (KEEP && ps) load8(ps + chunk(i), s);
            anew(wp[r][i]);
            widen8<T>(wp[r][i], w);
            times8(w, s, q);
            divide8(q, g[r], q);
          }
          if (MODE == Q_DIFF && (KEEP || ANEW)) { anew(wp[r][i]); widen8<T>(wp[r][i], w); }
        }
        if (row0 + r >= a.c_out) continue;
        if (MODE == Q_INT) {               // (the group is the row)
          int8_t* at = a.w8 + (int64_t)k * a.w8_cand_stride + (row0 + r) * a.ld8 + cl + i * STEP;
          if (in) emit8<T, SYM, MODE>(a, g[r], w, q, inv, cs, wsub, (uint16_t*)at, row0 + r, c);
          else if (cl + i * STEP < a.ld8) *reinterpret_cast<uint2*>(at) = make_uint2(0, 0);
        } else if (in) {
          emit8<T, SYM, MODE>(a, g[r], w, q, inv, cs, wsub,
                              MODE != Q_AUX ? a.what + (int64_t)k * a.what_cand_stride + (row0 + r) * a.c_in + c : nullptr, row0 + r, c);
        }
      }
    }
    if (MODE == Q_INT && cl == 0) {
      // an infinite weight gives an infinite step, and the finite weights beside it 0 times infinity: NaN, which the
      // integers cannot carry
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (row0 + r < a.c_out)
          a.steps[(int64_t)k * a.step_stride + row0 + r] = g[r].delta < __builtin_inff() ? g[r].delta : __builtin_nanf("");
    }
    if (MODE == Q_AUX && cl == 0) {
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (row0 + r < a.c_out) {
          if (a.zp) a.zp[(row0 + r) * G + gi] = (uint8_t)g[r].zpf;
          if (a.delta) a.delta[(row0 + r) * G + gi] = g[r].delta;
        }
    }
  }
}

// Groups beyond 16384 channels: one wave per (row, group), two sweeps over the group per candidate.
template <typename T, bool SYM, int MODE>
__global__ __launch_bounds__(256) void quant_any_kernel(QuantDev a) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t G = a.c_in / a.group;
  if (wave >= a.c_out * G) return;
  const int64_t row = wave / G;
  const int64_t c0 = (wave % G) * a.group;
  const float wsub = MODE == Q_DIFF ? diff_factor(a) : 0.0f;
  float s[8], inv[8], cs[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) { s[j] = 1.0f; inv[j] = 1.0f; cs[j] = 1.0f; }
  for (int k = 0; k < a.n_cand; ++k) {
    const float* sk = a.s_table ? a.s_table + (int64_t)k * a.c_in : nullptr;
    float mx = SYM ? 0.0f : -__builtin_inff(), mn = __builtin_inff();
    for (int64_t c = c0 + lane * 8; c < c0 + a.group; c += 512) {
      float ws[8];
      widen8<T>(*reinterpret_cast<const uint4*>(a.W + row * a.ldw + c), ws);
      if (sk) load8(sk + c, s);
#pragma unroll
      for (int j = 0; j < 8; ++j) ws[j] *= s[j];
      range8<SYM>(ws, mx, mn);
    }
    mx = lanes_reduce<true>(mx, 64);
    if (!SYM) mn = lanes_reduce<false>(mn, 64);
    const Grid g = grid_of<SYM>(mx, mn, a);
    for (int64_t c = c0 + lane * 8; c < c0 + a.group; c += 512) {
      float w[8], ws[8], n[8];
      widen8<T>(*reinterpret_cast<const uint4*>(a.W + row * a.ldw + c), w);
      if (sk) load8(sk + c, s);
      if (MODE != Q_AUX && a.inv_table) load8(a.inv_table + (int64_t)k * a.c_in + c, inv);
      if (MODE == Q_DIFF && a.col_scale) load8(a.col_scale + c, cs);
#pragma unroll
      for (int j = 0; j < 8; ++j) ws[j] = w[j] * s[j];
      if (!(rint_quotient8(ws, g, 0.0f, n) < g.lim)) divide8(ws, g, n);
      emit8<T, SYM, MODE>(a, g, w, n, inv, cs, wsub,
                          MODE != Q_AUX ? a.what + (int64_t)k * a.what_cand_stride + row * a.c_in + c : nullptr, row, c);
    }
    if (MODE == Q_AUX && lane == 0) {
      if (a.zp) a.zp[wave] = (uint8_t)g.zpf;
      if (a.delta) a.delta[wave] = g.delta;
    }
  }
}

// ---------------------------------------------------------------------------
// Q_a (Sec. 3.2.1 f_q; quantiser of Sec. 2.2 applied per token row):
//   xt = x * inv ; sigma = max(max_c |xt|, 1e-5) / (2^(n-1) - 1) ;
//   code = clip(rint(xt / sigma), -2^(n-1), 2^(n-1) - 1).
// A block owns eight rows, its waves strips of 512 channels.  A strip's tile (8 rows x 8 channels a lane) stays in
// registers for all candidates: first the row maxima of every candidate, which meet in LDS, then, with the tile
// read again (from cache), the codes.  Bound by vector ALU issue, 7 - 8 instructions an element and candidate.  The codes are
// fp16 integers (exact), so the contraction runs on the same MFMA path and the per-token step is applied to the
// accumulators in its epilogue.
// Four launches (maxima through shuffles and global atomics, one tie branch per element) -> one: one candidate
// of 3678 x 4096 24.0 -> 13.5 us, 128 x 4096 15.2 -> 6.2, 2000 x 13824 51 -> 30, 1000000 x 8 301 -> 164; 20 candidates of
// 3678 x 4096 250 -> 170 us (the 0.6 GB of codes at 3.5 TB/s); as int8 117 -> 105 with bytes cut out of biased floats.
constexpr int kAqRows = 8;      // rows per block
constexpr int kAqCols = 512;    // channels per strip (64 lanes x 8)
constexpr int kAqWaves = 8;     // waves per block at most
constexpr int kAqStep = 32;     // candidates per block at most (32 KB of LDS for their maxima)

template <typename T>
__device__ __forceinline__ void aq_load_tile(const uint16_t* __restrict__ X, int64_t n_tok, int64_t c_in,
                                             int64_t ldx, int64_t r0, int64_t c, float (&x)[kAqRows][8]) {
#pragma unroll
  for (int r = 0; r < kAqRows; ++r) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (r0 + r < n_tok && c < c_in) v = *reinterpret_cast<const uint4*>(X + (r0 + r) * ldx + c);
    widen8<T>(v, x[r]);
  }
}

// INT: int8 codes in rows of ldc bytes (zeros behind c_in) instead of fp16 ones in rows of c_in.
template <typename T, bool INT>
__global__ __launch_bounds__(kAqWaves * 64) void act_quant_kernel(const uint16_t* __restrict__ X, int64_t n_tok, int64_t c_in,
                                                                  int64_t ldx, const float* __restrict__ inv_table,
                                                                  int nb, int cand_step, float qa, float* __restrict__ sig,
                                                                  uint16_t* __restrict__ codes, int64_t ldc, bool nt) {
  extern __shared__ __attribute__((aligned(16))) float part[];   // [4 quarter waves of every wave][candidate][row]
  __shared__ __attribute__((aligned(16))) float step[kAqStep][kAqRows];
  const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t r0 = (int64_t)blockIdx.x * kAqRows;
  const int k0 = (int)blockIdx.y * cand_step;
  const int nk = nb - k0 < cand_step ? nb - k0 : cand_step;
  const int strips = (int)((c_in + kAqCols - 1) / kAqCols);
  float x[kAqRows][8], iv[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) iv[j] = 1.0f;

  const bool b0 = lane & 1, b1 = lane & 2;
  // (lanes 4 .. 15 of a quarter end up with copies of what lanes 0 .. 3 hold)
  float* mine = part + (wave * 4 + (lane >> 4)) * cand_step * kAqRows + (b0 ? 4 : 0) + (b1 ? 2 : 0);
  for (int strip = wave; strip < strips; strip += nw) {
    const int64_t c = (int64_t)strip * kAqCols + lane * 8;
    aq_load_tile<T>(X, n_tok, c_in, ldx, r0, c, x);
    for (int k = 0; k < nk; ++k) {
      if (inv_table && c < c_in) load8(inv_table + (int64_t)(k0 + k) * c_in + c, iv);
      float m[kAqRows];
#pragma unroll
      for (int r = 0; r < kAqRows; ++r) {
        m[r] = fabsf(x[r][0] * iv[0]);
#pragma unroll
        for (int j = 1; j < 8; ++j) m[r] = fmaxf(m[r], fabsf(x[r][j] * iv[j]));
        m[r] = fmaxf(m[r], 0.0f);      // (an all-NaN lane counts as zero)
      }
      // eight maxima over 16 lanes: two steps in which a lane passes half of its rows on, then two rotations
#pragma unroll
      for (int j = 0; j < 4; ++j) m[j] = fmaxf(b0 ? m[j + 4] : m[j], dpp<0xB1>(b0 ? m[j] : m[j + 4]));
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        m[j] = fmaxf(b1 ? m[j + 2] : m[j], dpp<0x4E>(b1 ? m[j] : m[j + 2]));
        m[j] = fmaxf(m[j], dpp<0x124>(m[j]));
        m[j] = fmaxf(m[j], dpp<0x128>(m[j]));
      }
      float2* at = reinterpret_cast<float2*>(mine + k * kAqRows);
      if ((lane & 15) < 4) {
        if (strip != wave) { const float2 o = *at; m[0] = fmaxf(m[0], o.x); m[1] = fmaxf(m[1], o.y); }
        *at = make_float2(m[0], m[1]);
      }
    }
  }
  __syncthreads();
  const int parts = (nw < strips ? nw : strips) * 4;
  for (int i = threadIdx.x; i < nk * kAqRows; i += blockDim.x) {
    float m = 0.0f;
    for (int w = 0; w < parts; ++w) m = fmaxf(m, part[w * cand_step * kAqRows + i]);
    const float sg = fmaxf(m, kRangeFloor) / qa;
    const int k = i / kAqRows, r = i % kAqRows;
    step[k][r] = sg;
    if (r0 + r < n_tok) sig[(int64_t)(k0 + k) * n_tok + r0 + r] = sg;
  }
  __syncthreads();
  for (int strip = wave; strip < strips; strip += nw) {
    const int64_t c = (int64_t)strip * kAqCols + lane * 8;
    if (c >= (INT ? ldc : c_in)) continue;
    aq_load_tile<T>(X, n_tok, c_in, ldx, r0, c, x);
    for (int k = 0; k < nk; ++k) {
      if (inv_table && (!INT || c < c_in)) load8(inv_table + (int64_t)(k0 + k) * c_in + c, iv);
      // (behind c_in any code will do, the weights are zeros there: a zero gives the code zero, unless the lane's last
      // factor was infinite)
      const int64_t at = ((int64_t)(k0 + k) * n_tok + r0) * ldc + c;
#pragma unroll
      for (int r = 0; r < kAqRows; ++r) {
        if (r0 + r >= n_tok) break;
        // (the quantiser's quotient: an approximate reciprocal, true divisions near a tie and for huge steps)
        Grid g;
        g.delta = step[k][r];
        g.rd = __builtin_amdgcn_rcpf(g.delta);
        // (the step came from a division by qa: no quotient is beyond qa and a rounding)
        g.lim = g.delta < 1e36f ? 0.49999976f - 4.8e-7f * (qa + 1.0f) : -1.0f;
        float xt[8], n[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) xt[j] = x[r][j] * iv[j];
        if (!(rint_quotient8(xt, g, 0.0f, n) < g.lim)) divide8(xt, g, n);
        if constexpr (INT) {
#pragma unroll
          for (int j = 0; j < 8; ++j) n[j] = __builtin_amdgcn_fmed3f(n[j], -qa - 1.0f, qa);
          store8((int8_t*)codes + at + r * ldc, pack_i8(n[0], n[1], n[2], n[3]), pack_i8(n[4], n[5], n[6], n[7]), nt);
          continue;
        }
        uint32_t o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          o[j] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(__builtin_amdgcn_fmed3f(n[2 * j], -qa - 1.0f, qa),
                                                                         __builtin_amdgcn_fmed3f(n[2 * j + 1], -qa - 1.0f, qa)));
        store16(codes + at + r * ldc, make_uint4(o[0], o[1], o[2], o[3]), nt);
      }
    }
  }
}

hipError_t launch_act_quant(const void* X, int64_t n_tok, int64_t c_in, int64_t ldx, bool bf16,
                            const float* inv_table, int k0, int nb, int act_bits, void* codes,
                            float* sigma, hipStream_t stream, int64_t ld8) {
  ProfScope ps("act_quant", stream, (double)n_tok * (double)c_in * (4.0 + (ld8 ? 1.0 : 2.0) * nb));
  const float qa = (float)((1 << (act_bits - 1)) - 1);
  const int64_t strips = ceil_div(c_in, kAqCols), blocks = ceil_div(n_tok, kAqRows);
  const int nw = (int)(strips < kAqWaves ? strips : kAqWaves);
  // few rows: the candidates of a block are split over the grid until every SIMD has two waves
  int64_t split = blocks * nw < 2048 ? 2048 / (blocks * nw) : 1;
  if (split > nb) split = nb;
  int cand_step = (int)ceil_div(nb, split);
  if (cand_step > kAqStep) cand_step = kAqStep;
  const dim3 grid((unsigned)blocks, (unsigned)ceil_div(nb, cand_step));
  const size_t lds = (size_t)nw * 4 * cand_step * kAqRows * sizeof(float);
  const float* inv = inv_table ? inv_table + (int64_t)k0 * c_in : nullptr;
  const bool nt = streams_past((ld8 ? 1.0 : 2.0) * (double)nb * (double)n_tok * (double)c_in);
  auto go = [&](auto kern) {
    kern<<<grid, nw * 64, lds, stream>>>((const uint16_t*)X, n_tok, c_in, ldx, inv, nb, cand_step, qa, sigma, (uint16_t*)codes,
                                  ld8 ? ld8 : c_in, nt);
  };
  if (ld8) bf16 ? go(act_quant_kernel<BF16, true>) : go(act_quant_kernel<F16, true>);
  else bf16 ? go(act_quant_kernel<BF16, false>) : go(act_quant_kernel<F16, false>);
  return hipGetLastError();
}

template <typename T, bool SYM, int MODE>
static void launch_quant(QuantDev d, hipStream_t stream) {
  // Enough blocks to fill the chip: the candidates of small matrices are split over blockIdx.y (W is
  // read again per stretch, from L2).  `waves` counts the waves of one stretch; 8192 = 8 per SIMD.
  auto grid = [&](int64_t blocks, int64_t waves, int most = 5) {
    int64_t split = waves < 8192 ? 8192 / waves : 1;
    if (split > d.n_cand) split = d.n_cand;
    d.cand_step = (int)ceil_div(d.n_cand, split);
    // Never more than five candidates a wave: what is written at any time are then a few stretches of memory and not
    // twenty (stores alone, 20 x 4096 x 4096: 4.3 TB/s with all candidates in a wave, 5.6 with five, 3.9 with one, which
    // reads W as often as it writes; this kernel, us by candidates a wave 2, 3, 5, 10, 20: 161, 148, 142, 151, 158; in cache,
    // 16 x 3000 x 3000 in whole rows 3, 5, 10, 16: 73, 70, 73, 89)
    if (d.cand_step > most) d.cand_step = (int)ceil_div(d.n_cand, ceil_div(d.n_cand, 5));
    return dim3((unsigned)blocks, (unsigned)ceil_div(d.n_cand, d.cand_step));
  };
  // A group below 64 that is no power of two would have a wave of quant_row_kernel to its 3 to 7 chunks: whole groups
  // share a wave instead (their number is a 32-bit index there).
  const bool pow2 = MODE != Q_INT && (d.group & (d.group - 1)) == 0;
  d.packed = MODE != Q_INT && !pow2 && d.group < 64 && d.c_out * (d.c_in / d.group) < (1LL << 30);
  if constexpr (MODE != Q_INT) if (d.packed || (pow2 && d.group <= 512)) {
    for (d.shift = 0; (8LL << d.shift) < d.group;) ++d.shift;
    // rows per wave by size: two share the scale loads once there is work for every SIMD anyway
    constexpr int R = MODE == Q_AUX ? 1 : 2;
    auto waves_of = [&](int64_t rows) {
      return d.packed ? ceil_div(rows * (d.c_in / d.group), 64 >> d.shift) : rows * ceil_div(d.c_in, 512);
    };
    const bool two = R == 2 && waves_of(ceil_div(d.c_out, 2)) * d.n_cand >= 8192;
    const int64_t waves = waves_of(ceil_div(d.c_out, two ? 2 : 1));
    // Up to nine stay together here while they fit the last-level cache, more or less: then it is the second reading of W that counts (a
    // search, us five at most -> nine: 4096 x 4096 in groups of 128, 6 candidates (201 MB) 112.3 -> 109.3, 9 (302 MB) 238.3 -> 234.5, in
    // groups of 40, 7 candidates 194 -> 187; 11,008 x 4096, 6 candidates (541 MB) 317 -> 347)
    const dim3 g = grid(ceil_div(waves, 4), waves, d.n_cand <= 9 && 2.0 * d.n_cand * d.c_out * d.c_in <= 400e6 ? 9 : 5);
    if (two && d.group == 128) quant_pow2_kernel<T, SYM, MODE, R, 16><<<g, 256, 0, stream>>>(d);
    else if (two) quant_pow2_kernel<T, SYM, MODE, R, 0><<<g, 256, 0, stream>>>(d);
    else if (d.group == 128) quant_pow2_kernel<T, SYM, MODE, 1, 16><<<g, 256, 0, stream>>>(d);
    else quant_pow2_kernel<T, SYM, MODE, 1, 0><<<g, 256, 0, stream>>>(d);
    return;
  }
  const int64_t G = d.c_in / d.group;
  auto one = [&](auto kern, int rows) {     // a wave per group
    const int64_t waves = ceil_div(d.c_out, rows) * G;
    const dim3 g = grid(ceil_div(waves, 4), waves);
    kern<<<g, 256, 0, stream>>>(d);
  };
  auto four = [&](auto kern, int rows) {    // a block per group
    const int64_t blocks = ceil_div(d.c_out, rows) * G;
    const dim3 g = grid(blocks, 4 * blocks);
    kern<<<g, 256, 0, stream>>>(d);
  };
  // rows x chunks: up to 8 packed register quads per lane (4 with one chunk); a block per group above 2048 channels
  // (a wave alone would need more than four chunks a lane)
  if constexpr (MODE == Q_INT) {       // (half the shapes: every instance lengthens the loading of the library)
    if (d.group <= 1024) one(quant_row_kernel<T, SYM, MODE, 1, 2, 2>, 2);
    else if (d.group <= 4096) four(quant_row_kernel<T, SYM, MODE, 4, 2, 2>, 2);
    else if (d.group <= 8192) four(quant_row_kernel<T, SYM, MODE, 4, 4, 2>, 2);
    else four(quant_row_kernel<T, SYM, MODE, 4, 8, 1>, 1);
    return;
  } else {
  if (d.group <= 512) one(quant_row_kernel<T, SYM, MODE, 1, 1, 4>, 4);
  else if (d.group <= 1024) one(quant_row_kernel<T, SYM, MODE, 1, 2, 2>, 2);
  else if (d.group <= 2048) one(quant_row_kernel<T, SYM, MODE, 1, 4, 1>, 1);
  else if (d.group <= 4096) four(quant_row_kernel<T, SYM, MODE, 4, 2, 2>, 2);
  else if (d.group <= 8192) four(quant_row_kernel<T, SYM, MODE, 4, 4, 2>, 2);
  else if (d.group <= 16384) four(quant_row_kernel<T, SYM, MODE, 4, 8, 1>, 1);
  else quant_any_kernel<T, SYM, MODE><<<(unsigned)ceil_div(d.c_out * G, 4), 256, 0, stream>>>(d);
  }
}

hipError_t launch_fake_quant(const QuantArgs& q, hipStream_t stream) {
  QuantDev d;
  d.W = (const uint16_t*)q.W; d.c_out = q.c_out; d.c_in = q.c_in; d.ldw = q.ldw;
  d.qmax = (float)((1 << q.bits) - 1);
  d.half = 1 << (q.bits - 1);
  d.qlo = -(float)d.half; d.qhi = (float)(d.half - 1);
  d.rq = 1.0f / (q.symmetric ? d.qhi : d.qmax);
  d.group = q.group == 0 ? q.c_in : q.group;
  d.s_table = q.s_table; d.inv_table = q.inv_table; d.n_cand = q.n_cand; d.cand_step = q.n_cand;
  d.what = (uint16_t*)q.what; d.what_cand_stride = q.what_cand_stride;
  d.codes = q.codes; d.zp = q.zp; d.delta = q.delta; d.wdq = (uint16_t*)q.wdq; d.ld_dq = q.ld_dq;
  d.diff = q.diff; d.xmax_bits = q.xmax_bits; d.col_scale = q.col_scale;
  d.w8 = q.w8; d.ld8 = q.ld8; d.w8_cand_stride = q.w8_cand_stride; d.steps = q.steps; d.step_stride = q.step_stride;
  if (q.w8 && (d.group != q.c_in || d.group > 16384 || (!q.symmetric && q.bits > 7))) return hipErrorInvalidValue;
  const double bytes = (double)q.c_out * (double)q.c_in * (2.0 + 2.0 * (q.what ? q.n_cand : 0) + 1.0 * (q.w8 ? q.n_cand : 0) +
                                                           (q.codes ? 1.0 : 0.0) + (q.wdq ? 2.0 : 0.0));
  // (20 candidates of 4096 x 4096 and 1200 tokens: the whole search 933 -> 892 us)
  d.nt = streams_past((q.w8 ? 1.0 : 2.0) * (double)q.n_cand * (double)q.c_out * (double)q.c_in);
  ProfScope ps("fake_quant", stream, bytes);
  auto pick = [&](auto t, auto sym) {
    using T = decltype(t);
    constexpr bool SYM = decltype(sym)::value;
    if (q.w8) launch_quant<T, SYM, Q_INT>(d, stream);
    else if (!q.what) launch_quant<T, SYM, Q_AUX>(d, stream);
    else if (q.diff) launch_quant<T, SYM, Q_DIFF>(d, stream);
    else launch_quant<T, SYM, Q_FOLD>(d, stream);
  };
  if (!q.bf16) q.symmetric ? pick(F16{}, std::true_type{}) : pick(F16{}, std::false_type{});
  else q.symmetric ? pick(BF16{}, std::true_type{}) : pick(BF16{}, std::false_type{});
  return hipGetLastError();
}

// Wout[o,c] = round16(Win[o,c] * inv_s[c]); dense output, row stride c_in.  A block owns 2048 channels and
// walks rows, so the eight factors of a lane are loaded once (HBM-bound; with a flat index the 64-bit
// division and the scalar factor loads took 105 us for 4096 x 11008).
template <typename T, typename TO>
__global__ __launch_bounds__(256) void fold_scale_kernel(const uint16_t* __restrict__ Win,
                                                         int64_t c_out, int64_t c_in, int64_t ldw,
                                                         const float* __restrict__ inv_s,
                                                         const uint32_t* __restrict__ xmax_bits,
                                                         uint16_t* __restrict__ Wout) {
  const int64_t c = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (c >= c_in) return;
  const float up = xmax_bits
      ? __builtin_bit_cast(float, (uint32_t)(127 + shift_from_bf16_bits(*xmax_bits)) << 23) : 1.0f;
  float inv[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) inv[j] = inv_s ? inv_s[c + j] : 1.0f;   // (no alignment promised for inv_s)
#pragma unroll 2
  for (int64_t row = blockIdx.y; row < c_out; row += gridDim.y) {
    float w[8];
    widen8<T>(*reinterpret_cast<const uint4*>(Win + row * ldw + c), w);
    uint32_t o[4] = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j >> 1] |= (uint32_t)TO::from_float(w[j] * inv[j] * up) << ((j & 1) * 16);
    *reinterpret_cast<uint4*>(Wout + row * c_in + c) = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

hipError_t launch_fold_scale(const void* Win, int64_t c_out, int64_t c_in, int64_t ldw, bool bf16,
                             const float* inv_s, const uint32_t* xmax_bits, bool out_f16, void* Wout,
                             hipStream_t stream) {
  ProfScope ps("fold_scale", stream, 4.0 * (double)c_out * (double)c_in);
  // rows per block: enough blocks for the chip first, then up to 16 rows per load of the factors
  const int64_t bx = ceil_div(c_in, 2048);
  int64_t by = 4096 / bx;
  by = by < 1 ? 1 : by;
  const dim3 grid((unsigned)bx, (unsigned)(c_out < by ? c_out : by));
  const uint16_t* in = (const uint16_t*)Win;
  uint16_t* out = (uint16_t*)Wout;
  if (!bf16) fold_scale_kernel<F16, F16><<<grid, 256, 0, stream>>>(in, c_out, c_in, ldw, inv_s, xmax_bits, out);
  else if (out_f16) fold_scale_kernel<BF16, F16><<<grid, 256, 0, stream>>>(in, c_out, c_in, ldw, inv_s, xmax_bits, out);
  else fold_scale_kernel<BF16, BF16><<<grid, 256, 0, stream>>>(in, c_out, c_in, ldw, inv_s, xmax_bits, out);
  return hipGetLastError();
}

}  // namespace tlq
