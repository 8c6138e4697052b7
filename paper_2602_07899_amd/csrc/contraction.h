// S3 + S4: the candidate-evaluation contraction with the loss fused into its
// epilogue (Sec. 3.2.1 objective; Sec. 2.2 smoothing identity), and the same
// contraction with a store epilogue (f_fp of Sec. 3.2.1; PassAct2 output).
//
// The kernels compute  D[o, t] = sum_c What[o, c] * X[t, c]  on fp16/bf16 MFMA
// with float accumulation.  `What` stacks the folded operands
// of all candidates ([n_cand * c_out, c_in]), so the alpha grid is simply an
// extra stretch of the o dimension and every X tile is shared by all
// candidates.  In the loss epilogue each lane owns one token column of its
// accumulator tiles: it subtracts the accumulators from Y_ref, squares, sums
// over its output rows, multiplies by that token's weight and the block
// reduces to ONE float per (candidate, tile).  Candidate outputs never reach
// HBM.
//
// The same kernels serve the second-moment form of the search (gram.hip): the product of the
// transposed, weighted tokens with themselves (store epilogue, only the tiles of one triangle,
// the long contraction split into "candidates" that are summed afterwards), and the quadratic
// form of every candidate's weight error in that matrix (EPI_DOT: accumulator times Y instead of
// the squared residual; SYMK: only the upper part of the symmetric operand is contracted).
//
// This file holds what the kernels share: operand types, tile epilogues, the block -> tile map and the body of the
// pipelined kernels (16x16x32 MFMA, operands brought into LDS by LDS-DMA loads, two 64 KB stages, hand-placed waits):
//   gemm_dma_kernel    (gemm.hip) tiles of 256 x 256 and 128 x 128;
//   gemm_width_kernel  (gemm_width.hip) 256 x 192 and 256 x 320, for launches that they suit better (gemm_tile);
//   gemm_half_kernel   (gemm_half.hip) 128 x 64, for launches of at most one of them a CU;
//   gemm_small_tok_kernel  (gemm_tok.hip) 128 x 128 with the errors of tokens;
//   gemm_i8_kernel     (gemm_i8.hip) integer codes, all four tiles;
//   gemm_kernel        (gemm.hip) for row strides of 2^21 elements and more (beyond the 32-bit offsets of the others):
//                      32x32x16 MFMA, register-staged loads.
// They are five files because the kernels of a file are loaded together, by the first call that needs one of them, and
// few programs need all (library, first product and first small search of a process: 9.7 ms with all that there were in one file, 7.6
// in the first three; on another box 7.5 in those three and 7.9 in five, where the first product, in tiles of 128 x 64, takes 2.2
// instead of 3.3 and the search loads the square tiles).
// Tiling (wave64): block tile 256 x 256 outputs, k-tile 64; waves own 128 x 64
// sub-tiles.  Both operands are K-contiguous in memory, so a fragment is one
// 16-byte LDS read per lane.  LDS rows are 128 B (64 halves) and the eight
// 16-byte chunks of a row are XOR-swizzled with (row/2)%8 so that the 16 lanes
// served together by a 128-bit LDS access touch 16 different bank groups, for
// the fragment reads and for the tile writes alike.
#pragma once
#include <type_traits>
#include <utility>

#include "common.h"

namespace tlq {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <typename T> struct Mma;
template <> struct Mma<F16> {
  static __device__ __forceinline__ f32x16 run(const uint4& a, const uint4& b, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                  __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mma<BF16> {
  static __device__ __forceinline__ f32x16 run(const uint4& a, const uint4& b, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};

typedef float f32x4 __attribute__((ext_vector_type(4)));
// 16x16x32: half the accumulator registers read and written per flop of the 32x32x16 shape.  The
// matrix cores are power-limited with real operands, and a register-only loop with random operands
// sustains 1840 TFLOP/s with this shape against 1585 with 32x32x16, so the pipelined kernel uses it.
template <typename T> struct Mma16;
template <> struct Mma16<F16> {
  static __device__ __forceinline__ f32x4 run(const uint4& a, const uint4& b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                  __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mma16<BF16> {
  static __device__ __forceinline__ f32x4 run(const uint4& a, const uint4& b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};

// Integer codes: a lane's 16-byte fragment holds 16 of them instead of eight halves, so everything up to the MFMA sees an
// int8 matrix as one of 16-bit elements with half the columns.  The accumulator registers hold integers, exact sums of
// at most 16384 * 2^14.
struct Int8 {};
typedef int i32x4 __attribute__((ext_vector_type(4)));
template <> struct Mma16<Int8> {
  static __device__ __forceinline__ f32x4 run(const uint4& a, const uint4& b, const f32x4& c) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a),
                                                                           __builtin_bit_cast(i32x4, b),
                                                                           __builtin_bit_cast(i32x4, c), 0, 0, 0));
  }
};

// How a wave's accumulators map to (output row, token).  With either MFMA shape (weights as the
// "A" operand, tokens as "B") a lane owns ONE token column per accumulator tile and groups of four
// consecutive output rows ("quads").  A layout names its quads q < NQ and token blocks tb < NTB:
//   tok(tb, lane)  token of the lane inside the wave tile,
//   row(q, lane)   first of the four output rows of quad q inside the wave tile,
//   get(acc, q, tb, r)  the accumulator of row(q) + r and tok(tb),
//   tok_sum(v)     sum of v over the lanes that hold the same token.
template <int FA, int FB> struct Acc32 {   // acc[FA][FB] of f32x16 (32x32x16)
  static constexpr int NQ = FA * 4, NTB = FB, WO = FA * 32, WT = FB * 32, STG = FB;
  static __device__ __forceinline__ int tok(int tb, int lane) { return tb * 32 + (lane & 31); }
  static __device__ __forceinline__ int row(int q, int lane) { return (q >> 2) * 32 + (q & 3) * 8 + (lane >> 5) * 4; }
  template <typename A> static __device__ __forceinline__ float get(const A& acc, int q, int tb, int r) {
    return acc[q >> 2][tb][(q & 3) * 4 + r];
  }
  static __device__ __forceinline__ float tok_sum(float v) { return v + __shfl_xor(v, 32, 64); }
};
template <int IA, int JB> struct Acc16 {   // acc[IA][JB] of f32x4 (16x16x32)
  static constexpr int NQ = IA, NTB = JB, WO = IA * 16, WT = JB * 16, STG = JB > 4 ? 2 : JB;
  static __device__ __forceinline__ int tok(int tb, int lane) { return tb * 16 + (lane & 15); }
  static __device__ __forceinline__ int row(int q, int lane) { return q * 16 + (lane >> 4) * 4; }
  template <typename A> static __device__ __forceinline__ float get(const A& acc, int q, int tb, int r) {
    return acc[q][tb][r];
  }
  static __device__ __forceinline__ float tok_sum(float v) {
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
  }
};

// EPI_DOT: partial = sum over the tile of acc * Y (Y read like Y_ref, one matrix per candidate, no
// token weights): the quadratic form of the second-moment search.
enum { EPI_LOSS = 0, EPI_LOSS_TOK = 1, EPI_STORE = 2, EPI_DOT = 3 };
constexpr int BK = 64;        // halves per k-tile
constexpr int ROWB = BK * 2;  // bytes per LDS row
// An L2 patch (one per XCD at a time) is po x pt tiles = 32 workgroups: 4 x 8 by default (4 operand
// panels that stay while the walk moves along the tokens + 8 token panels), or 8 x 4 for launches
// whose walk keeps the output-side panels and changes the token-side ones from patch to patch.
constexpr int PATCH_SLOTS = 32, kXcd = 8;

struct GemmDev {
  const uint16_t* X; int64_t n_tok, c_in, ldx, x_cand_stride;
  const float* tok_scale;  // [n_cand, n_tok] per-token factor on the accumulators, or NULL
  const uint16_t* Wh; int64_t c_out, ldw, w_cand_stride; int n_cand;
  const void* Yref; int64_t ldy; int ydt; const float* token_w;
  int64_t y_cand_stride;   // elements between per-candidate Y matrices (EPI_DOT; 0 = shared)
  int tri;                 // 1: only tiles with tile row <= tile column are computed (symmetric product)
  int cand_outer;          // 1: the candidate is the outermost level of the block order
  int64_t o_cand_stride;   // EPI_STORE: elements between per-candidate outputs
  float* partial; float* tok_partial;
  void* Yout; int64_t ldo; int odt;
  int tiles_o, tiles_t, npo, npt;  // tiles per candidate and patches per candidate
  int64_t n_patches;
  int cpt;          // token patches per chunk (see make_dev)
  int rag, rag_pt;  // tile rows of the last, incomplete patch row (0 = none) and its patch width in tiles
  int po, pt;       // patch shape in tiles (po * pt <= PATCH_SLOTS)
  int rot;          // XCD rotation from one round of patches to the next (see make_dev)
  int64_t strips;   // > 0: no patches, the launch has this many tiles (see decode_tile)
  const float* row_scale; int64_t row_scale_stride;   // integer codes: steps of the output rows per candidate
};

__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

__device__ __forceinline__ float load_y(const void* Y, int ydt, int64_t idx) {
  if (ydt == TLQ_F32) return ((const float*)Y)[idx];
  const uint16_t b = ((const uint16_t*)Y)[idx];
  return ydt == TLQ_F16 ? F16::to_float(b) : BF16::to_float(b);
}
__device__ __forceinline__ void load_y4(const void* Y, int ydt, int64_t idx, float y[4]) {
  if (ydt == TLQ_F32) {
    const float4 v = *reinterpret_cast<const float4*>((const float*)Y + idx);
    y[0] = v.x; y[1] = v.y; y[2] = v.z; y[3] = v.w;
  } else {
    const uint2 v = *reinterpret_cast<const uint2*>((const uint16_t*)Y + idx);
    if (ydt == TLQ_F16) {
      y[0] = F16::to_float((uint16_t)v.x); y[1] = F16::to_float((uint16_t)(v.x >> 16));
      y[2] = F16::to_float((uint16_t)v.y); y[3] = F16::to_float((uint16_t)(v.y >> 16));
    } else {
      y[0] = BF16::to_float((uint16_t)v.x); y[1] = BF16::to_float((uint16_t)(v.x >> 16));
      y[2] = BF16::to_float((uint16_t)v.y); y[3] = BF16::to_float((uint16_t)(v.y >> 16));
    }
  }
}
__device__ __forceinline__ void store_y4(void* Y, int odt, int64_t idx, const float y[4]) {
  if (odt == TLQ_F32) {
    *reinterpret_cast<float4*>((float*)Y + idx) = make_float4(y[0], y[1], y[2], y[3]);
  } else if (odt == TLQ_F16) {
    *reinterpret_cast<uint2*>((uint16_t*)Y + idx) =
        make_uint2((uint32_t)F16::from_float(y[0]) | ((uint32_t)F16::from_float(y[1]) << 16),
                   (uint32_t)F16::from_float(y[2]) | ((uint32_t)F16::from_float(y[3]) << 16));
  } else {
    *reinterpret_cast<uint2*>((uint16_t*)Y + idx) =
        make_uint2((uint32_t)BF16::from_float(y[0]) | ((uint32_t)BF16::from_float(y[1]) << 16),
                   (uint32_t)BF16::from_float(y[2]) | ((uint32_t)BF16::from_float(y[3]) << 16));
  }
}
__device__ __forceinline__ void store_y1(void* Y, int odt, int64_t idx, float y) {
  if (odt == TLQ_F32) ((float*)Y)[idx] = y;
  else ((uint16_t*)Y)[idx] = odt == TLQ_F16 ? F16::from_float(y) : BF16::from_float(y);
}



template <int I, int N, typename Fn>
__device__ __forceinline__ void static_for(Fn&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Per-lane part of the loss of one wave tile whose first output row is `ow` and first
// token is `tw`: sq[tb] = sum over this lane's rows of (Y_ref - acc)^2 for its token of
// token block tb; part = sum_tb token_w * sq[tb].  YDT is the type of Y_ref, k16Bit either 16-bit type; FULL promises that
// the whole wave tile lies inside the matrix.  Otherwise loads past it go to a valid place and their terms are dropped:
// a branch around each would put their latencies one after the other, and the tiles at the edges are the last ones of a
// launch that fits the chip in a few rounds.  NQ: the quads that hold live rows, straight code for half of them where the
// other half lies past the edge (and none for a wave that does as a whole): with 64 outputs in tiles of 256 the reads
// for nothing cost more than the product (100,000 x 64 x 64, us with a branch around each read, all reads, live halves:
// loss 24.7, 28.9, 19.0; 20 candidates 427, 458, 324; with 136 outputs the loss 36.0, 24.3, 24.1).  Token blocks past the
// edge end the walk (one token of 256 x 256: 14.3, 16.0, 13.4).
// DOT replaces the squared residual by the product acc * y and drops the token weight.
constexpr int k16Bit = -1;
template <int YDT, bool FULL, bool DOT, typename L, int NQ, typename Acc>
__device__ __forceinline__ void loss_rows(const GemmDev& a, const void* Yref, const Acc& acc, const float* tsc,
                                          int64_t ow, int64_t tw, float (&sq)[L::NTB], float& part) {
  const int lane = threadIdx.x & 63;
  const bool quads = FULL || a.c_out >= 4, ragged = !FULL && (!quads || (a.c_out & 3) != 0);
#pragma unroll
  for (int tb = 0; tb < L::NTB; ++tb) {
    if (!FULL && tw + L::tok(tb, 0) >= a.n_tok) break;      // (sq is zero there)
    const int64_t tl = tw + L::tok(tb, lane);
    const bool t_ok = FULL || tl < a.n_tok;
    const int64_t t = t_ok ? tl : a.n_tok - 1;
    float sumsq = 0.0f;
    // residual = y - sg * acc as one fused multiply-add; sg = 1 gives y - acc exactly
    const float nsg = tsc ? -tsc[t] : -1.0f;
    auto term = [&](int q, int r, float y) {
      if (DOT) { sumsq += L::get(acc, q, tb, r) * y; return; }
      const float d = __builtin_fmaf(nsg, L::get(acc, q, tb, r), y);
      sumsq += d * d;
    };
    if (quads) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int64_t o = ow + L::row(q, lane);
        const bool whole = FULL || o + 3 < a.c_out;
        float y[4];
        if constexpr (YDT == k16Bit) {
          const uint2 u = *reinterpret_cast<const uint2*>((const uint16_t*)Yref + t * a.ldy + (whole ? o : 0));
          const uint16_t h[4] = {(uint16_t)u.x, (uint16_t)(u.x >> 16), (uint16_t)u.y, (uint16_t)(u.y >> 16)};
#pragma unroll
          for (int r = 0; r < 4; ++r) y[r] = a.ydt == TLQ_F16 ? F16::to_float(h[r]) : BF16::to_float(h[r]);
        } else {
          load_y4(Yref, YDT, t * a.ldy + (whole ? o : 0), y);
        }
        const float before = sumsq;
#pragma unroll
        for (int r = 0; r < 4; ++r) term(q, r, y[r]);
        if (!whole) sumsq = before;
      }
    }
    if (ragged) {   // the last rows of a matrix whose height is no multiple of four
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int64_t o = ow + L::row(q, lane);
        if (o < a.c_out && o + 3 >= a.c_out) {
#pragma unroll
          for (int r = 0; r < 3; ++r)
            if (o + r < a.c_out) term(q, r, load_y(Yref, a.ydt, t * a.ldy + o + r));
        }
      }
    }
    if (!t_ok) sumsq = 0.0f;
    part += DOT ? sumsq : t_ok ? a.token_w[t] * sumsq : 0.0f;
    sq[tb] = sumsq;
  }
}

// A wave tile passes through LDS L::STG token blocks at a time, in this wave's own piece of WO x 16 STG 16-bit values
// (all of it at once up to 64 tokens; 80 would not fit beside each other's).  16-byte chunks of a token row are stored
// at chunk ^ row_key(token), which makes the 8-byte accesses conflict-free.
template <int CPR>   // rows of 256 B (CPR = 16) or 128 B (two of them span the banks once)
__device__ __forceinline__ int row_key(int row) { return CPR == 16 ? row & 15 : (row >> 1) & 7; }

// The LDS accesses of a wave are executed in order; this keeps the compiler from moving those of one lane across
// those of OTHER lanes of the wave
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
template <typename L> struct Staged {
  static constexpr int WO = L::WO, TBW = L::WT / L::NTB, CPR = WO / 8, RPI = 64 / CPR;   // RPI: rows per wave-wide copy
  static constexpr int GROUPS = (L::NTB + L::STG - 1) / L::STG;
  static_assert((CPR == 16 || CPR == 8) && TBW % RPI == 0, "copy shape");
  // token blocks of group G, and its 16-byte copies per lane
  template <int G> static constexpr int blocks() { return L::NTB - G * L::STG < L::STG ? L::NTB - G * L::STG : L::STG; }
  template <int G> static constexpr int copies() { return blocks<G>() * TBW / RPI; }
  // Four values of token block `b` of the group, quad `q` of the lane; and eight of copy number `j`.  The keys repeat
  // every 16 rows, so b and j only add constants
  static __device__ __forceinline__ uint2* at4(unsigned char* ylds, int b, int q) {
    const int lane = threadIdx.x & 63, tok = L::tok(0, lane), o = L::row(q, lane);   // (o a multiple of 4)
    return reinterpret_cast<uint2*>(ylds + tok * (WO * 2) + (((o >> 3) ^ row_key<CPR>(tok)) << 4) + ((o >> 2) & 1) * 8 +
                                    b * TBW * (WO * 2));
  }
  static __device__ __forceinline__ uint4* at8(unsigned char* ylds, int j) {
    constexpr int PER = 16 / RPI;
    const int lane = threadIdx.x & 63, row = (j % PER) * RPI + lane / CPR, chunk = lane % CPR;
    return reinterpret_cast<uint4*>(ylds + row * (WO * 2) + ((chunk ^ row_key<CPR>(row)) << 4) + j / PER * 16 * (WO * 2));
  }
  // group G of the wave's piece of a 16-bit matrix into LDS: whole-line loads (each 128-byte line is fetched once, 8
  // lines per instruction)
  template <int G>
  static __device__ __forceinline__ void fill(const void* Yref, int64_t ldy, int64_t ow, int64_t tw, unsigned char* ylds) {
    const int lane = threadIdx.x & 63, cr = lane / CPR, cc = lane % CPR;
    const uint16_t* Y = (const uint16_t*)Yref + (tw + G * L::STG * TBW + cr) * ldy + ow + cc * 8;
    if (G > 0) wave_lds_order();
    uint4 v[copies<G>()];
#pragma unroll
    for (int j = 0; j < copies<G>(); ++j) v[j] = *reinterpret_cast<const uint4*>(Y + j * RPI * ldy);
#pragma unroll
    for (int j = 0; j < copies<G>(); ++j) *at8(ylds, j) = v[j];
    wave_lds_order();
  }
  // ... and back out of LDS, whole lines again
  template <int G>
  static __device__ __forceinline__ void drain(void* Yout, int64_t ldo, int64_t ow, int64_t tw, unsigned char* ylds) {
    const int lane = threadIdx.x & 63, cr = lane / CPR, cc = lane % CPR;
    uint16_t* Y = (uint16_t*)Yout + (tw + G * L::STG * TBW + cr) * ldo + ow + cc * 8;
#pragma unroll
    for (int j = 0; j < copies<G>(); ++j) *reinterpret_cast<uint4*>(Y + j * RPI * ldo) = *at8(ylds, j);
  }
};
template <typename YT>
__device__ __forceinline__ void unpack4(uint2 u, float (&y)[4]) {
  y[0] = YT::to_float((uint16_t)(u.x & 0xffffu)); y[1] = YT::to_float((uint16_t)(u.x >> 16));
  y[2] = YT::to_float((uint16_t)(u.y & 0xffffu)); y[3] = YT::to_float((uint16_t)(u.y >> 16));
}

// Same sums as loss_rows for an interior wave tile with 16-bit Y_ref, but Y_ref goes through LDS and every lane picks
// its values from there.  Reading Y_ref straight from the accumulator layout touches 16 or 32 lines per
// instruction and each line 8 times (losses with token errors, us that way -> through LDS: 14,000 x 64 x 6144 with
// 256-token tiles 81, with 320 89 -> 64; 27,730 x 2048 x 10,728 1054 and 1048 -> 999).
template <typename YT, bool DOT, typename L, typename Acc>
__device__ __forceinline__ void loss_rows_lds(const GemmDev& a, const void* Yref, const Acc& acc, const float* tsc,
                                              int64_t ow, int64_t tw, float (&sq)[L::NTB], float& part,
                                              unsigned char* ylds) {
  using S = Staged<L>;
  const int lane = threadIdx.x & 63;
  // the bodies of the two types stay apart: merged, with a branch at every value, they need more registers than there are
  asm volatile("; values of type %0" ::"n"(std::is_same<YT, F16>::value ? TLQ_F16 : TLQ_BF16));
  float nsg[L::NTB];
#pragma unroll
  for (int tb = 0; tb < L::NTB; ++tb) nsg[tb] = -1.0f;
  if (tsc) {
#pragma unroll
    for (int tb = 0; tb < L::NTB; ++tb) nsg[tb] = -tsc[tw + L::tok(tb, lane)];
  }
  static_for<0, S::GROUPS>([&](auto gc) {
    constexpr int G = decltype(gc)::value;
    S::template fill<G>(Yref, a.ldy, ow, tw, ylds);
#pragma unroll
    for (int b = 0; b < S::template blocks<G>(); ++b) {
      const int tb = G * L::STG + b;
      float sumsq = 0.0f;
#pragma unroll
      for (int q = 0; q < L::NQ; ++q) {
        float y[4];
        unpack4<YT>(*S::at4(ylds, b, q), y);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (DOT) { sumsq += L::get(acc, q, tb, r) * y[r]; continue; }
          const float d = __builtin_fmaf(nsg[tb], L::get(acc, q, tb, r), y[r]);
          sumsq += d * d;
        }
      }
      part += DOT ? sumsq : a.token_w[tw + L::tok(tb, lane)] * sumsq;
      sq[tb] = sumsq;
      if (L::NTB > 4) __builtin_amdgcn_sched_barrier(0);
    }
  });
}

// Store epilogue of an interior wave tile with a 16-bit output, through LDS: every lane drops its rounded values there,
// then the wave writes whole lines.  Storing straight from the accumulator layout writes 8-byte pieces of
// 16 or 32 lines per instruction.
template <typename YT, typename L, typename Acc>
__device__ __forceinline__ void store_rows_lds(const GemmDev& a, void* Yout, const Acc& acc, const float* tsc,
                                               int64_t ow, int64_t tw, unsigned char* ylds) {
  using S = Staged<L>;
  const int lane = threadIdx.x & 63;
  static_for<0, S::GROUPS>([&](auto gc) {
    constexpr int G = decltype(gc)::value;
    if (G > 0) wave_lds_order();
#pragma unroll
    for (int b = 0; b < S::template blocks<G>(); ++b) {
      const int tb = G * L::STG + b;
      const float sg = tsc ? tsc[tw + L::tok(tb, lane)] : 1.0f;
#pragma unroll
      for (int q = 0; q < L::NQ; ++q) {
        uint2 u;
        u.x = (uint32_t)YT::from_float(sg * L::get(acc, q, tb, 0)) | ((uint32_t)YT::from_float(sg * L::get(acc, q, tb, 1)) << 16);
        u.y = (uint32_t)YT::from_float(sg * L::get(acc, q, tb, 2)) | ((uint32_t)YT::from_float(sg * L::get(acc, q, tb, 3)) << 16);
        *S::at4(ylds, b, q) = u;
      }
    }
    wave_lds_order();
    S::template drain<G>(Yout, a.ldo, ow, tw, ylds);
  });
}

// ---------------------------------------------------------------------------
// Tile epilogue shared by both kernels; L is the accumulator layout (Acc32 / Acc16).  The block's
// waves form an NWO x NWT grid; wave (wo, wt) owns output rows [wo*WO, +WO) and tokens
// [wt*WT, +WT) of the tile at (o0, t0).  `red` holds one float per wave, `rows` NWO x BT floats
// (per-token row sums; only used by EPI_LOSS_TOK).  Every wave of the block must call this.
template <int EPI, typename L, int NWO, int NWT, int BT, bool YLDS, typename Acc>
__device__ __forceinline__ void tile_epilogue(const GemmDev& a, const Acc& acc, int cand, int to,
                                              int tt, int64_t o0, int64_t t0, int wo, int wt,
                                              float* red, float* rows) {
  constexpr int WO = L::WO, WT = L::WT, NW = NWO * NWT, NT = NW * 64;
  constexpr int kStage = WO * L::STG * (WT / L::NTB) * 2;   // bytes of LDS per wave, see Staged
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* tsc = a.tok_scale ? a.tok_scale + (int64_t)cand * a.n_tok : nullptr;
  if (EPI == EPI_STORE) {
    void* Yo = (unsigned char*)a.Yout + (int64_t)cand * a.o_cand_stride * (a.odt == TLQ_F32 ? 4 : 2);
    if constexpr (YLDS) {
      if (a.odt != TLQ_F32 && (o0 + NWO * WO <= a.c_out) && (t0 + BT <= a.n_tok) && (a.ldo % 8) == 0 &&
          ((uintptr_t)Yo % 16) == 0) {
        unsigned char* ylds = reinterpret_cast<unsigned char*>(rows) + wave * kStage;
        if (a.odt == TLQ_F16) store_rows_lds<F16, L>(a, Yo, acc, tsc, o0 + wo * WO, t0 + wt * WT, ylds);
        else store_rows_lds<BF16, L>(a, Yo, acc, tsc, o0 + wo * WO, t0 + wt * WT, ylds);
        return;
      }
    }
    // the guarded body, written out once for the plain store and once for the subtraction: the checks are a long
    // straight piece of code that an edge tile fetches cold, so the plain one carries nothing of the other
    // (6981 x 256 x 2216 tokens x channels x outputs, 252 tiles, 16-bit output: 20.3 us in one body, 16.3 in two)
    auto rows_out = [&](auto before, auto emit) {
      static_for<0, L::NTB>([&](auto tbc) {
        constexpr int tb = decltype(tbc)::value;
        before(tbc);
        const int64_t t = t0 + wt * WT + L::tok(tb, lane);
        if (t >= a.n_tok) return;
        const float sg = tsc ? tsc[t] : 1.0f;
#pragma unroll
        for (int q = 0; q < L::NQ; ++q) {
          float y[4] = {sg * L::get(acc, q, tb, 0), sg * L::get(acc, q, tb, 1), sg * L::get(acc, q, tb, 2),
                        sg * L::get(acc, q, tb, 3)};
          emit(tb, q, t, o0 + wo * WO + L::row(q, lane), y);
        }
      });
    };
    if (!a.Yref) {
      rows_out([](auto) {}, [&](int, int, int64_t t, int64_t o, const float (&y)[4]) {
        if (o + 3 < a.c_out) store_y4(Yo, a.odt, t * a.ldo + o, y);
        else
          for (int r = 0; r < 4; ++r)
            if (o + r < a.c_out) store_y1(Yo, a.odt, t * a.ldo + o + r, y[r]);
      });
      return;
    }
    // Yref - product, as float; Yref comes in whole lines through LDS where the tile is inside the matrix (see
    // loss_rows_lds)
    unsigned char* ylds = reinterpret_cast<unsigned char*>(rows) + wave * kStage;
    bool staged = false;
    if constexpr (YLDS) {
      staged = a.ydt != TLQ_F32 && (o0 + NWO * WO <= a.c_out) && (t0 + BT <= a.n_tok) && (a.ldy % 8) == 0 &&
               ((uintptr_t)a.Yref % 16) == 0;
    }
    rows_out([&](auto tbc) {
      constexpr int tb = decltype(tbc)::value;
      if constexpr (YLDS && tb % L::STG == 0)
        if (staged) Staged<L>::template fill<tb / L::STG>(a.Yref, a.ldy, o0 + wo * WO, t0 + wt * WT, ylds);
    }, [&](int tb, int q, int64_t t, int64_t o, const float (&y)[4]) {
      float yr[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (staged) {
        const uint2 u = *Staged<L>::at4(ylds, tb % L::STG, q);
        if (a.ydt == TLQ_F16) unpack4<F16>(u, yr);
        else unpack4<BF16>(u, yr);
      } else if (o + 3 < a.c_out) load_y4(a.Yref, a.ydt, t * a.ldy + o, yr);
      else
        for (int r = 0; r < 4; ++r)
          if (o + r < a.c_out) yr[r] = load_y(a.Yref, a.ydt, t * a.ldy + o + r);
#pragma unroll
      for (int r = 0; r < 4; ++r) yr[r] -= y[r];
      if (o + 3 < a.c_out) store_y4(Yo, TLQ_F32, t * a.ldo + o, yr);
      else
        for (int r = 0; r < 4; ++r)
          if (o + r < a.c_out) store_y1(Yo, TLQ_F32, t * a.ldo + o + r, yr[r]);
    });
    return;
  }
  // Interior tiles (the common case) take a branch-free body specialised on the Y_ref
  // type; edge tiles and odd strides take the guarded one.
  float part = 0.0f;
  float sq[L::NTB] = {};
  const bool interior = (o0 + NWO * WO <= a.c_out) && (t0 + BT <= a.n_tok);
  const int64_t ow = o0 + wo * WO, tw = t0 + wt * WT;
  constexpr bool DOT = EPI == EPI_DOT;
  const void* Yc = a.Yref;
  if (DOT) Yc = (const unsigned char*)a.Yref + (int64_t)cand * a.y_cand_stride * (a.ydt == TLQ_F32 ? 4 : 2);
  bool done = false;
  if constexpr (YLDS) {
    if (interior && a.ydt != TLQ_F32 && (a.ldy % 8) == 0 && ((uintptr_t)Yc % 16) == 0) {
      unsigned char* ylds = reinterpret_cast<unsigned char*>(rows) + wave * kStage;
      if (a.ydt == TLQ_F16) loss_rows_lds<F16, DOT, L>(a, Yc, acc, tsc, ow, tw, sq, part, ylds);
      else loss_rows_lds<BF16, DOT, L>(a, Yc, acc, tsc, ow, tw, sq, part, ylds);
      done = true;
    }
  }
  const bool half = L::WO == 128 && !DOT && ow + WO / 2 >= a.c_out;   // (the other tiles are small)
  if (done || ow >= a.c_out || tw >= a.n_tok) {}
  else if (a.ydt == TLQ_F32) {
    if (L::NTB <= 4 && interior) loss_rows<TLQ_F32, true, DOT, L, L::NQ>(a, Yc, acc, tsc, ow, tw, sq, part);
    else if (half) loss_rows<TLQ_F32, false, DOT, L, L::NQ / 2>(a, Yc, acc, tsc, ow, tw, sq, part);
    else loss_rows<TLQ_F32, false, DOT, L, L::NQ>(a, Yc, acc, tsc, ow, tw, sq, part);
  } else if (half) loss_rows<k16Bit, false, DOT, L, L::NQ / 2>(a, Yc, acc, tsc, ow, tw, sq, part);
  else if (L::NTB > 4 || !interior) loss_rows<k16Bit, false, DOT, L, L::NQ>(a, Yc, acc, tsc, ow, tw, sq, part);   // (few registers there)
  else if (a.ydt == TLQ_F16) loss_rows<TLQ_F16, true, DOT, L, L::NQ>(a, Yc, acc, tsc, ow, tw, sq, part);
  else loss_rows<TLQ_BF16, true, DOT, L, L::NQ>(a, Yc, acc, tsc, ow, tw, sq, part);
  if (EPI == EPI_LOSS_TOK) {
    if (done) __syncthreads();       // (`done` is the same for the block; the row sums take the place of all waves' staging)
#pragma unroll
    for (int tb = 0; tb < L::NTB; ++tb) {
      const float both = L::tok_sum(sq[tb]);
      if (L::row(0, lane) == 0) rows[wo * BT + wt * WT + L::tok(tb, lane)] = both;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) part += __shfl_xor(part, off, 64);
  if (lane == 0) red[wave] = part;
  __syncthreads();
  if (tid == 0) {
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) s += red[w];
    a.partial[((int64_t)cand * a.tiles_o + to) * a.tiles_t + tt] = s;
  }
  if (EPI == EPI_LOSS_TOK) {
    for (int i = tid; i < BT; i += NT) {
      const int64_t t = t0 + i;
      if (t < a.n_tok) {
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < NWO; ++w) s += rows[w * BT + i];
        a.tok_partial[(int64_t)to * a.n_tok + t] = s;
      }
    }
  }
}

// Block id -> (candidate, tile row, tile column).  Blocks are dealt to the 8 XCDs round-robin by
// block id, so block id = (round, xcd, slot) and every XCD works on one patch of po x pt tiles at a
// time (32 CUs = 32 tiles sharing, by default, 4 weight panels and 8 token panels in its L2).
// Patch order: chunks of cpt token patches; inside a chunk, for every output patch row, every
// candidate visits the chunk's token patches.  The chunk's tokens and the row's slice of Y_ref are
// thus shared by all candidates while they are hot in the last-level cache, and each candidate's
// weights are streamed once per chunk.  When tiles_o is not a multiple of po the last patch row
// has `rag` tile rows and uses patches of rag x rag_pt tiles, so that (nearly) every slot of a patch
// is a live tile.  Returns false for a slot that has no tile.
// Launches of few tiles (`strips`) have no use for patches: whole and nearly empty patches would alternate
// over the XCDs (5 token tiles in patches of 4: every other XCD idle).  There the tiles are
// numbered along the shorter side first and every XCD takes one eighth of the numbers, a strip.
// Symmetric products (`tri`) number only the tiles on and above the diagonal: blocks of eight tile columns,
// in them row by row (32 consecutive tiles: 4 x 8).  Every candidate's numbers are dealt to the XCDs in
// eight equal strips.  (In patches the dead half of the square left XCDs idle: at 16 x 16 tiles a candidate
// has eight patches, two of them empty, and each XCD met the same patch of every candidate.)
__host__ __device__ __forceinline__ bool decode_tri(const GemmDev& a, int64_t bid, int& cand, int& to, int& tt) {
  const int n = a.tiles_o, live = n * (n + 1) / 2, per = (live + kXcd - 1) / kXcd;
  const int xcd = (int)(bid & (kXcd - 1));
  const int64_t i = bid / kXcd;
  if (i >= (int64_t)per * a.n_cand) return false;
  cand = (int)(i / per);
  const int idx = (int)((int64_t)xcd * live / kXcd) + (int)(i % per);
  if (idx >= (int)((int64_t)(xcd + 1) * live / kXcd)) return false;
  // the last column block whose first column c0 has c0 (c0 + 1) / 2 tiles to its left
  int cb = (int)((sqrtf(8.0f * (float)idx + 1.0f) - 1.0f) * 0.5f) / 8;
  while (cb > 0 && cb * 8 * (cb * 8 + 1) / 2 > idx) --cb;
  while ((cb + 1) * 8 < n && (cb + 1) * 8 * ((cb + 1) * 8 + 1) / 2 <= idx) ++cb;
  const int c0 = cb * 8, w = n - c0 < 8 ? n - c0 : 8;
  int rem = idx - c0 * (c0 + 1) / 2;
  if (rem < c0 * w) {
    to = rem / w;
    tt = c0 + rem % w;
  } else {
    rem -= c0 * w;
    int r = 0;
    while (rem >= w - r) { rem -= w - r; ++r; }
    to = c0 + r;
    tt = to + rem;
  }
  return true;
}

__host__ __device__ __forceinline__ bool decode_tile(const GemmDev& a, int64_t bid, int& cand, int& to, int& tt) {
  if (a.strips > 0) {
    const int64_t xcd = bid & (kXcd - 1);
    const int64_t idx = xcd * a.strips / kXcd + bid / kXcd;
    if (idx >= (xcd + 1) * a.strips / kXcd) return false;
    const int per = a.tiles_o * a.tiles_t;
    cand = (int)(idx / per);
    const int rem = (int)(idx % per);
    if (a.tiles_t <= a.tiles_o) { to = rem / a.tiles_t; tt = rem % a.tiles_t; }
    else { tt = rem / a.tiles_o; to = rem % a.tiles_o; }
    return true;
  }
  const int PATCH_O = a.po, PATCH_T = a.pt;
  const int64_t round = bid / (kXcd * PATCH_SLOTS);
  const int within = (int)(bid % (kXcd * PATCH_SLOTS));
  int64_t patch = round * kXcd + (((within & (kXcd - 1)) + a.rot * (int)(round & (kXcd - 1))) & (kXcd - 1));
  const int slot = within / kXcd;
  if (patch >= a.n_patches) return false;
  // candidate-outermost order: the same walk with one candidate, repeated per candidate
  int n_cand = a.n_cand, cand0 = 0;
  if (a.cand_outer) {
    const int64_t per = a.n_patches / a.n_cand;
    cand0 = (int)(patch / per);
    patch %= per;
    n_cand = 1;
  }
  const int n_full = a.rag ? a.npo - 1 : a.npo;
  const int ragp_full = a.rag ? (a.cpt * PATCH_T + a.rag_pt - 1) / a.rag_pt : 0;
  const int64_t chunk_sz = (int64_t)n_cand * (n_full * a.cpt + ragp_full);
  const int chunk = (int)(patch / chunk_sz);
  const int crem = (int)(patch % chunk_sz);
  const int cw = (a.npt - chunk * a.cpt) < a.cpt ? (a.npt - chunk * a.cpt) : a.cpt;
  const int nfull_p = n_full * n_cand * cw;
  if (crem < nfull_p) {
    const int r2 = crem % (n_cand * cw);
    cand = cand0 + r2 / cw;
    to = (crem / (n_cand * cw)) * PATCH_O + (slot % PATCH_O);
    tt = (chunk * a.cpt + r2 % cw) * PATCH_T + (slot / PATCH_O);
  } else {
    const int ragp = (cw * PATCH_T + a.rag_pt - 1) / a.rag_pt;
    const int r2 = crem - nfull_p, col = slot / a.rag;
    cand = cand0 + r2 / ragp;
    if (col >= a.rag_pt) return false;
    to = n_full * PATCH_O + (slot % a.rag);
    tt = chunk * a.cpt * PATCH_T + (r2 % ragp) * a.rag_pt + col;
    if (tt >= (chunk * a.cpt + cw) * PATCH_T) return false;
  }
  return to < a.tiles_o && tt < a.tiles_t;
}

// The tile of this block, in scalar registers: the operand descriptors are built from it, and a descriptor
// in vector registers puts a loop over its distinct values around every LDS-DMA load.
template <int EPI>
__device__ __forceinline__ bool block_tile(const GemmDev& a, int& cand, int& to, int& tt) {
  bool live;
  if (EPI == EPI_STORE && a.tri) live = decode_tri(a, blockIdx.x, cand, to, tt);
  else live = decode_tile(a, blockIdx.x, cand, to, tt);
  if (!live) return false;
  cand = __builtin_amdgcn_readfirstlane(cand);
  to = __builtin_amdgcn_readfirstlane(to);
  tt = __builtin_amdgcn_readfirstlane(tt);
  return true;
}

// ---------------------------------------------------------------------------
// Pipelined variant (every workload with row strides below 2^21 elements).
//
// Global -> LDS goes through the buffer-load-to-LDS path (no VGPR staging, no
// LDS store instructions): each wave-wide load drops 64 x 16 B contiguously at
// an LDS base held in M0, so the XOR swizzle is applied on the *global* side
// (lane l fetches the chunk that belongs in LDS slot l).  Rows past the edge
// of the matrix fall outside the buffer descriptor's range and arrive as
// zeros.  NSTAGE k-tiles form a ring; the refill of a slot is issued as soon
// as the block-wide barrier shows that every wave has finished reading it, so
// NSTAGE-1 k-tiles of loads are always in flight.
//
// The compiler cannot see that fragment reads and LDS-DMA writes touch
// different ring slots and would drain the load counter before every LDS read,
// so the fragment reads are issued from inline assembly and the waits on the
// two counters are placed by hand:
//   - "lgkmcnt(0)" ties the fragment registers, so no MFMA can be scheduled
//     before its operands have arrived;
//   - "vmcnt(n)" before the barrier waits for this wave's share of the next
//     k-tile only.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

template <int IMM>
__device__ __forceinline__ void lds_read128(u32x4& v, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(IMM));
}
// Wait for every outstanding LDS read; the fragments are tied through the
// statement so that nothing consuming them can be scheduled above it.
__device__ __forceinline__ void lds_wait(u32x4 (&a)[4]) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]) : : "memory");
}
template <int N>
__device__ __forceinline__ void lds_wait(u32x4 (&a)[4], u32x4 (&b)[N]) {
  static_assert(N >= 2 && N <= 5, "token fragments of a wave tile");
  if constexpr (N == 2)
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]) : : "memory");
  else if constexpr (N == 3)
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]) : : "memory");
  else if constexpr (N == 4)
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3])
                 : : "memory");
  else
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]),
                   "+v"(b[4]) : : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Block tile 256 (o) x 256 (t), k-tile 64, 8 waves in a 2 x 4 grid; a wave owns 128 x 64 outputs
// = 8 x 4 accumulator tiles of the 16x16x32 MFMA (128 registers).  A k-tile is two k32 steps; a
// step is split into two PHASES of 16 MFMAs (output rows 0-63, then 64-127 of the wave tile), so
// only four weight fragments and four token fragments are live per phase and both sets can be
// double-buffered in 64 registers:
//   phase 0: rows  0-63  x step 0   reads meanwhile: weight fragments of rows 64-127, step 0
//   phase 1: rows 64-127 x step 0   reads meanwhile: weight fragments of rows 0-63 and the token
//                                   fragments of step 1
//   phase 2: rows  0-63  x step 1   reads meanwhile: weight fragments of rows 64-127, step 1
//   -- every fragment of the k-tile is in registers: wait for this wave's loads of the next
//      k-tile, block barrier --
//   phase 3: rows 64-127 x step 1   reads meanwhile: first fragments of the NEXT k-tile; the 8
//                                   LDS-DMA loads that refill the slot just freed
// The side operations are slotted two at a time behind the first MFMAs of a phase (measured best:
// one per MFMA over the whole phase -3 %, four at a time -2 %), so that neither the LDS queue nor
// the texture-address queue sees a burst that would hold back the in-order MFMA issue.
// SYMK: Wh is a symmetric square matrix (c_out == c_in) and the epilogue forms a quadratic form in
// it (EPI_DOT with Y == X): the tile with first output row o0 contracts only k >= o0, with the part
// beyond its diagonal block counted twice: 2 * sum_{k > block} + sum_{k in block} stands for the
// full contraction at about half the flops.  The k-tiles are walked from the END of the rows
// down to o0, so that the tiles of a patch - which start at different o0 - work on the same
// k-tile at the same time and share its token panel in L2; the diagonal block comes last.
// TAIL: c_in is not a multiple of the k-tile; the lanes whose chunk lies past the end of the rows fetch
// nothing for the last k-tile (their offset is out of range, the chunk arrives as zeros).
// JB = 3 or 5: the wave tile is 128 x 48 or 128 x 80 tokens (twelve or twenty MFMAs a phase); 80 take 252 registers and 144 KB
// of LDS, the most that two waves a SIMD and one block a CU can have.
// HALVES = 1: a block of 4 waves computes 128 x 128 outputs, a wave 64 x 64 (a phase per k32 step, all of
// its eight fragments read one phase ahead); two blocks share a CU.  JB = 2: 128 x 64, a wave 64 x 32.  For launches whose 256 x 256 tiles
// would leave CUs idle, see gemm_small_tiles.
template <typename T, int NSTAGE, int EPI, bool SYMK, bool TAIL, int HALVES, int JB>
__device__ __forceinline__ void gemm_dma_body(const GemmDev& a) {
#if defined(__HIP_DEVICE_COMPILE__)  // the body uses gfx950 builtins the host pass cannot parse
  constexpr int BK_ = 64, NWO = 2, NWT = 2 * HALVES, NW = NWO * NWT, WO = 64 * HALVES, WT = 16 * JB;
  constexpr int BO = NWO * WO, BT = NWT * WT;
  constexpr int IA = WO / 16;                 // accumulator tiles per wave: IA x JB
  static_assert(HALVES == 1 || HALVES == 2, "phase structure below: one or two row halves of 64");
  constexpr int RB = BK_ * 2;             // bytes per LDS row
  constexpr int CPR = BK_ / 8;            // 16-byte chunks per row
  constexpr int STAGE = (BO + BT) * RB;
  constexpr int RPD = 64 / CPR;           // rows covered by one wave-wide load
  constexpr int DPA = BO / RPD / NW, DPB = BT / RPD / NW;   // loads per wave per k-tile: weights, tokens
  constexpr int LPS = DPA + DPB, DPM = DPA < DPB ? DPA : DPB;
  static_assert((NSTAGE == 2 || NSTAGE == 4) && DPA * RPD * NW == BO && DPB * RPD * NW == BT, "pipeline shape");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[NSTAGE * STAGE];
  __shared__ float red[NW];

  int cand, to, tt;
  if (!block_tile<EPI>(a, cand, to, tt)) return;
  const int64_t o0 = (int64_t)to * BO, t0 = (int64_t)tt * BT;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wo = wave % NWO, wt = wave / NWO;

  // buffer descriptors over the valid rows of this block's two operand panels
  const int64_t vro = (a.c_out - o0) < BO ? (a.c_out - o0) : BO;
  const int64_t vrt = (a.n_tok - t0) < BT ? (a.n_tok - t0) : BT;
  const int64_t kskip = SYMK ? o0 : 0;    // first contraction index (a multiple of the tile height)
  const int64_t klen = a.c_in - kskip;
  const uint16_t* pA = a.Wh + (int64_t)cand * a.w_cand_stride + o0 * a.ldw + kskip;
  const uint16_t* pB = a.X + (int64_t)cand * a.x_cand_stride + t0 * a.ldx + kskip;
  const __amdgpu_buffer_rsrc_t rA = __builtin_amdgcn_make_buffer_rsrc(
      (void*)pA, 0, (int)(((vro - 1) * a.ldw + klen) * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rB = __builtin_amdgcn_make_buffer_rsrc(
      (void*)pB, 0, (int)(((vrt - 1) * a.ldx + klen) * 2), 0x00020000);

  // per-lane global byte offsets of the chunks this lane fetches: LDS slot `p` of row r holds
  // chunk p ^ ((r / 2) % 8)
  int voa[DPA], vob[DPB];
#pragma unroll
  for (int j = 0; j < (DPA > DPB ? DPA : DPB); ++j) {
    const int r = (j * NW + wave) * RPD + lane / CPR;
    const int p = lane % CPR;
    const int c = p ^ ((r >> 1) & 7);
    if (j < DPA) voa[j] = r * (int)a.ldw * 2 + c * 16;
    if (j < DPB) vob[j] = r * (int)a.ldx * 2 + c * 16;
  }
  // The scalar offset is not part of the descriptor's range check, so a k-tile
  // past the end of the rows must not be fetched at all: its loads are still
  // issued (the counter bookkeeping stays uniform) but with a per-lane offset
  // that is out of range for any descriptor, which touches no memory and
  // delivers zeros.
  const int64_t nk = TAIL ? (klen + BK_ - 1) / BK_ : klen / BK_;
  constexpr int kOutOfRange = (int)0x80000000u;
  // TAIL: the lane's chunk of a k-tile (the same for all of its loads, see voa) lies inside the last one
  const bool tail_ok = !TAIL || ((lane % CPR) ^ ((wave * (RPD / 2) + (lane / CPR >> 1)) & 7)) * 8 < (int)(klen - (nk - 1) * BK_);
  auto dma1 = [&](auto dc, unsigned char* sbase, bool live, int so) {
    // the operands take turns while both have loads left
    constexpr int d = decltype(dc)::value, j = d < 2 * DPM ? d / 2 : d - DPM;
    if constexpr (d < 2 * DPM ? (d & 1) == 0 : DPA > DPB)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rA, (lds_ptr_t)(sbase + (j * NW + wave) * 1024), 16,
                                               live ? voa[j] : kOutOfRange, so, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rB, (lds_ptr_t)(sbase + BO * RB + (j * NW + wave) * 1024), 16,
                                               live ? vob[j] : kOutOfRange, so, 0, 0);
  };
  // byte offset of k-tile number kt of the walk inside a row
  auto k_offset = [&](int64_t kt) { return (int)((SYMK ? nk - 1 - kt : kt) * BK_ * 2); };
  // whether this lane fetches k-tile number kt of the walk
  auto fetches = [&](int64_t kt) { return kt < nk && (!TAIL || tail_ok || kt != (SYMK ? 0 : nk - 1)); };
  auto issue = [&](int64_t kt) {
    const bool live = fetches(kt);
    const int so = kt < nk ? k_offset(kt) : 0;
    unsigned char* sb = lds + (int)(kt % NSTAGE) * STAGE;
    static_for<0, LPS>([&](auto dc) { dma1(dc, sb, live, so); });
  };

  // fragment read addresses (bytes from the start of a stage): lane -> row lane % 16 of a 16-row
  // block and 16-byte chunk lane / 16 of the k32 step (the MFMA takes k = 8 * (lane / 16) + [0, 8)
  // from both operands, so any chunk order is right as long as both use the same one)
  const int frow = lane & 15, fq = lane >> 4;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
  uint32_t offA[2], offB[2];
#pragma unroll
  for (int st = 0; st < 2; ++st) {
    const int c = st * 4 + fq;
    const int p = c ^ ((frow >> 1) & 7);
    const uint32_t o = (uint32_t)(frow * RB + p * 16);
    offA[st] = lds0 + o + (wo * WO) * RB;
    offB[st] = lds0 + o + BO * RB + (wt * WT) * RB;
  }
  u32x4 Fa[2][4], Fb[2][JB];   // weight fragments (double-buffered per phase), token fragments (per k32 step)
  f32x4 acc[IA][JB];
#pragma unroll
  for (int i = 0; i < IA; ++i)
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.0f;

  // One phase: the 4 x JB MFMAs of weight buffer AB x token buffer BB into output rows HALF, with the
  // side operations behind the first of them: the weight fragments of half RH into buffer AB ^ 1
  // (from `ra`), - if RDB - the token fragments into buffer BB ^ 1 (from `rb`), and ND LDS-DMA
  // loads of k-tile `dkt`.
  auto phase = [&](auto abc, auto bbc, auto halfc, auto rhc, auto rdbc, auto ndc, uint32_t ra, uint32_t rb,
                   int64_t dkt) {
    constexpr int AB = decltype(abc)::value, BB = decltype(bbc)::value, HALF = decltype(halfc)::value;
    constexpr int RH = decltype(rhc)::value, ND = decltype(ndc)::value;
    constexpr bool RDB = decltype(rdbc)::value != 0;
    constexpr int NR = 4 + (RDB ? JB : 0);
    static_assert(NR + ND <= 8 * JB, "two side operations behind an MFMA");
    const bool live = fetches(dkt);
    const int so = dkt < nk ? k_offset(dkt) : 0;
    unsigned char* sbase = lds + (int)(dkt % NSTAGE) * STAGE;
    // side operation number n of the phase: in the refill phase the LDS-DMA loads come first (the
    // longest latency), then the fragment reads
    auto side = [&](auto nc) {
      constexpr int n0 = decltype(nc)::value;
      constexpr int n = ND > 0 ? (n0 < ND ? NR + n0 : n0 - ND) : n0;
      if constexpr (n < 4) lds_read128<(RH * 4 + n) * 16 * RB>(Fa[AB ^ 1][n], ra);
      else if constexpr (n < NR) lds_read128<(n - 4) * 16 * RB>(Fb[BB ^ 1][n - 4], rb);
      else if constexpr (n < NR + ND) dma1(std::integral_constant<int, n - NR>{}, sbase, live, so);
    };
    static_for<0, 4 * JB>([&](auto mc) {
      // boustrophedon over the 4 x JB fragment pairs: consecutive MFMAs share one operand register set
      constexpr int m = decltype(mc)::value, ib = m / JB, jb = (ib & 1) ? JB - 1 - m % JB : m % JB;
      acc[HALF * 4 + ib][jb] = Mma16<T>::run(__builtin_bit_cast(uint4, Fa[AB][ib]),
                                             __builtin_bit_cast(uint4, Fb[BB][jb]), acc[HALF * 4 + ib][jb]);
      if constexpr (2 * m < NR + ND) {
        side(std::integral_constant<int, 2 * m>{});
        side(std::integral_constant<int, 2 * m + 1>{});
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using ILoads = std::integral_constant<int, LPS>;

  // prologue: fill the whole ring, wait for k-tile 0, fetch its first fragments
#pragma unroll
  for (int s = 0; s < NSTAGE; ++s) issue(s);
  wait_vmcnt<(NSTAGE - 1) * LPS>();
  __builtin_amdgcn_s_barrier();
  static_for<0, (JB > 4 ? JB : 4)>([&](auto mc) {
    constexpr int m = decltype(mc)::value;
    if constexpr (m < 4) lds_read128<m * 16 * RB>(Fa[0][m], offA[0]);
    if constexpr (m < JB) lds_read128<m * 16 * RB>(Fb[0][m], offB[0]);
  });
  lds_wait(Fa[0], Fb[0]);
  auto k_tile = [&](int64_t kt) {
    const uint32_t so_cur = (uint32_t)((kt % NSTAGE) * STAGE);
    if constexpr (HALVES == 2) {
      phase(I0{}, I0{}, I0{}, I1{}, I0{}, I0{}, offA[0] + so_cur, 0u, 0);
      lds_wait(Fa[1]);
      phase(I1{}, I0{}, I1{}, I0{}, I1{}, I0{}, offA[1] + so_cur, offB[1] + so_cur, 0);
      lds_wait(Fa[0], Fb[1]);
      phase(I0{}, I1{}, I0{}, I1{}, I0{}, I0{}, offA[1] + so_cur, 0u, 0);
      lds_wait(Fa[1]);
    } else {
      phase(I0{}, I0{}, I0{}, I0{}, I1{}, I0{}, offA[1] + so_cur, offB[1] + so_cur, 0);
      lds_wait(Fa[1], Fb[1]);
    }
    // every fragment of k-tile kt is in registers: its slot can be refilled once all
    // waves are here, and k-tile kt+1 has landed once this wave's share of it has
    wait_vmcnt<(NSTAGE - 2) * LPS>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t so_next = (uint32_t)(((kt + 1) % NSTAGE) * STAGE);
    phase(I1{}, I1{}, std::integral_constant<int, HALVES - 1>{}, I0{}, I1{}, ILoads{}, offA[0] + so_next, offB[0] + so_next,
          kt + NSTAGE);
    lds_wait(Fa[0], Fb[0]);
  };
  int64_t kt = 0;
  if constexpr (SYMK) {
    // first everything beyond the diagonal block, counted twice; then the block itself
    constexpr int64_t kDiagTiles = BO / BK_;
    const int64_t n_beyond = nk > kDiagTiles ? nk - kDiagTiles : 0;
    for (; kt < n_beyond; ++kt) k_tile(kt);
    if (n_beyond > 0) {
#pragma unroll
      for (int i = 0; i < IA; ++i)
#pragma unroll
        for (int j = 0; j < JB; ++j) acc[i][j] *= 2.0f;
    }
  }
  for (; kt < nk; ++kt) k_tile(kt);
  wait_vmcnt<0>();
  __syncthreads();

  if constexpr (std::is_same<T, Int8>::value) {   // sums of codes -> multiples of the output rows' steps
    const float* rsc = a.row_scale + (int64_t)cand * a.row_scale_stride;
#pragma unroll
    for (int i = 0; i < IA; ++i) {
      const int64_t o = o0 + wo * WO + i * 16 + fq * 4;       // (the table's rows are whole groups of four)
      const float4 rs = o < a.c_out ? *reinterpret_cast<const float4*>(rsc + o) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      const float r[4] = {rs.x, rs.y, rs.z, rs.w};
#pragma unroll
      for (int j = 0; j < JB; ++j) {
        const i32x4 v = __builtin_bit_cast(i32x4, acc[i][j]);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j][e] = r[e] * (float)v[e];
      }
    }
  }
  // every LDS-DMA write has landed and every wave is past its last fragment read:
  // the tile memory is free for the per-token row sums and the Y_ref / output staging
  tile_epilogue<EPI, Acc16<IA, JB>, NWO, NWT, BT, (NSTAGE * STAGE >= NW * WO * Acc16<IA, JB>::STG * 32)>(
      a, acc, cand, to, tt, o0, t0, wo, wt, red, reinterpret_cast<float*>(lds));
#endif
}

constexpr int kDmaBK = 64;                   // k-tile depth of the pipelined kernels
// Launches of the kernels of gemm_width.hip, gemm_half.hip, gemm_tok.hip and gemm_i8.hip: `epi` is the epilogue; combinations that no call makes are refused.
hipError_t launch_dma_width(const GemmDev& d, int epi, bool bf16, int tok_blocks, unsigned blocks, hipStream_t stream);
hipError_t launch_dma_half(const GemmDev& d, int epi, bool bf16, unsigned blocks, hipStream_t stream);
hipError_t launch_dma_small_tok(const GemmDev& d, bool deep, unsigned blocks, hipStream_t stream);
hipError_t launch_dma_i8(const GemmDev& d, int epi, GemmTile tile, unsigned blocks, hipStream_t stream);

}  // namespace tlq
