// Internal declarations shared by the libtlq translation units (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "tlq.h"

namespace tlq {

constexpr float kXstatFloor = 6.103515625e-05f;  // 2^-14
constexpr float kRangeFloor = 1e-5f;

// 16-bit element types as raw bit patterns with exact widening to float.
struct F16 {
  using raw = _Float16;
  static __device__ __forceinline__ float to_float(uint16_t b) {
    return (float)__builtin_bit_cast(_Float16, b);
  }
  static __device__ __forceinline__ uint16_t from_float(float f) {
    return __builtin_bit_cast(uint16_t, (_Float16)f);  // round-to-nearest-even
  }
};
struct BF16 {
  using raw = __bf16;
  static __device__ __forceinline__ float to_float(uint16_t b) {
    return __builtin_bit_cast(float, (uint32_t)b << 16);
  }
  static __device__ __forceinline__ uint16_t from_float(float f) {
    // v_cvt_pk_bf16_f32: round-to-nearest-even, quiet NaN; bit-equal to the integer formula
    // (u + 0x7fff + lsb) >> 16 over all 2^32 floats, in one instruction for two values instead of
    // seven for one
    return __builtin_bit_cast(uint16_t, (__bf16)f);
  }
};

// 16-byte accesses.  NT: past the caches, for streams that no cache could hold until their next use (see streams_past)
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
template <bool NT>
__device__ __forceinline__ uint4 load16(const void* p) {
  u32x4v v;
  if constexpr (NT) v = __builtin_nontemporal_load(reinterpret_cast<const u32x4v*>(p));
  else v = *reinterpret_cast<const u32x4v*>(p);
  return make_uint4(v[0], v[1], v[2], v[3]);
}
template <bool NT>
__device__ __forceinline__ void store16(void* p, const uint4& v) {
  const u32x4v t = {v.x, v.y, v.z, v.w};
  if constexpr (NT) __builtin_nontemporal_store(t, reinterpret_cast<u32x4v*>(p));
  else *reinterpret_cast<u32x4v*>(p) = t;
}
template <bool NT>
__device__ __forceinline__ void store8(void* p, uint32_t a, uint32_t b) {
  typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
  const u32x2v t = {a, b};
  if constexpr (NT) __builtin_nontemporal_store(t, reinterpret_cast<u32x2v*>(p));
  else *reinterpret_cast<u32x2v*>(p) = t;
}
// the same by a flag that is the same for the whole launch (the empty statements keep the compiler from making one
// plain store of the two)
__device__ __forceinline__ void store16(void* p, const uint4& v, bool nt) {
  if (nt) { asm volatile("" ::: "memory"); store16<true>(p, v); asm volatile("" ::: "memory"); } else store16<false>(p, v);
}
__device__ __forceinline__ void store8(void* p, uint32_t a, uint32_t b, bool nt) {
  if (nt) { asm volatile("" ::: "memory"); store8<true>(p, a, b); asm volatile("" ::: "memory"); } else store8<false>(p, a, b);
}
// Bytes of a call from which what it only reads is better off past the 256 MB last-level cache, us plain -> past it: the residual
// sum, 288 MB read and written 43.8 -> 44.8, 384 MB 65.7 -> 57.8, 1152 MB 194 -> 175; gradient norms, 256 MB 46.7 ->
// 46.8, 320 MB 62 -> 58, 1500 MB 306 -> 263; the statistic, 256 MB 40.9 -> 49.4, 320 MB 63.4 -> 60.5, 1500 MB 279 -> 267.
inline bool streams_past(double bytes) { return bytes > 320e6; }
// Bytes of an output from which it is: below, the call that reads it next finds it there, all the more if the inputs went
// past.  Two calls in a row, us all plain, loads past, loads and stores past: residual sum and norm with an output of
// 107 MB 94, 92, 99, of 168 MB 137, 132, 147; gate of 113 MB and the product behind it 222, 183, 253, of 224 MB 323, 301, 313,
// of 252 MB 342, 331, 338; norm and product, 200 MB 273, 232, 265, 240 MB 310, 302, 300; bf16 tokens to fp16 and a loss, 201 MB
// 235, 197, 210, 224 MB 253, 216, 223, 240 MB 262, 234, 231, 252 MB 269, 247, 237.  (A producer alone, over and over the same
// buffers, has no reader: there the conversion of 200 MB takes 110 us with plain stores, 95 with stores past.)
inline bool outgrows_cache(double bytes) { return bytes > 230e6; }

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---- profiling hooks (profile.cpp) ----------------------------------------
struct ProfScope {
  ProfScope(const char* name, hipStream_t stream, double work);
  ~ProfScope();
  int slot;
  hipStream_t stream;
  unsigned generation;
};

// ---- kernel launchers (each enqueues on `stream`, returns hipGetLastError) --
// S0: column mean/max of |X|; partial: double [n_chunks, c_in]
int xstat_chunks(int64_t n_tok);
// Rows up to which one launch is faster than two (a whole search of 20 candidates, us two launches -> one, at 512 and at
// 4096 channels: 256 rows 39.4 -> 37.6 and 86.0 -> 84.0, 1024 rows 40.0 -> 38.8 and 87.9 -> 87.4, 2048 rows
// 41.2 -> 41.8 and 97.8 -> 100.0; the statistic alone, calls in a row: 16 - 512 rows 7.9 -> 4.7, 1024 x 4096 7.9 -> 5.1).  Not
// where the token maximum is taken along: a block sees 64 channels only.
constexpr int64_t kDirectRows = 1024;
// Channels up to which that holds for the statistic alone: one block a CU, a second round of them costs more than the other launch
// (us two -> one, mean and maximum: 64 x 16,384 6.2 -> 5.4 and 6.7 -> 5.7, 1000 x 16,384 8.5 -> 6.4 and 9.5 -> 7.6; 64 x 18,432 6.3 -> 7.5
// and 6.8 -> 8.7, 1000 x 18,432 10.4 -> 10.8 and 12.2 -> 14.2, 64 x 131,072 9.3 -> 21.6 and 10.2 -> 28.2).
constexpr int64_t kDirectCols = 64 * 256;
// pos_mask (optional): only rows r with pos_mask[r % period] != 0 take part
hipError_t launch_xstat(const void* X, int64_t n_tok, int64_t c_in, int64_t ldx, bool bf16,
                        int kind, double* partial, float* x_stat, hipStream_t stream,
                        const uint8_t* pos_mask = nullptr, int64_t period = 1);
// gradient-guided token selection (select.hip)
hipError_t launch_token_importance(const void* G, int64_t n_samples, int64_t n_pos, int64_t c, int64_t ldg,
                                   bool bf16, bool l2, double* row_norm, double* sum_n, hipStream_t stream);
hipError_t launch_topk_mask(const double* sum_n, int64_t n_pos, int64_t k, uint8_t* mask, hipStream_t stream);
// S1
// inv_table (optional) = 2^shift / s, where shift comes from `xmax_bits` (see launch_xprep) or is 0; s_copy
// (optional): a second place for the table
hipError_t launch_scale_table(const float* x_stat, int64_t c_in, const float* alpha, int n_alpha,
                              float* s_table, float* s_copy, float* inv_table, const uint32_t* xmax_bits,
                              hipStream_t stream);
// S0 + S1 without the statistic itself.  block_max (bf16 tokens; optional): scratch of xstat_block_max_words words; then
// max|X| comes from the same pass, goes to *xmax_out and sets the shift instead of xmax_bits
size_t xstat_block_max_words(int64_t n_tok, int64_t c_in);
hipError_t launch_xstat_table(const void* X, int64_t n_tok, int64_t c_in, int64_t ldx, bool bf16, int kind, double* partial,
                              const float* alpha, int n_alpha, float* s_table, float* s_copy, float* inv_table,
                              const uint32_t* xmax_bits, uint32_t* block_max, uint32_t* xmax_out, hipStream_t stream);
// inv[c] = 2^shift / s[c]
hipError_t launch_recip(const float* s, int64_t c_in, const uint32_t* xmax_bits, float* inv,
                        hipStream_t stream);

// bf16 activations re-expressed in fp16.  A bf16 value has 8 significant bits, so
// X * 2^-shift is exact in fp16 once shift keeps the largest magnitude below 2^15
// (values more than 2^32 below that maximum lose low bits - far below anything the
// loss can see).  xmax_bits receives the bit pattern of max|X|; every consumer derives
// the same shift from it.  The folded weights carry the factor 2^shift, so the
// contraction is unchanged while its computed operand is rounded to 11 instead of 8
// significant bits.
// Tokens up to this size go through one launch (calls in a row, us, three launches -> one: 8 - 256 KB 10.4 -> 4.9, 512 KB 10.5
// -> 7.1; at 1 MB every block would read as much as 64 KB cost in launches).  Beyond it, with room for words, two: products
// of bf16 tokens with their own reciprocals, 4000 x 640 x 600 36.4 -> 23.4, 1200 x 5120 x 13824 205 -> 200.
inline bool xprep_whole(int64_t n_tok, int64_t c_in) { return n_tok * c_in * 2 <= 512 << 10; }
// have_max: xmax_bits holds the maximum already.  words: scratch of `room` bytes for the maxima of blocks, which saves a launch
// (NULL: none).  s, inv: also inv[c] = 2^shift / s[c] (NULL: not).
hipError_t launch_xprep(const void* X, int64_t n_tok, int64_t c_in, int64_t ldx, uint32_t* xmax_bits,
                        void* Xh, hipStream_t stream, bool have_max = false, uint32_t* words = nullptr, size_t room = 0,
                        const float* s = nullptr, float* inv = nullptr);
__host__ __device__ inline int shift_from_bf16_bits(uint32_t bits) {
  const int k = (int)((bits >> 7) & 0xffu) - 141;  // |x| < 2^(e-126); want < 2^15
  return k < 0 ? 0 : (k > 24 ? 24 : k);
}

// S2.  Quantises W*diag(s_k) for n_cand candidates (s_table row stride c_in).
// what:  folded operand deq/s as fp16 [n_cand, c_out, c_in] (row stride c_in), or NULL: then
// codes/zp/delta/wdq, the single-candidate outputs (each may be NULL), are written instead
struct QuantArgs {
  const void* W; int64_t c_out, c_in, ldw; bool bf16;
  int bits, group, symmetric;
  const float* s_table;   // [n_cand, c_in] or NULL (ones)
  const float* inv_table; // [n_cand, c_in] or NULL (ones); used only for `what`
  int n_cand;
  void* what; int64_t what_cand_stride;  // elements between candidates
  uint8_t* codes; uint8_t* zp; float* delta; void* wdq; int64_t ld_dq;
  // difference form: `what` receives deq*inv - W*2^shift (shift from xmax_bits, 0 when NULL)
  bool diff; const uint32_t* xmax_bits;
  const float* col_scale;   // [c_in] factor applied to `what` after everything else, or NULL
  // integer form (w8 given; a group must be a whole row of at most 16384 channels): instead of `what`, the codes less
  // their zero point as int8 rows of `ld8` bytes (zeros behind c_in) and the steps [n_cand, step_stride]
  int8_t* w8; int64_t ld8, w8_cand_stride; float* steps; int64_t step_stride;
};
hipError_t launch_fake_quant(const QuantArgs& a, hipStream_t stream);

// Q_a: per-token symmetric activation fake-quant of X * diag(inv_k) for candidates k0 .. k0+nb-1.
// inv_table: [.., c_in] rows (row k used for candidate k) or NULL (ones).
// codes: fp16 integers [nb, n_tok, c_in], or with ld8 > 0 int8 rows of ld8 bytes, zeros behind c_in; sigma: float
// [nb, n_tok] (already offset to k0).
hipError_t launch_act_quant(const void* X, int64_t n_tok, int64_t c_in, int64_t ldx, bool bf16,
                            const float* inv_table, int k0, int nb, int act_bits, void* codes,
                            float* sigma, hipStream_t stream, int64_t ld8 = 0);

// Wout[o,c] = round16(Win[o,c] * inv_s[c])
hipError_t launch_fold_scale(const void* Win, int64_t c_out, int64_t c_in, int64_t ldw, bool bf16,
                             const float* inv_s, const uint32_t* xmax_bits, bool out_f16, void* Wout,
                             hipStream_t stream);

// S4 final combine + S5 selection: losses[k] = inv_c_out * factor * the sum of partial[k, 0 .. tiles), the first
// smallest of them, its row of the table.  best_idx, best_scales and factor (then 1) may be NULL.
struct FinalDev {
  const float* partial; int n_cand; int64_t tiles; double inv_c_out; const double* factor;
  const float* s_table; int64_t c_in; float* losses; int32_t* best_idx; float* best_scales;
};

// Output tile of the pipelined contraction: 256 rows x 64 tok_blocks tokens (3, 4 or 5 blocks of 16 tokens a wave; 0 = 4),
// or small: 128 rows x 32 tok_blocks (0 = 4, or 2: 128 x 64, not of integer codes), for stores (with tri only 128 x 128) and fp16 losses
// (128 x 128 with tok_partial: tok_blocks has to say 4).
// gemm_tile says which is the fastest.
struct GemmTile { bool small; int tok_blocks; };
// S3+S4 / plain GEMM with store epilogue.
struct GemmArgs : GemmTile {
  GemmTile& tile() { return *this; }
  const void* X; int64_t n_tok, c_in, ldx;     // tokens  [n_tok, c_in]
  int64_t x_cand_stride;                        // elements between per-candidate token matrices (0 = shared)
  const float* tok_scale;                       // [n_cand, n_tok] factor on the accumulators or NULL
  const void* Wh; int64_t c_out, ldw;           // operand [n_cand, c_out, c_in]
  int64_t w_cand_stride; int n_cand; bool bf16;
  // loss epilogue
  const void* Yref; int64_t ldy; int yref_dtype; const float* token_w;
  int64_t y_cand_stride;   // launch_gemm_dot: elements between per-candidate Y matrices
  bool tri;                // launch_gemm_store of a symmetric product (X == Wh): tiles with tile row <= tile column only
  bool cand_outer;         // walk the candidates one after the other instead of inside every patch row
  bool wide_patch;         // L2 patches of 8 x 4 tiles (output rows x tokens) instead of 4 x 8
  bool sym_k;              // launch_gemm_dot: Wh is symmetric [c_in, c_in] and Y == X (a quadratic form)
  int64_t o_cand_stride;   // launch_gemm_store with n_cand > 1: elements between per-candidate outputs
  float* partial;          // [n_cand, tiles_o, tiles_t] float
  float* tok_partial;      // [tiles_o, n_tok] float or NULL (single candidate only)
  // integer codes (i8_k = their number per row, 0: floating point): X and Wh hold int8 rows padded with zeros to whole
  // k-tiles of 128 codes, and c_in, ldx, ldw and the strides count 16-bit units; row_scale [n_cand, c_out] are the
  // steps of the weight rows.  Losses without tok_partial, and stores
  int64_t i8_k; const float* row_scale; int64_t row_scale_stride;
  // store epilogue: Y[t,o]; with Yref given Yref - Y (float output and one candidate only, else an error)
  void* Yout; int64_t ldo; int yout_dtype;
};
void gemm_tile_counts(int64_t n_tok, int64_t c_out, GemmTile tile, int64_t* tiles_o, int64_t* tiles_t);
// The tile for a launch of g's sizes, candidates and order.  kinds: tiles besides 256 x 256 that the launch has (stores and
// fp16 losses: all; fp16 losses with tok_partial: not the narrow one; the quadratic form: the wide one); max_tiles: tiles per candidate
// that the caller has room for, at least those of 256 x 256
enum { kTileSmall = 1, kTileNarrow = 2, kTileWide = 4, kTileAll = 7, kTileHalf = 8 };
GemmTile gemm_tile(const GemmArgs& g, int kinds, int64_t max_tiles);
bool gemm_small_triangle(const GemmArgs& g);   // whether a store with tri is faster in tiles of 128 x 128
// row strides that the pipelined kernel (and with it any tile but 256 x 256) takes
bool gemm_strides_ok(int64_t ldx, int64_t ldw);
int64_t gemm_blocks(const GemmArgs& g);   // workgroups of the launch (sizes, tile and order are read, no pointer)
int64_t tile_map_defects(int64_t n_tok, int64_t c_in, int64_t c_out, int n_cand);
hipError_t launch_gemm_loss(const GemmArgs& a, hipStream_t stream);
hipError_t launch_gemm_store(const GemmArgs& a, hipStream_t stream);
// partial[k, tile] = sum over the tile of (X_k Wh^T)[t,o] * Y_k[t,o]  (no token weights), fp16, for a symmetric
// Wh (sym_k): about half the flops, same partial sums
hipError_t launch_gemm_dot(const GemmArgs& a, hipStream_t stream);

// Second-moment form (gram.hip).  out[c, t] = fp16(X[t,c] * sqrt(w_t / max w)) as [c_in, kp] with zero
// columns for n_tok <= t < kp; *wmax receives max_t w_t.
hipError_t launch_gram_operand(const void* X, int64_t n_tok, int64_t c_in, int64_t ldx, bool bf16,
                               const float* token_w, float* wmax, void* out, int64_t kp, hipStream_t stream);
// H: n_split float [c_in, c_in] partial products of that operand with itself (tiles with column
// tile <= row tile), split_stride elements apart; they are summed into the first.  Writes the
// balanced fp16 matrix C, the per-channel factors of the weight errors and the factor that turns
// d'^T C d' into the loss; e is scratch [c_in].
hipError_t launch_gram_finish(float* H, int64_t c_in, int n_split, int64_t split_stride, const float* wmax,
                              int* e, double* factor, float* col_scale, void* C, int side, hipStream_t stream);

hipError_t launch_finalize(const FinalDev& f, hipStream_t stream);
// the same with one candidate and no selection, and err[t] = inv_c_out * the sum of column t of tok_partial [tiles_o, n_tok]
hipError_t launch_layer_err(const FinalDev& f, const float* tok_partial, int64_t tiles_o, int64_t n_tok, float* err, hipStream_t stream);


// chain glue (glue.hip)
hipError_t launch_rmsnorm_mul(const void* Z, int64_t ldz, const void* Zb, int64_t ldzb, int64_t n_tok,
                              int64_t c, bool bf16, const float* m_a, const float* m_b, int period,
                              int split, void* out, int64_t ldo, hipStream_t stream);

// decoder-block glue (block.hip): head width 128, rows in blocks of seq_len
hipError_t launch_causal_attention(const void* Q, int64_t ldq, const void* K, int64_t ldk, const void* V,
                                   int64_t ldv, int64_t n_tok, int n_heads, int seq_len, bool bf16, void* O,
                                   int64_t ldo, hipStream_t stream);
// mode 0: out = SiLU(A) * B; mode 1: out = A + B (c % 8 == 0; out may alias A or B)
hipError_t launch_pairwise(int mode, const void* A, int64_t lda, const void* B, int64_t ldb, int64_t n_tok,
                           int64_t c, bool bf16, void* out, int64_t ldo, hipStream_t stream);

}  // namespace tlq
