// The contraction's square tiles, the general kernel for very wide rows, the choice of a launch's tile and the launches
// (what the kernels share is in contraction.h).
#include <cmath>
#include <cstdlib>

#include "contraction.h"

namespace tlq {

// General kernel: two LDS stages; the global loads of k-tile i+1 are issued before the MFMAs of
// k-tile i and written to the other stage afterwards; one barrier per k-tile.
template <typename T, int BO, int BT, int WO, int WT, int EPI>
__global__ __launch_bounds__((BO / WO) * (BT / WT) * 64) void gemm_kernel(GemmDev a) {
  constexpr int NWO = BO / WO, NWT = BT / WT, NW = NWO * NWT, NT = NW * 64;
  constexpr int FA = WO / 32, FB = WT / 32;
  constexpr int CH_A = BO * 8 / NT, CH_B = BT * 8 / NT;  // 16-byte chunks per thread per k-tile
  static_assert(BO * 8 % NT == 0 && BT * 8 % NT == 0, "tile/thread mismatch");
  constexpr int STAGE = (BO + BT) * ROWB;
  __shared__ __attribute__((aligned(16))) unsigned char lds[2 * STAGE];
  __shared__ float red[NW];

  int cand, to, tt;
  if (!block_tile<EPI>(a, cand, to, tt)) return;
  const int64_t o0 = (int64_t)to * BO, t0 = (int64_t)tt * BT;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wo = wave % NWO, wt = wave / NWO;
  const uint16_t* Wc = a.Wh + (int64_t)cand * a.w_cand_stride;

  // ---- global -> register staging
  const uint16_t* pa[CH_A]; bool oka[CH_A]; int la[CH_A];
  const uint16_t* pb[CH_B]; bool okb[CH_B]; int lb[CH_B];
  const int lchunk = tid & 7;
#pragma unroll
  for (int i = 0; i < CH_A; ++i) {
    const int r = (i * NT + tid) >> 3;
    oka[i] = (o0 + r) < a.c_out;
    pa[i] = Wc + (oka[i] ? (o0 + r) : 0) * a.ldw + lchunk * 8;
    la[i] = r * ROWB + (swz(r, lchunk) << 4);
  }
#pragma unroll
  for (int i = 0; i < CH_B; ++i) {
    const int r = (i * NT + tid) >> 3;
    okb[i] = (t0 + r) < a.n_tok;
    pb[i] = a.X + (int64_t)cand * a.x_cand_stride + (okb[i] ? (t0 + r) : 0) * a.ldx + lchunk * 8;
    lb[i] = BO * ROWB + r * ROWB + (swz(r, lchunk) << 4);
  }
  uint4 ga[CH_A], gb[CH_B];
  auto gload = [&](int64_t k0) {
    const bool kok = (k0 + lchunk * 8) < a.c_in;
#pragma unroll
    for (int i = 0; i < CH_A; ++i) {
      ga[i] = make_uint4(0, 0, 0, 0);
      if (oka[i] && kok) ga[i] = *reinterpret_cast<const uint4*>(pa[i] + k0);
    }
#pragma unroll
    for (int i = 0; i < CH_B; ++i) {
      gb[i] = make_uint4(0, 0, 0, 0);
      if (okb[i] && kok) gb[i] = *reinterpret_cast<const uint4*>(pb[i] + k0);
    }
  };
  auto lstore = [&](int stage) {
    unsigned char* base = lds + stage * STAGE;
#pragma unroll
    for (int i = 0; i < CH_A; ++i) *reinterpret_cast<uint4*>(base + la[i]) = ga[i];
#pragma unroll
    for (int i = 0; i < CH_B; ++i) *reinterpret_cast<uint4*>(base + lb[i]) = gb[i];
  };

  // ---- fragment read offsets: lane -> row (lane%32), k-chunk (lane/32) + 2*kk
  const int frow = lane & 31, fhi = lane >> 5;
  int offk[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) offk[kk] = frow * ROWB + (swz(frow, kk * 2 + fhi) << 4);
  const int a_base = (wo * WO) * ROWB;
  const int b_base = BO * ROWB + (wt * WT) * ROWB;

  f32x16 acc[FA][FB];
#pragma unroll
  for (int i = 0; i < FA; ++i)
#pragma unroll
    for (int j = 0; j < FB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

  const int64_t nk = (a.c_in + BK - 1) / BK;
  gload(0);
  lstore(0);
  __syncthreads();
  for (int64_t kt = 0; kt < nk; ++kt) {
    const int cur = (int)(kt & 1);
    if (kt + 1 < nk) gload((kt + 1) * BK);
    const unsigned char* sb = lds + cur * STAGE;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      uint4 fa[FA], fb[FB];
#pragma unroll
      for (int i = 0; i < FA; ++i)
        fa[i] = *reinterpret_cast<const uint4*>(sb + a_base + i * 32 * ROWB + offk[kk]);
#pragma unroll
      for (int j = 0; j < FB; ++j)
        fb[j] = *reinterpret_cast<const uint4*>(sb + b_base + j * 32 * ROWB + offk[kk]);
#pragma unroll
      for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int j = 0; j < FB; ++j) acc[i][j] = Mma<T>::run(fa[i], fb[j], acc[i][j]);
    }
    if (kt + 1 < nk) lstore(cur ^ 1);
    __syncthreads();
  }

  // the tile memory is free now: row sums of the per-token variant reuse it
  tile_epilogue<EPI, Acc32<FA, FB>, NWO, NWT, BT, false>(a, acc, cand, to, tt, o0, t0, wo, wt, red,
                                                         reinterpret_cast<float*>(lds));
}

template <typename T, int NSTAGE, int EPI, bool SYMK, bool TAIL, int HALVES>
__global__ __launch_bounds__(HALVES * 256) void gemm_dma_kernel(GemmDev a) {
  gemm_dma_body<T, NSTAGE, EPI, SYMK, TAIL, HALVES, 4>(a);
}

// ---- host side ---------------------------------------------------------------
constexpr int kBO = 256, kBT = 256, kWO = 128, kWT = 64;   // (the general kernel has this tile only)
constexpr int kSmall = 128;                  // rows and columns of a small tile
constexpr int64_t kChunkBytes = (int64_t)128 << 20;
// Up to this many tiles (of 256 tokens, or small ones) a launch is dealt in strips (us, patches -> strips: 480 tiles 252 -> 224, 640 318 ->
// 308, 960 428 -> 401; 1080 664 -> 667, 1720 762 -> 815: there a strip no longer fits an L2).
constexpr int64_t kStripTiles = 1024;

static int64_t tile_tokens(GemmTile t) { return (t.small ? 32 : 64) * (t.tok_blocks ? t.tok_blocks : 4); }
void gemm_tile_counts(int64_t n_tok, int64_t c_out, GemmTile tile, int64_t* tiles_o, int64_t* tiles_t) {
  *tiles_o = ceil_div(c_out, tile.small ? kSmall : kBO);
  *tiles_t = ceil_div(n_tok, tile_tokens(tile));
}

// Of the square tiles, whether the small one is faster.  Two small blocks share a CU: up to 512 of them
// are one round, where big tiles leave CUs idle (store epilogue, us big -> small: 640 x 4096 x 4096
// tokens x channels x outputs 93 -> 49, 1200 x 5120 x 5120 122 -> 82, 1800 x 4096 x 4096 100 -> 71; from 640
// small tiles on the big ones win, 98 against 113).  Just past one round of big tiles the second
// round is nearly empty and the small ones win again (1200 x 5120 x 13824, 270 big tiles: 243 -> 213; 320: 201
// -> 188; 384: 206 -> 211).
static bool gemm_small_tiles(int64_t n_tok, int64_t c_out, int n_cand) {
  const int64_t big = ceil_div(c_out, kBO) * ceil_div(n_tok, kBT) * n_cand;
  const int64_t small = ceil_div(c_out, kSmall) * ceil_div(n_tok, kSmall) * n_cand;
  return small <= 512 || (big > 256 && small <= 1280);
}

static GemmDev make_dev(const GemmArgs& g) {
  GemmDev d;
  d.X = (const uint16_t*)g.X; d.n_tok = g.n_tok; d.c_in = g.c_in; d.ldx = g.ldx;
  d.x_cand_stride = g.x_cand_stride; d.tok_scale = g.tok_scale;
  d.Wh = (const uint16_t*)g.Wh; d.c_out = g.c_out; d.ldw = g.ldw;
  d.w_cand_stride = g.w_cand_stride; d.n_cand = g.n_cand;
  d.Yref = g.Yref; d.ldy = g.ldy; d.ydt = g.yref_dtype; d.token_w = g.token_w;
  d.y_cand_stride = g.y_cand_stride; d.tri = g.tri ? 1 : 0;
  d.cand_outer = g.cand_outer ? 1 : 0; d.o_cand_stride = g.o_cand_stride;
  d.partial = g.partial; d.tok_partial = g.tok_partial;
  d.Yout = g.Yout; d.ldo = g.ldo; d.odt = g.yout_dtype;
  d.row_scale = g.row_scale; d.row_scale_stride = g.row_scale_stride;
  int64_t to, tt;
  gemm_tile_counts(g.n_tok, g.c_out, g, &to, &tt);
  d.tiles_o = (int)to; d.tiles_t = (int)tt;
  d.po = g.wide_patch ? 8 : 4; d.pt = PATCH_SLOTS / d.po;
  // few token tiles: one patch across all of them (5 tiles in patches of 4 would alternate full and nearly
  // empty patches over the XCDs: 20 candidates of 1200 x 5120 x 5120 1578 -> 1110 us)
  if (tt < 8 && tt % d.pt && !g.sym_k) { d.pt = (int)tt; d.po = PATCH_SLOTS / d.pt; }
  const int PATCH_O = d.po, PATCH_T = d.pt;
  d.npo = (int)ceil_div(to, PATCH_O); d.npt = (int)ceil_div(tt, PATCH_T);
  d.rag = (int)(to % PATCH_O);
  d.rag_pt = d.rag == 0 ? PATCH_T : PATCH_SLOTS / d.rag;   // e.g. 3 rows -> patches of 3 x 10
  // Tokens of one chunk.  While all tokens fit in half of the 256 MB last-level cache there is one
  // chunk.  Otherwise a chunk holds the largest power-of-two number of token patches within that
  // budget: with 1, 2, 4 or 8 patches per (candidate, patch row) the round-robin deal keeps every XCD
  // on the same token patch from one candidate to the next, which measured steadier (and on most
  // boxes faster) on 153,600-token inputs than 3, 5 or 6 patches, whose speed flips between
  // launches by up to 8 %.
  const int64_t patch_bytes = (int64_t)PATCH_T * tile_tokens(g) * g.c_in * 2;
  if ((int64_t)d.npt * patch_bytes <= kChunkBytes) {
    d.cpt = d.npt;
  } else {
    d.cpt = 1;
    while (d.cpt * 2 <= kXcd && (int64_t)d.cpt * 2 * patch_bytes <= kChunkBytes) d.cpt *= 2;
  }
  const int64_t tiles = to * tt * g.n_cand;
  // (tiles of a symmetric contraction differ in work along the rows: strips would not be equal)
  d.strips = (g.small ? tiles : tiles * tile_tokens(g) / kBT) <= kStripTiles && !g.tri && !g.sym_k ? tiles : 0;
  if (g.tri) {
    d.n_patches = ceil_div(ceil_div(to * (to + 1) / 2, kXcd) * g.n_cand, PATCH_SLOTS) * kXcd;
  } else if (d.strips) {
    // one strip per XCD, rounded up to whole blocks of eight
    d.n_patches = ceil_div(ceil_div(tiles, kXcd), PATCH_SLOTS) * kXcd;
  } else {
    const int n_full = d.rag ? d.npo - 1 : d.npo;
    const int64_t full_chunks = d.npt / d.cpt;
    const int cw_last = d.npt % d.cpt;
    auto per_cand = [&](int cw) {
      return (int64_t)n_full * cw + (d.rag ? (cw * PATCH_T + d.rag_pt - 1) / d.rag_pt : 0);
    };
    d.n_patches = (int64_t)g.n_cand * (full_chunks * per_cand(d.cpt) + (cw_last ? per_cand(cw_last) : 0));
  }
  // Where a candidate has a multiple of eight patches and candidates are walked one after the other, every XCD
  // meets the same patches each time, and they differ in work: the upper rows of a symmetric contraction
  // are the long ones, the last token patch may be ragged.  Turned by five XCDs a round they
  // alternate (quadratic form, 16 x 16 tiles, 20 candidates: 1.77 -> 1.40 ms; 16 x 15 tiles with per-candidate
  // tokens: 2.34 -> 2.29 ms a search).  Where the count is no multiple the turn only costs shared panels (quadratic form,
  // 43 x 16 tiles: 8.4 -> 9.4 ms).
  d.rot = g.cand_outer && !g.tri && (d.n_patches / g.n_cand) % kXcd == 0 ? 5 : 0;
  return d;
}

// Rounds of 256 tiles that a launch takes.  An XCD works on its own patches only, and where every candidate (or every
// second one) has as many patches as there are XCDs, the short patches at the end of the tokens always meet the same
// ones: 13 token tiles in patches of four leave two XCDs a quarter of the work of the others.  An idle XCD leaves
// power to the busy ones, so that the time lies halfway between the average and the busiest XCD's work (4096 x 4096 x
// 4096 x 20 with 320-token tiles: 16.25 and 20 rounds, and the time of 18).
static double launch_rounds(const GemmDev& d, bool sym) {
  const int64_t tiles = (int64_t)d.tiles_o * d.tiles_t * d.n_cand;
  if (d.strips) return (double)tiles / (kXcd * PATCH_SLOTS);
  // (in a symmetric contraction the tile row r contracts tiles_o - r of the tiles_o blocks along k)
  auto rows = [&](int first, int n) { return sym ? (int64_t)n * (d.tiles_o - first) - (int64_t)n * (n - 1) / 2 : n; };
  int64_t load[kXcd] = {}, p = 0;
  auto deal = [&](int64_t live) {
    const int64_t round = p / kXcd;
    load[(p - d.rot * (round & (kXcd - 1))) & (kXcd - 1)] += live;
    ++p;
  };
  const int n_full = d.rag ? d.npo - 1 : d.npo, inner = d.cand_outer ? 1 : d.n_cand;
  for (int k = 0; k < (d.cand_outer ? d.n_cand : 1); ++k)      // (the walk of decode_tile, patch by patch)
    for (int64_t t0 = 0; t0 < d.tiles_t; t0 += (int64_t)d.cpt * d.pt) {
      const int64_t chunk = (int64_t)d.cpt * d.pt, end = t0 + chunk < d.tiles_t ? t0 + chunk : d.tiles_t;
      auto row_of_patches = [&](int64_t high, int wide) {
        for (int c = 0; c < inner; ++c)
          for (int64_t t = t0; t < end; t += wide) deal(high * (end - t < wide ? end - t : wide));
      };
      for (int r = 0; r < n_full; ++r) row_of_patches(rows(r * d.po, d.po), d.pt);
      if (d.rag) row_of_patches(rows(n_full * d.po, d.rag), d.rag_pt);
    }
  double most = 0.0, sum = 0.0;
  for (int64_t l : load) { sum += (double)l; most = (double)l > most ? (double)l : most; }
  return 0.5 * (most / PATCH_SLOTS + sum / (kXcd * PATCH_SLOTS)) / (sym ? 0.5 * (d.tiles_o + 1) : 1.0);
}

// The tile that takes the least time (any result is the same up to the order of the loss sums: an output's own
// products are added in the same order).  A launch of up to eight rounds takes whole rounds of one block per
// CU (small tiles: two), longer ones drift apart and pay for their tiles.  The cost of a round, in rounds of 256 x 256,
// from store launches of one round with 4096 channels (us): 128 x 128 59, 192 tokens 79, 256 97, 320 114.  Over several
// rounds the narrow one comes to 0.80 - 0.91; two rounds of small ones cost what one of wide ones does (1300 x 1024 x
// 11904 35 and 36 us, 1300 x 4096 x 11904 117 and 114), three a little more than two of narrow ones.  The wide tile
// reads fewer fragments and fetches fewer panels per product, so it is ahead of the square one also where the
// count of rounds does not decide, unless its last token tile is short or its patches meet the XCDs unevenly.
// us by tile (128, 192, 256, 320), tokens x channels x outputs [x candidates]:
//   store   1200 x 5120 x 13824 207 185 214 140      search  10,240 x 4096 x 4096 x 20  6241 5797 5213 5031
//   store   2500 x 4096 x 4096   99  74  88 101      search  40,000 x 5120 x 5120 x 20   41.1  37.9  33.1  30.7 ms
//   store   3678 x 4096 x 4096  111 137  96 110      search     640 x 4096 x 4096 x 20   690  632  594  550
//   store   4800 x 4096 x 4096  151 146 171 114      search  W4A8 3678 x 4096 x 4096    1499 1370 1277 1218
//   store  10,240 x 11008 x 4096 833 959 805 642     search    1839 x 1152 x 1400 x 12   129  125  133  128
//   store  40,960 x 4096 x 11008  3.28 2.94 2.77 2.61 ms   quadratic form 5120 x 5120 - - 2824 2654; 4096 x 1024 - - 448 523
//   store  6144 x 5120 x 13824    -  850 702 686     search    4096 x 4096 x 4096 x 20     -  2588 2370 2591
//   quadratic form 5120 x 4096 - - 2327 2586         search    8192 x 4096 x 1024 x 20     -  1237 1119 1255
// Over 228 launches of three rounds and more the choice costs 0.2 % against the best of the three (1.0 % with
// the plain count of tiles, whose worst cases were 21 % and 12 %).
// The tiles of a symmetric contraction differ in length and fill each other's rounds: beyond two tiles a CU they are not
// rounded up (4416 x 1057 and 2624 x 1061, channels x rows, 7 and 11 candidates, us 256 and 320: 215 and 178, 139 and 188);
// up to there the plain count is the better guess (768 x 2840 x 7 45 and 58, 1408 x 528 x 20 58 and 51).  Over 220 quadratic
// forms of 0.4 to 20 rounds the choice costs 2.5 % against the better of the two, 4.9 % by the plain count throughout
// and 2.7 % with the XCDs' shares rounded up, 12 to 28 % behind the plain count in eight of those below two rounds.
GemmTile gemm_tile(const GemmArgs& args, int kinds, int64_t max_tiles) {
  GemmArgs g = args;
  GemmTile best{false, 4};
  double best_cost = 1e300;
  int64_t to, tt;
  gemm_tile_counts(g.n_tok, g.c_out, best, &to, &tt);
  const bool few = to * tt * g.n_cand <= 512;
  // at most one tile of 128 x 64 a CU (gemm_half.hip)
  gemm_tile_counts(g.n_tok, g.c_out, GemmTile{true, 2}, &to, &tt);
  if ((kinds & kTileHalf) && to * tt * g.n_cand <= 256 && to * tt <= max_tiles) return GemmTile{true, 2};
  auto consider = [&](GemmTile t, double first, double each) {
    gemm_tile_counts(g.n_tok, g.c_out, t, &to, &tt);
    if (to * tt > max_tiles) return;
    g.tile() = t;
    const double even = (double)(to * tt) * g.n_cand / (t.small ? 512 : 256);
    const double rounds = t.small || (g.sym_k && few) ? even : launch_rounds(make_dev(g), g.sym_k);
    const double whole = rounds <= 8.0 ? std::ceil(rounds - 1e-9) : rounds + 0.5;
    const double cost = first + each * (g.sym_k && !few ? rounds : whole);
    if (cost < best_cost) { best = t; best_cost = cost; }
  };
  if ((kinds & kTileSmall) && gemm_small_tiles(g.n_tok, g.c_out, g.n_cand)) consider(GemmTile{true, 0}, 0.06, 0.56);
  if (best_cost == 1e300) consider(GemmTile{false, 4}, 0.0, 1.0);
  if (kinds & kTileNarrow) consider(GemmTile{false, 3}, 0.0, 0.86);
  if (kinds & kTileWide) consider(GemmTile{false, 5}, 0.0, 1.19);
  return best;
}

static int64_t dev_blocks(const GemmDev& d) { return ceil_div(d.n_patches, kXcd) * kXcd * PATCH_SLOTS; }
int64_t gemm_blocks(const GemmArgs& g) { return dev_blocks(make_dev(g)); }

// the pipelined kernel needs 32-bit byte offsets inside a 256-row panel
bool gemm_strides_ok(int64_t ldx, int64_t ldw) { return ldw < (1 << 21) && ldx < (1 << 21); }
static bool pipelined_ok(const GemmArgs& g) { return gemm_strides_ok(g.ldx, g.ldw); }

// Up to two small tiles a CU, as in gemm_small_tiles: few channels have few big tiles, with a long contraction each (the whole
// token product, us big -> small, tokens x channels: 600 x 256 38 -> 27, 10,640 x 896 135 -> 71, 64,699 x 640 151 -> 120, 465
// tiles of 4096 x 3840 137 -> 112; beyond, 528 tiles of 4200 x 4096 146 -> 156, 780 of 44,166 x 1536 197 -> 220).
bool gemm_small_triangle(const GemmArgs& g) {
  const int64_t side = ceil_div(g.c_out, kSmall);
  return pipelined_ok(g) && side * (side + 1) / 2 * g.n_cand <= 512;
}

// Only the instances that some launch reaches are compiled: the loading of the code object is part of a
// program's first call.  The searches' operands are fp16 in every form, so bf16 operands meet the loss only
// in the single-candidate call, which keeps the big tiles; the quadratic
// form is fp16, big and symmetric.
template <typename T, int EPI>
static hipError_t launch_dma(const GemmDev& d, GemmTile tile, unsigned blocks, hipStream_t stream) {
  constexpr bool SYMK = EPI == EPI_DOT;
  constexpr bool SMALL = EPI == EPI_STORE || (EPI == EPI_LOSS && std::is_same<T, F16>::value);
  const bool tail = (d.c_in % kDmaBK) != 0;
  if (!tile.small) {
    if (tile.tok_blocks == 3 || tile.tok_blocks == 5)
      return launch_dma_width(d, EPI, std::is_same<T, BF16>::value, tile.tok_blocks, blocks, stream);
    if (!tail) gemm_dma_kernel<T, 2, EPI, SYMK, false, 2><<<blocks, 512, 0, stream>>>(d);
    else gemm_dma_kernel<T, 2, EPI, SYMK, true, 2><<<blocks, 512, 0, stream>>>(d);
    return hipGetLastError();
  }
  if (tile.tok_blocks == 2) return launch_dma_half(d, EPI, std::is_same<T, BF16>::value, blocks, stream);
  // one block per CU at most: four LDS stages hide the latency that a second block would
  const bool deep = (int64_t)d.tiles_o * d.tiles_t * d.n_cand <= 256;
  // (a caller has to say that its token sums have rows for these tiles)
  if constexpr (EPI == EPI_LOSS_TOK && std::is_same<T, F16>::value)
    return tile.tok_blocks != 4 ? hipErrorInvalidValue : launch_dma_small_tok(d, deep, blocks, stream);
  if constexpr (SMALL) {
    if (!tail && deep) gemm_dma_kernel<T, 4, EPI, SYMK, false, 1><<<blocks, 256, 0, stream>>>(d);
    else if (!tail) gemm_dma_kernel<T, 2, EPI, SYMK, false, 1><<<blocks, 256, 0, stream>>>(d);
    else if (deep) gemm_dma_kernel<T, 4, EPI, SYMK, true, 1><<<blocks, 256, 0, stream>>>(d);
    else gemm_dma_kernel<T, 2, EPI, SYMK, true, 1><<<blocks, 256, 0, stream>>>(d);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <typename T, int EPI>
static hipError_t launch_gemm(const GemmArgs& g, const char* name, hipStream_t stream) {
  const bool dma = pipelined_ok(g);
  constexpr bool kHasInt = std::is_same<T, F16>::value && (EPI == EPI_LOSS || EPI == EPI_STORE);
  if (g.i8_k && (!kHasInt || !dma || !g.row_scale || (g.c_in % kDmaBK) != 0)) return hipErrorInvalidValue;
  if (g.small && g.tok_blocks != 0 && g.tok_blocks != 4 && (g.tok_blocks != 2 || g.i8_k || g.tri)) return hipErrorInvalidValue;
  if (!dma && (g.small || (g.tok_blocks && g.tok_blocks != 4))) return hipErrorInvalidValue;   // (the callers ask gemm_strides_ok first)
  const GemmDev d = make_dev(g);
  const int64_t blocks = dev_blocks(d);
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  // (a symmetric product computes the tiles on and above the diagonal, a symmetric contraction
  // the k range from the diagonal block on: about half either way)
  const double tile_frac = (g.tri || EPI == EPI_DOT) ? 0.5 * (1.0 + 1.0 / (double)d.tiles_o) : 1.0;
  const double k = (double)(g.i8_k ? g.i8_k : g.c_in);
  ProfScope ps(name, stream, 2.0 * (double)g.n_tok * k * (double)g.c_out * g.n_cand * tile_frac);
  if constexpr (kHasInt) {
    if (g.i8_k) return launch_dma_i8(d, EPI, g, (unsigned)blocks, stream);
  }
  if (dma) return launch_dma<T, EPI>(d, g, (unsigned)blocks, stream);
  if constexpr (EPI != EPI_DOT) {
    constexpr int NT = (kBO / kWO) * (kBT / kWT) * 64;
    gemm_kernel<T, kBO, kBT, kWO, kWT, EPI><<<(unsigned)blocks, NT, 0, stream>>>(d);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

// Host-side check of the block -> tile map for one problem shape: both block orders (candidates inside every
// patch row, and candidate-outermost, which may turn the XCDs), both patch shapes and all tile sizes, the
// quadratic form's map, and those of the symmetric products over c_out and c_in.  Each walk takes every block
// id of its launch and counts how often each (candidate, tile) is produced; a walk whose tiles are not
// of the size it is there for counts as a defect too.  Returns the number of tiles that are not produced
// exactly once (0 = all maps are bijections onto the tiles), or -1 if memory runs out.
int64_t tile_map_defects(int64_t n_tok, int64_t c_in, int64_t c_out, int n_cand) {
  int64_t bad = 0;
  // walks 0 - 19: bit 0 the order, bit 1 the patch shape, the others the tile
  const GemmTile tiles_of[5] = {{false, 0}, {true, 0}, {false, 3}, {false, 5}, {true, 2}};
  const int side_of[5] = {256, 128, 192, 320, 64};
  enum { kQuadratic = 20, kTriOut, kTriIn, kSmallTriOut, kSmallTriIn, kWalks };
  for (int walk = 0; walk < kWalks; ++walk) {
    GemmArgs g{};
    g.n_tok = n_tok; g.c_in = c_in; g.c_out = c_out; g.n_cand = n_cand;
    if (walk < kQuadratic) {
      g.cand_outer = (walk & 1) != 0;
      g.wide_patch = (walk & 2) != 0;
      g.tile() = tiles_of[walk >> 2];
    } else if (walk == kQuadratic) {
      g.cand_outer = g.wide_patch = g.sym_k = true;
    } else {
      g.tri = true;
      g.small = walk >= kSmallTriOut;
      g.n_tok = g.c_out = walk == kTriOut || walk == kSmallTriOut ? c_out : c_in;
    }
    const GemmDev d = make_dev(g);
    const int64_t side_o = g.small ? 128 : 256, side_t = walk < kQuadratic ? side_of[walk >> 2] : side_o;
    if (d.tiles_o != (g.c_out + side_o - 1) / side_o || d.tiles_t != (g.n_tok + side_t - 1) / side_t) ++bad;
    const int64_t blocks = dev_blocks(d);
    const int64_t tiles = (int64_t)n_cand * d.tiles_o * d.tiles_t;
    unsigned char* seen = (unsigned char*)calloc((size_t)tiles, 1);
    if (!seen) return -1;
    for (int64_t b = 0; b < blocks; ++b) {
      int cand, to, tt;
      if (!(g.tri ? decode_tri(d, b, cand, to, tt) : decode_tile(d, b, cand, to, tt))) continue;
      if (cand < 0 || cand >= n_cand || to < 0 || tt < 0) { ++bad; continue; }
      unsigned char& c = seen[((int64_t)cand * d.tiles_o + to) * d.tiles_t + tt];
      if (c < 255) ++c;
    }
    for (int64_t i = 0; i < tiles; ++i) {
      const int64_t row = i / d.tiles_t % d.tiles_o, col = i % d.tiles_t;
      bad += seen[i] != (g.tri && row > col ? 0 : 1);
    }
    free(seen);
  }
  return bad;
}

hipError_t launch_gemm_loss(const GemmArgs& g, hipStream_t stream) {
  if (g.tok_partial)
    return g.bf16 ? launch_gemm<BF16, EPI_LOSS_TOK>(g, "gemm_loss_tok", stream)
                  : launch_gemm<F16, EPI_LOSS_TOK>(g, "gemm_loss_tok", stream);
  return g.bf16 ? launch_gemm<BF16, EPI_LOSS>(g, "gemm_loss", stream) : launch_gemm<F16, EPI_LOSS>(g, "gemm_loss", stream);
}
hipError_t launch_gemm_store(const GemmArgs& g, hipStream_t stream) {
  if (g.tri && g.n_tok != g.c_out) return hipErrorInvalidValue;
  if (g.n_cand != 1 && g.o_cand_stride == 0) return hipErrorInvalidValue;
  // the 16-bit store through LDS does not subtract, and Yref has no stride per candidate
  if (g.Yref && (g.yout_dtype != TLQ_F32 || g.n_cand != 1)) return hipErrorInvalidValue;
  const char* name = g.tri ? "gemm_gram" : "gemm_store";
  return g.bf16 ? launch_gemm<BF16, EPI_STORE>(g, name, stream) : launch_gemm<F16, EPI_STORE>(g, name, stream);
}
hipError_t launch_gemm_dot(const GemmArgs& g, hipStream_t stream) {
  // (row strides of 2^21 and more would mean a matrix of 8 TB)
  if (g.bf16 || g.small || !g.sym_k || g.c_out != g.c_in || !pipelined_ok(g)) return hipErrorInvalidValue;
  return launch_gemm<F16, EPI_DOT>(g, "gemm_gram_loss", stream);
}

}  // namespace tlq
