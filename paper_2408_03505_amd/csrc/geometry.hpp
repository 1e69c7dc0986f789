// Host-side launch geometry that fixes workspace sizes: shared by the kernel
// launchers and the C-ABI size queries (plain C++, no device code).
#pragma once

#include <stddef.h>

#include <algorithm>

namespace optimus {

// ---- LayerNorm backward: 256-thread blocks, up to kLnBwdBlocks of them, each
// writing one row of fp32 column partials per gradient (dgamma, dbeta).
constexpr int kLnThreads = 256;
constexpr int kLnBwdBlocks = 256;

// Threads per row: one wave up to 2048 columns (four rows in flight per
// block), the whole block beyond.
inline int ln_bwd_tpr(int cols) { return (cols >> 3) > 256 ? 256 : 64; }

// Rows per block (a multiple of the rows in flight).
inline int ln_bwd_rows_per_block(int rows, int cols) {
  const int rg = kLnThreads / ln_bwd_tpr(cols);
  int rpb = (rows + kLnBwdBlocks - 1) / kLnBwdBlocks;
  rpb = (rpb + rg - 1) / rg * rg;
  return rpb < rg ? rg : rpb;
}

inline int ln_bwd_blocks(int rows, int cols) {
  const int rpb = ln_bwd_rows_per_block(rows, cols);
  return (rows + rpb - 1) / rpb;
}

inline size_t ln_bwd_ws_bytes(int rows, int cols) {
  return static_cast<size_t>(ln_bwd_blocks(rows, cols)) * static_cast<size_t>(cols) * 2 * sizeof(float);
}

// ---- QK-norm backward: 16-lane groups, 16 per 256-thread block, at most
// 1024 blocks, each writing 4 x head_dim fp32 partials.
constexpr int kQkGroups = 16;

inline int qk_norm_bwd_blocks(int M, int heads) {
  const long pairs = static_cast<long>(M) * heads;
  const long want = (pairs + kQkGroups - 1) / kQkGroups;
  return static_cast<int>(want < 1024 ? want : 1024);
}

inline size_t qk_norm_bwd_ws_bytes(int M, int heads, int d) {
  return static_cast<size_t>(qk_norm_bwd_blocks(M, heads)) * 4 * d * sizeof(float);
}

// ---- Attention backward: the D vector, one fp32 per (sequence, head, query).
inline size_t attn_bwd_ws_bytes(int B, int S, int heads) {
  return static_cast<size_t>(B) * heads * S * sizeof(float);
}

// ---- GEMM tile choice.  The direct-to-LDS kernels come in these output
// tiles; per_cu workgroups of a tile share a CU.  cost[kind] is the time in us
// of one workgroup per 64-wide k-step and on top of them (prologue, epilogue):
// {step, rest} alone on its CU and, where two share a CU, {step, rest} of such
// a pair, which is never less; {} where a tile is not offered.
//
// Fitted to 5850 unsplit products (50 to 8224 rows, widths 192 to 24576), every
// tile timed on each, with the operands in the 256 MB cache and with weights
// and outputs rotated past it, weighted towards the tiles near each product's
// best one: it is the picks that count.  Predicted times are 9-11% off on
// average over all tiles.  The picks take 0.1-0.2% longer in total than each
// product's best tile (weight gradients 0.5%).  Against the tiles that area and
// rounds chose on the kernels before these they take 31 to 45% less, and no
// forward or input-gradient pick is more than 1.1% slower (weight gradients: 8
// of 1650 by more than 3%, at most 6.3%).  Small tiles pay more per flop (each
// loads (bm + bn) / (bm * bn) operand bytes per flop into LDS, and a short
// k-step is bound by its barrier and LDS latency) but fill the 256 CUs.
//
// Products with a GELU or GELU' epilogue have the same steps and a longer rest:
// alone, the epilogue of a 256x256 tile takes 17 and 20 us there against 9 and
// 6.  The forward GELU is not offered 192x128 tiles: timed by themselves they
// are its best choice at times (1028 x 16384, K = 4096: 131 us against 151 on
// 256x192), but in a layer, with the weights from HBM, they took 178 against 164.
enum GemmLayout { kFwd = 0, kDgrad = 1, kWgrad = 2, kFwdGelu = 3, kDgradGelu = 4, kSplit = 5, kWgradSplit = 6 };

// Row of the cost table of an unsplit product with operands A, B (AT, BT:
// stored k-major) and, with `gelu`, a GELU or GELU' epilogue.
constexpr GemmLayout gemm_layout(bool AT, bool BT, bool gelu) {
  return AT ? kWgrad : BT ? (gelu ? kDgradGelu : kDgrad) : (gelu ? kFwdGelu : kFwd);
}

struct TileShape {
  int bm, bn;
};

struct TileCost {
  int bm, bn, per_cu;
  float cost[7][4];  // [GemmLayout]: step, rest, step of a pair, rest of a pair
};

constexpr TileCost kTiles[] = {
    {256, 256, 1, {{1.20, 9.39}, {1.26, 6.30}, {1.38, 12.56}, {1.20, 16.96}, {1.26, 20.43}, {}, {1.11, 8.96}}},
    {256, 192, 1, {{1.03, 9.40}, {1.06, 5.94}, {1.19, 7.90}, {1.03, 13.74}, {1.06, 13.64}, {}, {0.93, 8.59}}},
    {128, 256, 1, {{0.72, 5.89}, {0.75, 4.48}, {0.76, 6.64}, {0.72, 8.84}, {0.75, 10.19}, {}, {0.60, 6.00}}},
    {128, 192, 1, {{0.59, 5.51}, {0.61, 4.11}, {0.61, 5.05}, {0.59, 6.53}, {0.61, 7.78}, {}, {0.49, 5.42}}},
    {192, 128, 2, {{0.75, 5.08, 1.14, 8.27}, {0.70, 3.66, 1.16, 4.36}, {0.78, 4.79, 1.21, 7.49}, {}, {0.70, 7.24, 1.16, 10.45}, {}, {0.68, 4.73, 1.10, 4.80}}},
    {128, 128, 2, {{0.63, 4.05, 0.85, 6.47}, {0.63, 3.08, 0.82, 3.45}, {0.64, 4.25, 0.88, 4.71}, {0.63, 5.04, 0.85, 6.76}, {0.63, 5.47, 0.82, 7.93}, {0.59, 3.34, 0.78, 4.53}, {0.53, 3.43, 0.77, 3.43}}},
    {64, 192, 1, {{0.46, 4.79}, {0.40, 3.55}, {0.42, 4.30}, {0.46, 5.42}, {0.40, 5.45}, {0.32, 3.46}, {}}},
    {64, 128, 2, {{0.30, 3.78, 0.62, 3.96}, {0.29, 3.23, 0.55, 3.23}, {0.30, 3.55, 0.53, 3.78}, {0.30, 4.09, 0.62, 4.62}, {0.29, 4.51, 0.55, 4.55}, {0.26, 3.42, 0.51, 3.46}, {}}},
    {64, 64, 2, {{0.20, 3.46, 0.33, 3.56}, {0.20, 3.14, 0.35, 3.14}, {0.27, 3.08, 0.36, 3.11}, {0.20, 3.66, 0.33, 3.70}, {0.20, 3.79, 0.35, 3.79}, {0.17, 3.27, 0.31, 3.27}, {}}}};

// Whether the table offers a tile to the products of a row.
constexpr bool tile_offered(int bm, int bn, GemmLayout l) {
  for (const TileCost &t : kTiles)
    if (t.bm == bm && t.bn == bn) return t.cost[l][0] != 0.f;
  return false;
}

// Every split tile of a weight gradient is one of its unsplit tiles too: the
// same kernels run both.
constexpr bool split_tiles_run_unsplit() {
  for (const TileCost &t : kTiles)
    if (t.cost[kWgradSplit][0] != 0.f && t.cost[kWgrad][0] == 0.f) return false;
  return true;
}
static_assert(split_tiles_run_unsplit(), "weight-gradient tiles");

// Predicted time (us) of `wgs` workgroups of a tile with nk k-steps each, in
// rounds of per_cu workgroups on every CU.
inline float gemm_cost(const TileCost &t, GemmLayout l, long wgs, int nk) {
  const float *c = t.cost[l];
  if (t.per_cu == 1) return static_cast<float>((wgs + 255) / 256) * (nk * c[0] + c[1]);
  const long full = wgs / 512, rem = wgs - full * 512;
  const float one = nk * c[0] + c[1], two = nk * c[2] + c[3];
  return static_cast<float>(full) * two + (rem == 0 ? 0.f : rem > 256 ? two : one);
}

inline long tile_count(const TileCost &t, int M, int N) {
  return static_cast<long>((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
}

struct TilePick {
  TileShape tile;
  float us;
};

// Whether a tile may run an output [M, N].  The 256-row kernels load a tile in
// halves, the second one up to 64 rows (columns) of the operand further by a
// scalar offset.  The buffer's range check takes that offset off the operand's
// size, so it must not be larger: more than 64 rows and columns.  (No product
// of that kind is fastest on a 256-row tile.)
inline bool tile_allowed(const TileCost &t, int M, int N) { return t.bm < 256 || (M > 64 && N > 64); }

inline TilePick pick_tile(int M, int N, int K, GemmLayout l) {
  TilePick best{{0, 0}, 0.f};
  for (const TileCost &t : kTiles) {
    // weight gradients over a few k-steps are their fp32 stores: 64-row tiles
    // (whose loop is cheap, not their epilogue) only beyond five of them, and
    // tiles alone on their CU only beyond ten, as two to a CU overlap one's
    // stores with the other's loop over several rounds (306 tokens, 4480 x
    // 23488: 109 us on 128x128 tiles, 129 on 256x256, 122 before these kernels)
    if (l == kWgrad && ((t.bm < 128 && K <= 5 * 64) || (t.per_cu == 1 && K <= 10 * 64))) continue;
    if (t.cost[l][0] == 0.f || !tile_allowed(t, M, N)) continue;
    const float us = gemm_cost(t, l, tile_count(t, M, N), (K + 63) / 64);
    if (best.tile.bm == 0 || us < best.us) best = {{t.bm, t.bn}, us};
  }
  return best;
}

inline TileShape choose_tile(int M, int N, int K, GemmLayout l) { return pick_tile(M, N, K, l).tile; }

// ---- Split of the contraction (the tokens, for a weight gradient), for
// products whose output is small: each split writes fp32 partials and a second
// kernel adds them in split order (deterministic).  Weight gradients of at
// most 64 tiles of 256x256, and forward and input-gradient products of at most
// 32, split when their contraction holds two splits of kMinSplitTokens; which
// products split is part of what callers size their workspaces by, and is not
// weighed against the unsplit product.  Tile and number of splits minimise the
// cost model's time plus the traffic of the second kernel (at 4.5 TB/s; its
// launch is the same for all).  The splits' rows of the cost table are fitted
// to 1620 products, every tile and split timed, forward and input gradients in
// one row as they share a plan: predicted times are 9% off on average (weight
// gradients 6%), and the picks are no slower than 128x128 splits were on the
// kernels before these (1080 forward and input-gradient products: two by more
// than 3%, at most 15%; 540 weight gradients: at most 2%).  Splits are whole 64-wide k-steps of equal length,
// rounded up, of kMinSplitTokens on average or more: the last takes what
// remains, which can be little.  Tiles below 128x128 are worth it only for
// forward and input-gradient products, where they fill the CUs.
constexpr int kMinSplitTokens = 512, kMaxSplits = 16;

struct SplitPlan {
  int splits, k_chunk;
  TileShape tile;
};

// Longest split of a weight gradient (tokens): that of a grid of 128x128
// workgroups, two to a CU.  dW is returned in fp32, and the error of a sum
// against 64 bits grows with its length: 1.3e-7 (2-norm, relative) in splits of
// 512 tokens, 1.9e-7 of 1024, 2.7e-7 of 2048.  The cost model alone would save
// the partials' traffic by summing twice as long.
inline int wgrad_max_chunk(int M, int N, int K) {
  const long tiles = static_cast<long>((M + 127) / 128) * ((N + 127) / 128);
  const int s = static_cast<int>(std::min<long>(512 / tiles, std::min(K / kMinSplitTokens, kMaxSplits)));
  return ((K + s - 1) / s + 63) / 64 * 64;
}

inline SplitPlan best_split(int M, int N, int K, GemmLayout l) {
  SplitPlan best{1, K, {0, 0}};
  float best_us = 0.f;
  const int max_s = std::min(K / kMinSplitTokens, kMaxSplits);
  const int max_chunk = l == kWgrad ? wgrad_max_chunk(M, N, K) : K;
  const GemmLayout row = l == kWgrad ? kWgradSplit : kSplit;
  for (const TileCost &t : kTiles) {
    if (t.cost[row][0] == 0.f || !tile_allowed(t, M, N)) continue;
    const bool small = t.bm * t.bn < 128 * 128;
    const long n = tile_count(t, M, N);
    for (int s = 2; s <= max_s && (s == 2 || n * s <= 1024); ++s) {
      if (small && n * s <= 256) continue;
      const int kc = ((K + s - 1) / s + 63) / 64 * 64;
      if ((K + kc - 1) / kc != s || kc > max_chunk) continue;
      const float us = gemm_cost(t, row, n * s, kc / 64) +
                       static_cast<float>(s + 1) * static_cast<float>(M) * static_cast<float>(N) * (4.f / 4.5e6f);
      if (best.splits == 1 || us < best_us) {
        best_us = us;
        best = {s, kc, {t.bm, t.bn}};
      }
    }
  }
  return best;
}

inline long tiles_256(int M, int N) { return static_cast<long>((M + 255) / 256) * ((N + 255) / 256); }

// Weight gradient: M output rows, N output columns, K tokens.
inline SplitPlan wgrad_split_plan(int M, int N, int K) {
  if (K >= 2 * kMinSplitTokens && tiles_256(M, N) <= 64) {
    const SplitPlan sp = best_split(M, N, K, kWgrad);
    if (sp.splits > 1) return sp;
  }
  return {1, K, choose_tile(M, N, K, kWgrad)};
}

// Forward / input-gradient product (output [M, N], contraction K over
// k-contiguous rows, so K a multiple of 64).  One plan for both: their
// workspace query does not tell them apart.
inline SplitPlan gemm_split_plan(int M, int N, int K) {
  if (K % 64 == 0 && K >= 2 * kMinSplitTokens && tiles_256(M, N) <= 32) {
    const SplitPlan sp = best_split(M, N, K, kFwd);
    if (sp.splits > 1) return sp;
  }
  return {1, K, choose_tile(M, N, K, kFwd)};
}

// Whether the direct-to-LDS kernels take a product (operands A(m, k) and
// B(n, k) with leading dimensions lda, ldb; AT / BT: stored k-major):
// contiguous-k operands need whole 64-wide k-steps, and the operand extents
// that bound the buffer loads keep every offset below 2^32.  The others run
// the register-staged kernel.
inline bool lds_fits(int M, int N, int K, int lda, int ldb, bool AT, bool BT) {
  if ((!AT || !BT) && K % 64 != 0) return false;
  const unsigned long long lim = (1ull << 32) - 1;
  const unsigned long long a_bytes = static_cast<unsigned long long>(AT ? K : M) * lda * 2;
  const unsigned long long b_bytes = static_cast<unsigned long long>(BT ? K : N) * ldb * 2;
  return a_bytes + 600ull * lda * 2 <= lim && b_bytes + 600ull * ldb * 2 <= lim;
}

// Tile of the register-staged kernel: 256x128 once that grid has 512 tiles,
// else 128x128.
inline TileShape any_tile(int M, int N) {
  const long big = static_cast<long>((M + 255) / 256) * ((N + 127) / 128);
  return big >= 512 ? TileShape{256, 128} : TileShape{128, 128};
}

// Output tile and contraction splits of a product as the launchers take it
// when given a workspace of the queried size (forward: AT = BT = false;
// input gradient: BT; weight gradient: AT and BT, M output rows, N output
// columns, K tokens; gelu: with a GELU or GELU' epilogue).
struct GemmPlan {
  TileShape tile;
  int splits;
};

inline GemmPlan gemm_plan(int M, int N, int K, int lda, int ldb, bool AT, bool BT, bool gelu) {
  const bool wgrad = AT && BT;
  const bool fits = lds_fits(M, N, K, lda, ldb, AT, BT);
  const SplitPlan sp = wgrad ? wgrad_split_plan(M, N, K) : gemm_split_plan(M, N, K);
  const bool split_ok = wgrad ? M % 4 == 0 && N % 4 == 0 : N % 8 == 0;
  if (sp.splits > 1 && split_ok && fits) return {sp.tile, sp.splits};
  if (fits) return {choose_tile(M, N, K, gemm_layout(AT, BT, gelu)), 1};
  return {any_tile(M, N), 1};
}

inline size_t ws_round256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

// Workspace of a split forward or input-gradient product: the fp32 partials
// [S][M][N]; 0 when the plan does not split.
inline size_t gemm_ws_bytes(int M, int N, int K) {
  const SplitPlan sp = gemm_split_plan(M, N, K);
  return sp.splits > 1 ? ws_round256(static_cast<size_t>(sp.splits) * M * N * sizeof(float)) : 0;
}

// Workspace of a split weight gradient: the fp32 partials of dW [S][M][N]
// and of db [S][M], each 256-byte aligned; 0 when the plan does not split.
inline size_t gemm_wgrad_ws_bytes(int M, int N, int K) {
  const SplitPlan sp = wgrad_split_plan(M, N, K);
  if (sp.splits <= 1) return 0;
  return ws_round256(static_cast<size_t>(sp.splits) * M * N * sizeof(float)) +
         ws_round256(static_cast<size_t>(sp.splits) * M * sizeof(float));
}

}  // namespace optimus
