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
// a pair.  Fitted to 28 products per layout (ViT-Tiny to ViT-10B and the
// ViT-22B shard: outputs 192 to 16384 wide, contractions 192 to 16384, every
// tile timed on each): the fit is within 3-8% of the measured times on
// average, and the tiles it picks took 1.5% longer in total than the best tile
// of each product, 18% less than the rule this replaces (256x256, 256x192 or
// 128x128 tiles by area and rounds).  Small tiles pay more per flop (each
// loads (bm + bn) / (bm * bn) operand bytes per flop into LDS, and a short
// k-step is bound by its barrier and LDS latency) but fill the 256 CUs.
// Products with a GELU or GELU' epilogue have rows of their own: the epilogue
// of a 256x256 tile takes 21 and 24 us there against 10 and 7, and tiles two
// to a CU hide it behind each other's loops (ViT-Base MLP-up forward 46 us on
// 128x128 tiles against 59 on 256x192).
enum GemmLayout { kFwd = 0, kDgrad = 1, kWgrad = 2, kFwdGelu = 3, kDgradGelu = 4 };

struct TileShape {
  int bm, bn;
};

struct TileCost {
  int bm, bn, per_cu;
  float cost[5][4];  // [GemmLayout]: step, rest, step of a pair, rest of a pair
};

constexpr TileCost kTiles[] = {
    {256, 256, 1, {{0.94, 9.75}, {0.93, 7.29}, {1.24, 9.25}, {0.94, 20.98}, {0.93, 24.05}}},
    {256, 192, 1, {{0.78, 9.38}, {0.83, 6.73}, {1.02, 8.98}, {0.78, 18.60}, {0.83, 19.00}}},
    {128, 256, 1, {{0.60, 6.15}, {0.64, 4.66}, {0.61, 8.57}, {0.60, 12.24}, {0.64, 13.03}}},
    {128, 192, 1, {{0.53, 5.89}, {0.55, 4.33}, {0.56, 5.71}, {0.53, 9.03}, {0.55, 9.02}}},
    {192, 128, 2, {{0.72, 5.00, 0.97, 7.44}, {0.74, 4.50, 1.07, 2.36}, {0.75, 4.32, 1.13, 7.78}, {0.72, 9.50, 0.97, 20.00}, {0.74, 8.06, 1.07, 12.80}}},
    {128, 128, 2, {{0.54, 7.89, 0.73, 5.68}, {0.59, 2.84, 0.74, 4.58}, {0.66, 0.77, 0.88, 4.44}, {0.54, 5.38, 0.73, 9.17}, {0.59, 4.71, 0.74, 9.63}}},
    {64, 192, 1, {{0.39, 3.37}, {0.38, 2.90}, {0.40, 3.47}, {0.39, 5.62}, {0.38, 6.43}}},
    {64, 128, 2, {{0.29, 2.50, 0.54, 2.18}, {0.28, 1.92, 0.53, 1.72}, {0.30, 2.66, 0.55, 2.21}, {0.29, 5.90, 0.54, 3.62}, {0.28, 7.95, 0.53, 3.77}}},
    {64, 64, 2, {{0.17, 3.20, 0.36, 0.94}, {0.20, 0.86, 0.37, 0.77}, {0.25, 0.24, 0.39, 0.42}, {0.12, 2.94, 0.36, 1.46}, {0.20, 2.00, 0.37, 2.40}}}};

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

inline TilePick pick_tile(int M, int N, int K, GemmLayout l) {
  TilePick best{{0, 0}, 0.f};
  for (const TileCost &t : kTiles) {
    // weight gradients over a few k-steps are their fp32 stores: 64-row tiles
    // (whose loop is cheap, not their epilogue) only beyond five of them
    if (l == kWgrad && t.bm < 128 && K <= 5 * 64) continue;
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
// products split is part of what callers size their workspaces by.  Tile and
// number of splits minimise the cost model's time plus the second kernel's (5
// us and its traffic at 4.5 TB/s, as measured on outputs of 0.3 to 2.4 M
// values); every split covers at least kMinSplitTokens in whole 64-wide
// k-steps (the last takes the remainder).  Tiles below 128x128 are worth it
// only for forward and input-gradient products, where they fill the CUs.
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
  for (const TileCost &t : kTiles) {
    const bool small = t.bm * t.bn < 128 * 128;
    if (l == kWgrad ? t.bm < 128 : !small && (t.bm != 128 || t.bn != 128)) continue;
    const long n = tile_count(t, M, N);
    for (int s = 2; s <= max_s && (s == 2 || n * s <= 1024); ++s) {
      if (l != kWgrad && small && n * s <= 256) continue;
      const int kc = ((K + s - 1) / s + 63) / 64 * 64;
      if ((K + kc - 1) / kc != s || kc > max_chunk) continue;
      const float us = gemm_cost(t, l, n * s, kc / 64) +
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
// columns, K tokens).
struct GemmPlan {
  TileShape tile;
  int splits;
};

inline GemmPlan gemm_plan(int M, int N, int K, int lda, int ldb, bool AT, bool BT) {
  const bool wgrad = AT && BT;
  const bool fits = lds_fits(M, N, K, lda, ldb, AT, BT);
  const SplitPlan sp = wgrad ? wgrad_split_plan(M, N, K) : gemm_split_plan(M, N, K);
  const bool split_ok = wgrad ? M % 4 == 0 && N % 4 == 0 : N % 8 == 0;
  if (sp.splits > 1 && split_ok && fits) return {sp.tile, sp.splits};
  if (fits) return {choose_tile(M, N, K, wgrad ? kWgrad : BT ? kDgrad : kFwd), 1};
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
