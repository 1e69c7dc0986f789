// bf16 MFMA GEMM family for the four projections of the encoder layer, in
// their forward, input-gradient and weight-gradient forms.
//
//   C[m, n] = sum_k A(m, k) * B(n, k),  fp32 accumulation on
//   v_mfma_f32_16x16x32_bf16 (32x32x16 in the register-staged kernel).
//
// Three families.  gemm_half_kernel (256-row tiles) and gemm_ring_kernel
// (smaller tiles) copy tiles straight to LDS: operands whose contraction index
// is contiguous in memory as [row][k], read with ds_read_b128; strided ones
// (the weight in the input gradient, both operands of the weight gradient) as
// they lie, [k][row], read with the transposing ds_read_b64_tr_b16.
// gemm_kernel takes what they don't (contiguous contractions that are no
// multiple of 64, operands of 4 GiB and more): it stages through registers,
// transposing strided operands as 8x8 bf16 blocks with v_perm_b32, into
// [row][k] tiles of rows padded by 16 bytes, double-buffered.
//
// The MFMA is issued as D = Btile * Atile^T so that each lane owns one output
// row m and runs of four consecutive output columns n.
// Epilogues fuse bias, residual, GELU (writing both pre- and post-activation),
// GELU' (for the MLP input gradient) and, for weight gradients, the bias
// gradient as row sums of the transposed A operand (deterministic).
//
// Workgroup order is XCD-aware: MI355X dispatches workgroup i to XCD i % 8,
// so each XCD is given its own block of the tile grid, walked M-fastest in
// groups of row tiles, which keeps the operand panels it shares in its L2.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "kernels.hpp"
#include "lds_dma.hpp"
#include "reduce.hpp"

namespace optimus {

namespace {

// Phi(-|u|) = erfc(|u| / sqrt 2) / 2 for the GELU epilogues, from Abramowitz &
// Stegun, Handbook of Mathematical Functions (1964), formula 7.1.26: for
// x >= 0, erfc(x) = (a1 t + a2 t^2 + a3 t^3 + a4 t^4 + a5 t^5) e^(-x^2) with
// t = 1 / (1 + p x), absolute error <= 1.5e-7 (here halved, the halves taken
// into a1..a5 and 1 / sqrt 2 into p).  The tail is computed directly, so the
// negative side does not cancel in fp32.  On the hardware reciprocal and
// exponential this is a fraction of the library erff's instructions; the
// epilogue evaluates it for every output element and is bound by it (two
// quarter-rate instructions and a dozen others), and results are rounded to bf16.
// Also returns e^(-u^2 / 2), which GELU' needs as well.
__device__ __forceinline__ float phi_tail(float u, float &ex2) {
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, fabsf(u), 1.0f));
  const float v = u * 0.84932180028801904f;  // sqrt(log2(e) / 2)
  ex2 = __builtin_amdgcn_exp2f(-(v * v));
  const float poly = fmaf(
      t, fmaf(t, fmaf(t, fmaf(t, 0.5f * 1.061405429f, -0.5f * 1.453152027f), 0.5f * 1.421413741f), -0.5f * 0.284496736f),
      0.5f * 0.254829592f);
  return poly * (t * ex2);
}

// GELU(u) = u Phi(u) and GELU'(u) = Phi(u) + u phi(u), with Phi(u) =
// 1 - Phi(-u) and phi(u) = e^(-u^2 / 2) / sqrt(2 pi).
__device__ __forceinline__ float gelu_f(float u) {
  float ex2;
  const float h = phi_tail(u, ex2);
  return u * (u >= 0.0f ? 1.0f - h : h);
}

__device__ __forceinline__ float gelu_grad_f(float u) {
  float ex2;
  const float h = phi_tail(u, ex2);
  return fmaf(u * 0.39894228040143268f, ex2, u >= 0.0f ? 1.0f - h : h);
}

// Logical tile for this workgroup.  MI355X dispatches workgroup i to XCD
// i % 8.  When the tile grid splits evenly, the XCDs form two halves along M,
// the four XCDs of a half split its column tiles, and each XCD walks its block
// of tiles in groups of GM row tiles that sweep the block's columns.  Otherwise
// (also when a half has fewer than GM row tiles) each XCD takes one contiguous
// range of logical tiles, grouped by 8 row tiles.  GM is 4 for 256-row tiles
// (on the twelve ViT-22B layer GEMMs 0.7% less time in total than the
// contiguous order) and 8 for the others: the tiles in flight on an XCD, R rows
// by C columns, fetch R * BM + C * BN operand rows, which for 128- and 64-row
// tiles is 14-33% less with R = 8 than with R = 4.
template <int GM>
__device__ __forceinline__ void tile_of(int tiles_m, int tiles_n, int &tm, int &tn) {
  const int pid = blockIdx.x, nb = gridDim.x;
  const int xcd = pid & 7, local = pid >> 3;
  if (tiles_m % 2 == 0 && tiles_n % 4 == 0 && tiles_m >= 2 * GM) {
    const int rows_p = tiles_m / 2, cols_x = tiles_n / 4;
    const int gs = GM * cols_x;
    const int g = local / gs, first_m = g * GM;
    const int gm = min(rows_p - first_m, GM);
    const int in_g = local - g * gs;
    tm = (xcd >> 2) * rows_p + first_m + in_g % gm;
    tn = (xcd & 3) * cols_x + in_g / gm;
    return;
  }
  const int per = nb >> 3, rem = nb & 7;
  const int logical = (xcd < rem) ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
  constexpr int GROUP_M = 8;
  const int group_size = GROUP_M * tiles_n;
  const int g = logical / group_size;
  const int first_m = g * GROUP_M;
  const int gm = min(tiles_m - first_m, GROUP_M);
  const int in_g = logical - g * group_size;
  tm = first_m + in_g % gm;
  tn = in_g / gm;
}

// Split of the contraction handled by this workgroup.  With p.splits > 1 the
// grid holds splits x tiles work items, listed split-major and M-fastest
// within a split; each XCD (workgroup i runs on XCD i % 8) takes one
// contiguous range of that list, so the items on one XCD mostly share a
// split and with it the operand panels of its k-range (the tiles of one
// tile column share the weight-gradient rows' panel, those of one tile row
// the other operand's).  Returns the split; kbeg/klen give its contraction
// range.
template <int GM>
__device__ __forceinline__ int split_of(const GemmArgs &p, int tiles_m, int tiles_n, int &tm, int &tn, int &kbeg,
                                       int &klen) {
  if (p.splits > 1) {
    const int nt = tiles_m * tiles_n;
    const int pid = blockIdx.x, nb = gridDim.x;
    const int xcd = pid & 7, local = pid >> 3, per = nb >> 3, rem = nb & 7;
    const int item = (xcd < rem) ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
    const int split = item / nt, t = item - split * nt;
    tm = t % tiles_m;
    tn = t / tiles_m;
    kbeg = split * p.k_chunk;
    klen = min(p.K - kbeg, p.k_chunk);
    return split;
  }
  tile_of<GM>(tiles_m, tiles_n, tm, tn);
  kbeg = 0;
  klen = p.K;
  return 0;
}

// Output pointers of split `split`: its own partial slice, overwritten.
__device__ __forceinline__ GemmArgs split_outputs(const GemmArgs &p, int split) {
  GemmArgs q = p;
  if (p.splits > 1) {
    q.Wf = p.Wf + static_cast<size_t>(split) * p.split_stride;
    if (q.db) q.db = p.db + static_cast<size_t>(split) * p.M;
    q.accumulate = 0;
  }
  return q;
}

// Epilogue of one wave tile: lane owns row m and columns nb..nb+3 of each
// 32x32 fragment (the MFMA is issued as D = Btile * Atile^T).
template <Epi EPI, int FM, int FN, int WTM, int WTN>
__device__ __forceinline__ void store_tile(const GemmArgs &p, const f32x16_t (&acc)[FM][FN], int m0, int n0, int wm,
                                           int wn, int lane) {
  const int lrow = lane & 31;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int m = m0 + wm * WTM + i * 32 + lrow;
    if (m >= p.M) continue;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int nb = n0 + wn * WTN + j * 32 + q * 8 + (lane >> 5) * 4;
        if (nb >= p.N) continue;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[i][j][q * 4 + e];
        const size_t off = static_cast<size_t>(m) * p.ldy + nb;
        if constexpr (EPI == Epi::kF32) {
          f32x4_t w{v[0], v[1], v[2], v[3]};
          if (p.accumulate) w += *reinterpret_cast<const f32x4_t *>(p.Wf + off);
          *reinterpret_cast<f32x4_t *>(p.Wf + off) = w;
        } else {
          if constexpr (EPI == Epi::kBias || EPI == Epi::kBiasResid || EPI == Epi::kBiasGelu) {
            const u32x2_t bw = *reinterpret_cast<const u32x2_t *>(p.bias + nb);
            v[0] += lo_bf(bw[0]);
            v[1] += hi_bf(bw[0]);
            v[2] += lo_bf(bw[1]);
            v[3] += hi_bf(bw[1]);
          }
          if constexpr (EPI == Epi::kBiasResid || EPI == Epi::kResid) {
            const u32x2_t rw = *reinterpret_cast<const u32x2_t *>(p.R + off);
            v[0] += lo_bf(rw[0]);
            v[1] += hi_bf(rw[0]);
            v[2] += lo_bf(rw[1]);
            v[3] += hi_bf(rw[1]);
          }
          if constexpr (EPI == Epi::kGeluGrad) {
            const u32x2_t uw = *reinterpret_cast<const u32x2_t *>(p.R + off);
            v[0] *= gelu_grad_f(lo_bf(uw[0]));
            v[1] *= gelu_grad_f(hi_bf(uw[0]));
            v[2] *= gelu_grad_f(lo_bf(uw[1]));
            v[3] *= gelu_grad_f(hi_bf(uw[1]));
          }
          *reinterpret_cast<u32x2_t *>(p.Y + off) = u32x2_t{pack2(v[0], v[1]), pack2(v[2], v[3])};
          if constexpr (EPI == Epi::kBiasGelu) {
            *reinterpret_cast<u32x2_t *>(p.Y2 + off) =
                u32x2_t{pack2(gelu_f(v[0]), gelu_f(v[1])), pack2(gelu_f(v[2]), gelu_f(v[3]))};
          }
        }
      }
    }
  }

}

// Epilogue through LDS (direct-to-LDS kernels; the k-loop's buffers are free
// by then).  The tile is written out in chunks of 64 rows: the waves owning a
// chunk store their fp32 results (bias added) into LDS, row-major with a
// 16-byte row pad (conflict-free for the 64-bank LDS), then every thread
// streams whole rows out with 16-byte accesses, applying the residual, GELU,
// GELU' or the fp32 accumulation on the way.  Output rows are written in full
// 128-byte lines instead of 8-byte pieces scattered over 32 rows, with
// non-temporal stores: every CU writes its tile at about the same time, and
// streaming the burst past the caches measured 2% faster over the layer (the
// fp32 weight gradients most, and the LayerNorm backward that reads a GEMM
// output next).
constexpr int kEpiRows = 64;

template <Epi EPI, int BM, int BN, int WM, int WN>
__device__ __forceinline__ void store_tile_lds(const GemmArgs &p, const f32x4_t (&acc)[BM / WM / 16][BN / WN / 16],
                                               int m0, int n0, int wm, int wn, int lane, float *lds) {
  constexpr int NT = WM * WN * 64;
  constexpr int WTM = BM / WM, WTN = BN / WN, FM = WTM / 16, FN = WTN / 16;
  constexpr int LDR = BN + 4;  // floats per LDS row (16-byte pad)
  constexpr int NCH = BM / kEpiRows;
  static_assert(BM % kEpiRows == 0 && kEpiRows % 16 == 0, "epilogue chunking");
  constexpr bool kHasBias = EPI == Epi::kBias || EPI == Epi::kBiasResid || EPI == Epi::kBiasGelu;
  // a second per-element input: the residual, or the saved pre-activation u
  constexpr bool kHasR = EPI == Epi::kBiasResid || EPI == Epi::kResid || EPI == Epi::kGeluGrad;
  constexpr int PRB = BN / 8;                        // 16-byte bf16 segments per row
  constexpr int SEGS = (kEpiRows * PRB + NT - 1) / NT;  // per thread and chunk
  const int tid = threadIdx.x;
  // a lane owns row lane % 16 and four columns of each 16x16 fragment
  const int lrow = lane & 15, lcol = (lane >> 4) * 4;

  // Every load of the epilogue is issued before its first store: loads and
  // stores retire in issue order, so a load issued behind the stores of the
  // previous chunk would wait for them.
  u32x2_t bias_w[kHasBias ? FN : 1];
  if constexpr (kHasBias) {
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int nb = n0 + wn * WTN + j * 16 + lcol;
      bias_w[j] = nb < p.N ? *reinterpret_cast<const u32x2_t *>(p.bias + nb) : u32x2_t{0u, 0u};
    }
  }
  u32x4_t rin[kHasR ? NCH : 1][kHasR ? SEGS : 1];
  if constexpr (kHasR) {
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int sg = 0; sg < SEGS; ++sg) {
        const int it = tid + NT * sg;
        const int gm = m0 + c * kEpiRows + it / PRB, gn = n0 + (it % PRB) * 8;
        const bool in = it < kEpiRows * PRB && gm < p.M && gn < p.N;
        rin[c][sg] = in ? ldg16(p.R + static_cast<size_t>(gm) * p.ldy + gn) : u32x4_t{0u, 0u, 0u, 0u};
      }
  }

#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    __syncthreads();  // LDS free (k-loop reads or the previous chunk's readers done)
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int r0 = wm * WTM + i * 16;  // fragment's first tile row
      if (r0 < c * kEpiRows || r0 >= (c + 1) * kEpiRows) continue;
      const int rl = r0 - c * kEpiRows + lrow;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        f32x4_t v = acc[i][j];
        if constexpr (kHasBias) {
          v[0] += lo_bf(bias_w[j][0]);
          v[1] += hi_bf(bias_w[j][0]);
          v[2] += lo_bf(bias_w[j][1]);
          v[3] += hi_bf(bias_w[j][1]);
        }
        *reinterpret_cast<f32x4_t *>(lds + rl * LDR + wn * WTN + j * 16 + lcol) = v;
      }
    }
    __syncthreads();
    if constexpr (EPI == Epi::kF32) {
      constexpr int PER_ROW = BN / 4;
      for (int it = tid; it < kEpiRows * PER_ROW; it += NT) {
        const int r = it / PER_ROW, cc = (it % PER_ROW) * 4;
        const int gm = m0 + c * kEpiRows + r, gn = n0 + cc;
        if (gm >= p.M || gn >= p.N) continue;
        f32x4_t v = *reinterpret_cast<const f32x4_t *>(lds + r * LDR + cc);
        const size_t off = static_cast<size_t>(gm) * p.ldy + gn;
        if (p.accumulate) v += *reinterpret_cast<const f32x4_t *>(p.Wf + off);
        stg16_nt(p.Wf + off, v);
      }
    } else {
#pragma unroll
      for (int sg = 0; sg < SEGS; ++sg) {
        const int it = tid + NT * sg;
        const int r = it / PRB, cc = (it % PRB) * 8;
        const int gm = m0 + c * kEpiRows + r, gn = n0 + cc;
        if (it >= kEpiRows * PRB || gm >= p.M || gn >= p.N) continue;
        const f32x4_t a = *reinterpret_cast<const f32x4_t *>(lds + r * LDR + cc);
        const f32x4_t b = *reinterpret_cast<const f32x4_t *>(lds + r * LDR + cc + 4);
        float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
        const size_t off = static_cast<size_t>(gm) * p.ldy + gn;
        if constexpr (EPI == Epi::kBiasResid || EPI == Epi::kResid) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[2 * e] += lo_bf(rin[c][sg][e]);
            v[2 * e + 1] += hi_bf(rin[c][sg][e]);
          }
        }
        if constexpr (EPI == Epi::kGeluGrad) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[2 * e] *= gelu_grad_f(lo_bf(rin[c][sg][e]));
            v[2 * e + 1] *= gelu_grad_f(hi_bf(rin[c][sg][e]));
          }
        }
        u32x4_t o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = pack2(v[2 * e], v[2 * e + 1]);
        stg16_nt(p.Y + off, o);
        if constexpr (EPI == Epi::kBiasGelu) {
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = pack2(gelu_f(v[2 * e]), gelu_f(v[2 * e + 1]));
          stg16_nt(p.Y2 + off, o);
        }
      }
    }
  }
}

// Global -> register -> LDS staging of one [ROWS x BK] operand tile.
template <int ROWS, int BK, int NT, bool TRANS>
struct TileLoader;

// Contraction-contiguous operand: X(r, k) = X[r * ld + k].
template <int ROWS, int BK, int NT>
struct TileLoader<ROWS, BK, NT, false> {
  static constexpr int KC = BK / 8;  // 16-byte chunks per row
  static constexpr int CH = ROWS * KC / NT;
  static_assert(ROWS * KC % NT == 0, "tile chunks must divide the threads");
  u32x4_t r[CH];

  __device__ __forceinline__ void load(const bf16_t *__restrict__ X, int ld, int rows, int K, int r0, int k0,
                                       int tid) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = tid + NT * i;
      const int row = c / KC, kc = c % KC;
      const int gr = r0 + row, gk = k0 + kc * 8;
      if (gr < rows && gk < K)
        r[i] = ldg16(X + static_cast<size_t>(gr) * ld + gk);
      else
        r[i] = u32x4_t{0u, 0u, 0u, 0u};
    }
  }
  template <int LDK>
  __device__ __forceinline__ void store(bf16_t *lds, int tid) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = tid + NT * i;
      const int row = c / KC, kc = c % KC;
      *reinterpret_cast<u32x4_t *>(lds + row * LDK + kc * 8) = r[i];
    }
  }
};

// Contraction-strided operand: X(r, k) = X[k * ld + r]; rows come in whole
// groups of 8 (every row count here is a multiple of 8).
template <int ROWS, int BK, int NT>
struct TileLoader<ROWS, BK, NT, true> {
  static constexpr int KB = BK / 8;
  static constexpr int NBLK = (ROWS / 8) * KB;
  static constexpr int TB = (NBLK + NT - 1) / NT;
  u32x4_t r[TB][8];

  __device__ __forceinline__ void load(const bf16_t *__restrict__ X, int ld, int rows, int K, int r0, int k0,
                                       int tid) {
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      const int b = tid + NT * t;
      const int kb = b % KB, rb = b / KB;
      const int gr = r0 + rb * 8;
      const bool rok = (NBLK % NT == 0 || b < NBLK) && gr < rows;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int gk = k0 + kb * 8 + j;
        if (rok && gk < K)
          r[t][j] = ldg16(X + static_cast<size_t>(gk) * ld + gr);
        else
          r[t][j] = u32x4_t{0u, 0u, 0u, 0u};
      }
    }
  }
  template <int LDK>
  __device__ __forceinline__ void store(bf16_t *lds, int tid) {
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      const int b = tid + NT * t;
      if (NBLK % NT != 0 && b >= NBLK) continue;
      const int kb = b % KB, rb = b / KB;
      u32x4_t o[8];
      transpose8x8(r[t], o);
#pragma unroll
      for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4_t *>(lds + (rb * 8 + i) * LDK + kb * 8) = o[i];
    }
  }
  // Row sums over the 8 staged k values of each of the 8 rows of block t.
  __device__ __forceinline__ void rowsum(float acc[TB][8]) const {
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[t][i] += (i & 1) ? hi_bf(r[t][j][i >> 1]) : lo_bf(r[t][j][i >> 1]);
  }
};

template <int BM, int BN, int BK, int WM, int WN, bool AT, bool BT, Epi EPI>
__global__ __launch_bounds__(WM *WN * 64) void gemm_kernel(GemmArgs p) {
  constexpr int NT = WM * WN * 64;
  constexpr int LDK = BK + 8;
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int FM = WTM / 32, FN = WTN / 32;
  constexpr int STAGE = (BM + BN) * LDK;
  static_assert(WTM % 32 == 0 && WTN % 32 == 0 && BK % 16 == 0, "tile shape");
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];

  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int wm = wid / WN, wn = wid % WN;
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
  int tm, tn;
  tile_of<4>(tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;

  TileLoader<BM, BK, NT, AT> la;
  TileLoader<BN, BK, NT, BT> lb;
  constexpr bool kDb = (EPI == Epi::kF32) && AT;
  constexpr int DB_TB = AT ? TileLoader<BM, BK, NT, true>::TB : 1;
  float dbacc[DB_TB][8];
  const bool do_db = kDb && p.db != nullptr && tn == 0;
  if constexpr (kDb) {
#pragma unroll
    for (int t = 0; t < DB_TB; ++t)
#pragma unroll
      for (int i = 0; i < 8; ++i) dbacc[t][i] = 0.f;
  }

  f32x16_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x16_t{};

  const int nk = (p.K + BK - 1) / BK;
  la.load(p.A, p.lda, p.M, p.K, m0, 0, tid);
  lb.load(p.B, p.ldb, p.N, p.K, n0, 0, tid);
  if constexpr (kDb) {
    if (do_db) la.rowsum(dbacc);
  }
  la.template store<LDK>(smem, tid);
  lb.template store<LDK>(smem + BM * LDK, tid);
  __syncthreads();

  const int lrow = lane & 31, lk = (lane >> 5) * 8;
  for (int t = 0; t < nk; ++t) {
    const bf16_t *As = smem + (t & 1) * STAGE;
    const bf16_t *Bs = As + BM * LDK;
    const bool more = (t + 1) < nk;
    if (more) {
      la.load(p.A, p.lda, p.M, p.K, m0, (t + 1) * BK, tid);
      lb.load(p.B, p.ldb, p.N, p.K, n0, (t + 1) * BK, tid);
    }
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      bf16x8_t af[FM], bfr[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i)
        af[i] = *reinterpret_cast<const bf16x8_t *>(As + (wm * WTM + i * 32 + lrow) * LDK + kk * 16 + lk);
#pragma unroll
      for (int j = 0; j < FN; ++j)
        bfr[j] = *reinterpret_cast<const bf16x8_t *>(Bs + (wn * WTN + j * 32 + lrow) * LDK + kk * 16 + lk);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = mfma32(bfr[j], af[i], acc[i][j]);
    }
    if (more) {
      if constexpr (kDb) {
        if (do_db) la.rowsum(dbacc);
      }
      bf16_t *Ns = smem + ((t + 1) & 1) * STAGE;
      la.template store<LDK>(Ns, tid);
      lb.template store<LDK>(Ns + BM * LDK, tid);
    }
    __syncthreads();
  }

  store_tile<EPI, FM, FN, WTM, WTN>(p, acc, m0, n0, wm, wn, lane);

  // ---- fused bias gradient: row sums of A over all k (column tile 0 only)
  if constexpr (kDb) {
    if (do_db) {
      constexpr int KB = BK / 8;
#pragma unroll
      for (int t = 0; t < DB_TB; ++t) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          float s = dbacc[t][i];
#pragma unroll
          for (int o = 1; o < KB; o <<= 1) s += __shfl_xor(s, o, kWave);
          dbacc[t][i] = s;
        }
        const int b = tid + NT * t;
        const int rb = b / KB;
        const int gr = m0 + rb * 8;
        if ((b % KB) == 0 && b < TileLoader<BM, BK, NT, true>::NBLK && gr < p.M) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            float s = dbacc[t][i];
            if (p.accumulate) s += p.db[gr + i];
            p.db[gr + i] = s;
          }
        }
      }
    }
  }
}

// ===========================================================================
// Direct-to-LDS pipeline (the large-problem path).
//
// Tiles go from HBM straight into LDS with buffer_load_dwordx4 ... lds (no
// staging registers), some k-steps ahead of the MFMAs that read them (each
// pipeline below says how many).  The buffer resource bounds every
// operand tensor: rows past its end (tokens past M, weight rows past N, or
// contraction rows past K of a transposed operand) read as zero.
//
// LDS tile layouts (16-byte chunks, XOR-swizzled against bank conflicts):
//  - contraction-contiguous operand: [row][BK], chunk c of row r stored at
//    c ^ ((r / RP) % CPR) (RP rows share one 128-byte line); MFMA operands
//    are single ds_read_b128.
//  - contraction-strided operand: [BK][ROWS] exactly as in memory, its
//    chunks swizzled by t_swz; MFMA operands are two ds_read_b64_tr_b16, whose
//    16-lane transpose delivers a lane one column of consecutive k-rows.
// ===========================================================================

// LDS is 64 banks x 4 bytes (256 bytes per cycle); a 16-lane quarter-wave
// of ds_read_b128 and a half-wave of ds_read_b64_tr_b16 must hit distinct
// banks.  nt tiles: RP rows share one 256-byte bank line, so chunk c of row
// r goes to c ^ ((r / RP) % CPR).  Transposed tiles: t_swz below.
template <int BK>
struct NtTile {
  static constexpr int RB = BK * 2;                          // bytes per row
  static constexpr int RP = (256 / RB) > 0 ? (256 / RB) : 1;  // rows per bank line
  static constexpr int CPR = BK / 8;                         // 16-byte chunks per row
  __device__ static __forceinline__ int off(int r, int c) { return r * RB + ((c ^ ((r / RP) % CPR)) << 4); }
};

// Chunk swizzle of k-row k of a transposed tile: the eight k-rows that a
// half-wave of transpose reads touches (0..3 and 8..11 of 16, or 4..7 and
// 12..15) go to eight disjoint 32-byte ranges.
__device__ __forceinline__ int t_swz(int k) { return ((k & 3) << 1) | (((k >> 3) & 1) << 3); }

template <int BM, int BN, int BK, int WM, int WN, bool AT, bool BT, Epi EPI>
bool launch_cfg(const GemmArgs &a, hipStream_t s) {
  constexpr int NT = WM * WN * 64;
  constexpr size_t lds = 2 * static_cast<size_t>(BM + BN) * (BK + 8) * sizeof(bf16_t);
  auto kern = gemm_kernel<BM, BN, BK, WM, WN, AT, BT, EPI>;
  const int tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  hipLaunchKernelGGL(kern, dim3(tiles), dim3(NT), lds, s, a);
  return true;
}

// Tile choice: 256x128 tiles (4 waves of 128x64) when the problem yields at
// least two waves of such tiles on 256 CUs; else 128x128 (4 waves of 64x64).
template <bool AT, bool BT, Epi EPI>
bool launch_any(const GemmArgs &a, hipStream_t s) {
  if (any_tile(a.M, a.N).bm == 256) return launch_cfg<256, 128, 64, 2, 2, AT, BT, EPI>(a, s);
  return launch_cfg<128, 128, 64, 2, 2, AT, BT, EPI>(a, s);
}

// ---------------------------------------------------------------------------
// Half-tile pipeline: 8 waves, two per SIMD (waves w and w + 4), in two groups
// one slot apart, so that on every SIMD one wave issues MFMAs while the other
// reads LDS and issues loads.  Each operand's k-step (64 wide) is two half
// tiles: the first and the second half of every wave's rows.  A k-step is four
// pairs of slots, one quadrant of the output each; X is the B half that is
// already in registers, Y the other one:
//   L0 reads A0          M0 = A0 x X
//   L1 reads Y           M1 = A0 x Y
//   L2 reads A1          M2 = A1 x Y
//   L3 reads Y of t + 1  M3 = A1 x X     (X and Y swap from step to step)
// A barrier ends every slot.  A wave's reads of an L slot retire in its M
// slot (the MFMAs wait for them one by one, so the latency of the later reads
// hides behind the earlier MFMAs), before the barrier that ends it.  Each L
// slot also issues a load two k-steps ahead, into the half tile that was read
// two L slots before: both groups' reads of it have retired by then.  A load
// thus has 10 slots, 1.25 k-steps, before the wait that precedes its first
// read, and up to 6 of the 8 half tiles in LDS are in flight.
//
// What bounds it: the loop holds no vector instructions other than MFMAs and LDS
// reads (addresses in registers, scalar load addressing).  Over one round of
// tiles and 1024 to 1920 k-steps, where starts and epilogues count for little,
// the matrix cores are busy 0.91 of the cycles at a clock of 1.5 GHz (forward,
// 256x256), 0.83 at 1.7 (forward, 256x192), 0.82 at 1.7 (input gradient) and
// 0.72 at 1.85 (weight gradient), where the nominal clock is 2.4: the busier
// they are, the lower the clock that the power budget leaves.  So the fragments
// are 16x16x32: a register-only loop (enc_calib_mfma) runs 2.04 to 2.16 PFLOP/s
// on them against 1.80 to 1.95 on 32x32x16.  With transpose reads (strided
// operands) the LDS pipe's instruction rate binds next: about 4.3 cycles each,
// 24 per wave and k-step for one strided operand, 36 or 48 for two.  In the
// ViT-22B layer itself the products are at 0.49 to 0.77 busy: there their
// rounds' starts and epilogues are not hidden.  Measured on that layer (us,
// against the kernels this replaced, on 32x32x16 with a whole k-step per
// barrier): QKV forward 401 -> 342, out-projection forward 136 -> 118, MLP-up
// forward 548 -> 473, MLP-down forward 532 -> 451, MLP-down input gradient
// 540 -> 478, MLP-up 551 -> 511, QKV 417 -> 391, weight gradients 526 -> 513,
// 537 -> 520, 410 -> 397.
// ---------------------------------------------------------------------------

// One 1 KB wave load straight to LDS at base + OFF + 16 * lane.  M0 (the LDS
// address) is left set: nothing else here reads it without setting it.
template <int OFF>
__device__ __forceinline__ void issue_lds16(const u32x4_t &rsrc, uint32_t base, uint32_t voff, uint32_t soff) {
  asm volatile(
      "s_add_u32 m0, %0, %4\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %1, %2, %3 offen lds"
      :
      : "s"(base), "v"(voff), "s"(rsrc), "s"(soff), "i"(OFF)
      : "memory", "scc");
}
// The same for the lanes of `mask` only.
template <int OFF>
__device__ __forceinline__ void issue_lds16(const u32x4_t &rsrc, uint32_t base, uint32_t voff, uint32_t soff,
                                            uint64_t mask) {
  asm volatile(
      "s_add_u32 m0, %0, %4\n\t"
      "s_mov_b64 exec, %5\n\t"
      "buffer_load_dwordx4 %1, %2, %3 offen lds\n\t"
      "s_mov_b64 exec, -1"
      :
      : "s"(base), "v"(voff), "s"(rsrc), "s"(soff), "i"(OFF), "s"(mask)
      : "memory", "scc");
}

// One operand's half tiles: NWV waves of 2 * FH fragments of 16 rows each;
// half h holds each wave's fragments [h * FH, (h + 1) * FH).
template <int NWV, int FH, bool TRANS>
struct HalfTile {
  static constexpr int BK = 64, KS = 2;                      // two 32-wide contraction steps
  static constexpr int HR = FH * 16, WROWS = 2 * HR;         // rows per wave in a half, in the tile
  static constexpr int ROWS = NWV * HR;                      // rows of a half tile
  static constexpr int LROWS = TRANS ? 128 : ROWS;           // (transposed rows are padded)
  static constexpr int BYTES = LROWS * BK * 2;               // LDS bytes of a half tile
  static constexpr int WB = BYTES / 8;                       // per wave
  static constexpr int NI = (WB + 1023) / 1024;              // loads per wave and half tile
  static constexpr bool MASKED = ROWS != LROWS || WB % 1024 != 0;
  static_assert(ROWS <= 128 && WB % 16 == 0, "half tile shape");
  static constexpr int NOFF = TRANS ? FH : KS;
  uint32_t voff[NI];
  uint64_t mask[NI];
  uint32_t half_off;
  u32x4_t rsrc;
  int off[NOFF];  // LDS offset of this wave's fragments in a half tile

  __device__ __forceinline__ void init(const bf16_t *base, uint32_t nbytes, int ld, int r0, int w, int wid, int lane,
                                       int lds_base) {
    rsrc = make_rsrc(base, nbytes);
    half_off = __builtin_amdgcn_readfirstlane(TRANS ? HR * 2 : static_cast<uint32_t>(HR) * ld * 2);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int o = wid * WB + i * 1024 + lane * 16;
      bool live = i * 1024 + lane * 16 < WB;
      if constexpr (!TRANS) {
        using T = NtTile<BK>;
        const int br = o / T::RB, pch = (o % T::RB) >> 4;
        const int c = pch ^ ((br / T::RP) % T::CPR);
        const int r = br / HR * WROWS + br % HR;
        voff[i] = static_cast<uint32_t>(((r0 + r) * static_cast<long>(ld) + c * 8) * 2);
      } else {
        const int k = o / (LROWS * 2), pch = (o % (LROWS * 2)) >> 4;
        const int bc = (pch ^ t_swz(k)) * 8;
        live = live && bc < ROWS;
        const int c = bc / HR * WROWS + bc % HR;
        voff[i] = static_cast<uint32_t>((k * static_cast<long>(ld) + r0 + c) * 2);
      }
      mask[i] = __ballot(live);
    }
    // fragment f of k-step kk: lane holds row lane % 16 of the fragment and
    // contraction elements 8 * (lane / 16) .. + 7
    if constexpr (!TRANS) {
#pragma unroll
      for (int kk = 0; kk < KS; ++kk)
        off[kk] = lds_base + NtTile<BK>::off(w * HR + (lane & 15), kk * 4 + (lane >> 4));
    } else {
      const int k = 8 * (lane >> 4) + ((lane & 15) >> 2);
#pragma unroll
      for (int f = 0; f < FH; ++f) {
        const int n = w * HR + f * 16 + 4 * (lane & 3);
        off[f] = lds_base + k * (LROWS * 2) + (((n >> 3) ^ t_swz(k)) << 4) + (n & 7) * 2;
      }
    }
    // addresses stay in registers: computed in the loop they would take issue
    // slots from the other group's MFMAs
#pragma unroll
    for (int i = 0; i < NOFF; ++i) asm volatile("" : "+v"(off[i]));
  }
  template <int OFF>
  __device__ __forceinline__ void issue(uint32_t wbase, uint32_t soff) const {
    issue_one<OFF, 0>(wbase, soff);
    if constexpr (NI > 1) issue_one<OFF, 1>(wbase, soff);
  }
  template <int OFF, int I>
  __device__ __forceinline__ void issue_one(uint32_t wbase, uint32_t soff) const {
    if constexpr (MASKED)
      issue_lds16<OFF + I * 1024>(rsrc, wbase, voff[I], soff, mask[I]);
    else
      issue_lds16<OFF + I * 1024>(rsrc, wbase, voff[I], soff);
  }
  __device__ __forceinline__ bf16x8_t get(const lds_char *half, int f, int kk) const {
    if constexpr (!TRANS) {
      return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8_t *>(half + off[kk] + f * 16 * BK * 2);
    } else {
      const lds_char *q = half + off[f] + kk * 32 * LROWS * 2;
      return lds_read_tr(q, q + 4 * LROWS * 2);
    }
  }
};

template <int N>
using cnt = std::integral_constant<int, N>;

template <int WM, int WN, int FMH, int FNH, bool AT, bool BT, Epi EPI>
__global__ __launch_bounds__(512, 1) void gemm_half_kernel(GemmArgs p, uint32_t a_bytes, uint32_t b_bytes) {
  static_assert(WM * WN == 8, "eight waves, two per SIMD");
  constexpr int BM = WM * FMH * 32, BN = WN * FNH * 32, BK = 64, KS = 2;
  constexpr int WTM = BM / WM, FM = 2 * FMH, FN = 2 * FNH;
  using TA = HalfTile<WM, FMH, AT>;
  using TB = HalfTile<WN, FNH, BT>;
  constexpr int NA = TA::NI, NB = TB::NI;
  // LDS: [A: stage 0 half 0, half 1, stage 1 half 0, half 1] [B: the same]
  constexpr int B_BASE = 4 * TA::BYTES;
  // A fragments read one L slot early when A takes transpose reads (twice the
  // LDS instructions): evens the L slots out
  constexpr int PRE = AT ? FMH / 2 : 0;
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
  const lds_char *smem = (const lds_char *)(smem_raw);

  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wid >> 2;
  const int wm = wid / WN, wn = wid % WN;
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
  int tm, tn, kbeg, klen;
  const int split = split_of<4>(p, tiles_m, tiles_n, tm, tn, kbeg, klen);
  const int m0 = tm * BM, n0 = tn * BN;

  TA la;
  TB lb;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  la.init(p.A, a_bytes, p.lda, m0, wm, wid, lane, 0);
  lb.init(p.B, b_bytes, p.ldb, n0, wn, wid, lane, B_BASE);
  const uint32_t a_step = AT ? static_cast<uint32_t>(BK) * p.lda * 2 : BK * 2;
  const uint32_t b_step = BT ? static_cast<uint32_t>(BK) * p.ldb * 2 : BK * 2;
  // byte offsets of the k-step whose loads are issued next
  uint32_t so_a = AT ? static_cast<uint32_t>(kbeg) * p.lda * 2 : static_cast<uint32_t>(kbeg) * 2;
  uint32_t so_b = BT ? static_cast<uint32_t>(kbeg) * p.ldb * 2 : static_cast<uint32_t>(kbeg) * 2;
  const uint32_t wa = __builtin_amdgcn_readfirstlane(lds0 + wid * TA::WB);
  const uint32_t wb = __builtin_amdgcn_readfirstlane(lds0 + B_BASE + wid * TB::WB);

  f32x4_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // Weight gradient: the bias gradient db[m] = sum_k A(m, k), summed from the
  // A fragments in registers by the first column tile's workgroups; each wave
  // column takes the fragments i % WN == wn of a half (fixed order:
  // deterministic).
  constexpr bool kDb = (EPI == Epi::kF32) && AT;
  constexpr int DBF = (FMH + WN - 1) / WN;
  const bool do_db = kDb && p.db != nullptr && tn == 0;
  float dbacc[2][DBF];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < DBF; ++i) dbacc[h][i] = 0.f;

  const int nk = (klen + BK - 1) / BK;
  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};
  auto issue_a = [&](auto st, auto h) {
    la.template issue<(st.value * 2 + h.value) * TA::BYTES>(wa, so_a + (h.value ? la.half_off : 0u));
  };
  auto issue_b = [&](auto st, auto h) {
    lb.template issue<(st.value * 2 + h.value) * TB::BYTES>(wb, so_b + (h.value ? lb.half_off : 0u));
  };
  auto barrier = [] {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  bf16x8_t a[KS][FMH], b0[KS][FNH], b1[KS][FNH], pre[2][PRE > 0 ? PRE : 1];
  auto read_pre = [&](auto st, auto h) {
    if constexpr (PRE > 0) {
#pragma unroll
      for (int i = 0; i < PRE; ++i) pre[h.value][i] = la.get(smem + (st.value * 2 + h.value) * TA::BYTES, i, 0);
    }
  };
  auto read_a = [&](auto st, auto h) {
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
#pragma unroll
      for (int i = 0; i < FMH; ++i)
        if (kk > 0 || i >= PRE) a[kk][i] = la.get(smem + (st.value * 2 + h.value) * TA::BYTES, i, kk);
  };
  auto read_b = [&](auto st, auto h) {
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
#pragma unroll
      for (int j = 0; j < FNH; ++j)
        (h.value ? b1 : b0)[kk][j] = lb.get(smem + (st.value * 2 + h.value) * TB::BYTES, j, kk);
  };
  // one quadrant; SUM: also add this A half's rows into the bias gradient
  auto mma = [&](auto ahc, auto bhc, auto sum) {
    constexpr int ah = decltype(ahc)::value, bh = decltype(bhc)::value;
    auto fa = [&](int kk, int i) { return (kk == 0 && i < PRE) ? pre[ah][i < PRE ? i : 0] : a[kk][i]; };
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
#pragma unroll
      for (int i = 0; i < FMH; ++i)
#pragma unroll
        for (int j = 0; j < FNH; ++j)
          acc[ah * FMH + i][bh * FNH + j] =
              mfma16((bh ? b1 : b0)[kk][j], fa(kk, i), acc[ah * FMH + i][bh * FNH + j]);
    wait_vmcnt<63, 0>();  // this slot's reads retired before the barrier (the data was used above)
    if constexpr (decltype(sum)::value) {
#pragma unroll
      for (int i = 0; i < FMH; ++i) {
        if (i % WN != wn) continue;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
          const u32x4_t w = __builtin_bit_cast(u32x4_t, fa(kk, i));
#pragma unroll
          for (int e = 0; e < 4; ++e) dbacc[ah][i / WN] = add_pair(w[e], dbacc[ah][i / WN]);
        }
      }
    }
  };

  // k-steps 0 and 1, in the order the loop reads them (X of step 0 is B0, of
  // step 1 B1)
  issue_b(c0, c0);
  issue_a(c0, c0);
  issue_b(c0, c1);
  issue_a(c0, c1);
  so_a += a_step;
  so_b += b_step;
  if (nk > 1) {
    issue_b(c1, c1);
    issue_a(c1, c0);
    issue_b(c1, c0);
    so_b += b_step;
    wait_vmcnt<2 * NA + 3 * NB>();
  } else {
    wait_vmcnt<NA + NB>();
  }
  barrier();
  read_b(c0, c0);
  read_pre(c0, c0);
  wait_vmcnt<63, 0>();
  barrier();
  if (grp == 1) barrier();  // group 1 runs one slot behind

  // Waits of the steady state (both k-steps t + 1 and t + 2 exist), of the
  // last but one k-step and of the last: each leaves in flight exactly the
  // loads younger than what the next L slot reads.
  auto wait3 = [](bool more2, bool more1, auto n2, auto n1, auto n0) {
    if (more2)
      wait_vmcnt<n2.value>();
    else if (more1)
      wait_vmcnt<n1.value>();
    else
      wait_vmcnt<n0.value>();
  };
  // One k-step in stage st.  FULL: k-steps t + 1 and t + 2 exist.
  auto step = [&](auto st, auto full, auto db, int t) {
    constexpr bool FULL = decltype(full)::value;
    constexpr std::integral_constant<int, st.value> X{};
    constexpr std::integral_constant<int, 1 - st.value> Y{};
    constexpr int PA = PRE > 0 ? NA : 0;  // (the early reads need A one slot sooner)
    const bool more2 = FULL || t + 2 < nk, more1 = FULL || t + 1 < nk;
    // ---- L0, M0
    if (more1) issue_a(Y, c1);
    so_a += a_step;
    read_a(st, c0);
    wait3(more2, more1, cnt<3 * NA + 2 * NB - PA>(), cnt<3 * NA + 2 * NB - PA>(), cnt<NA - PA>());
    barrier();
    mma(c0, X, db);
    barrier();
    // ---- L1, M1
    if (more2) issue_b(st, X);
    read_b(st, Y);
    read_pre(st, c1);
    wait3(more2, more1, cnt<2 * NA + 3 * NB>(), cnt<2 * (NA + NB)>(), c0);
    barrier();
    mma(c0, Y, c0);
    barrier();
    // ---- L2, M2
    if (more2) issue_a(st, c0);
    read_a(st, c1);
    wait3(more2, more1, cnt<3 * NA + 2 * NB - PA>(), cnt<2 * NA + NB - PA>(), c0);
    barrier();
    mma(c1, Y, db);
    barrier();
    // ---- L3, M3 (after the last k-step the reads return stale data, unused)
    if (more2) issue_b(st, Y);
    read_b(Y, Y);
    read_pre(Y, c0);
    wait3(more2, more1, cnt<2 * NA + 3 * NB>(), cnt<NA + NB>(), c0);
    barrier();
    mma(c1, X, c0);
    so_b += b_step;
    barrier();
  };
  auto k_loop = [&](auto db) {
    int t = 0;
    for (; t + 3 < nk; t += 2) {
      step(c0, c1, db, t);
      step(c1, c1, db, t + 1);
    }
    for (;;) {
      step(c0, c0, db, t);
      if (++t >= nk) break;
      step(c1, c0, db, t);
      if (++t >= nk) break;
    }
  };
  if constexpr (kDb) {
    // two copies of the loop: a test of do_db inside it costs every workgroup
    if (do_db)
      k_loop(c1);
    else
      k_loop(c0);
  } else {
    k_loop(c0);
  }
  if (grp == 0) barrier();  // match group 1's extra barrier

  const GemmArgs q = split_outputs(p, split);
  store_tile_lds<EPI, BM, BN, WM, WN>(q, acc, m0, n0, wm, wn, lane, reinterpret_cast<float *>(smem_raw));
  if constexpr (kDb) {
    if (do_db) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < DBF; ++i) {
          // the four 16-lane groups hold the k residues of row lane % 16
          float tot = dbacc[h][i] + __shfl_xor(dbacc[h][i], 16, kWave);
          tot += __shfl_xor(tot, 32, kWave);
          const int f = i * WN + wn;
          const int row = m0 + wm * WTM + (h * FMH + f) * 16 + (lane & 15);
          if (f < FMH && lane < 16 && row < q.M) q.db[row] = q.accumulate ? q.db[row] + tot : tot;
        }
    }
  }
}

template <int WM, int WN, int FMH, int FNH, bool AT, bool BT, Epi EPI>
bool launch_half_cfg(const GemmArgs &a, uint32_t a_bytes, uint32_t b_bytes, hipStream_t s) {
  constexpr int BM = WM * FMH * 32, BN = WN * FNH * 32;
  constexpr size_t pipe = 4 * (HalfTile<WM, FMH, AT>::BYTES + HalfTile<WN, FNH, BT>::BYTES);
  constexpr size_t epi = static_cast<size_t>(kEpiRows) * (BN + 4) * sizeof(float);
  constexpr size_t lds = pipe > epi ? pipe : epi;
  static_assert(lds <= 160 * 1024, "LDS budget");
  const int tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN) * (a.splits > 1 ? a.splits : 1);
  hipLaunchKernelGGL((gemm_half_kernel<WM, WN, FMH, FNH, AT, BT, EPI>), dim3(tiles), dim3(512), lds, s, a, a_bytes,
                     b_bytes);
  return true;
}

// ---------------------------------------------------------------------------
// Ring pipeline for smaller tiles: 8 waves in two groups one slot apart, as
// above, with one pair of slots per k-step (64 wide): L reads all of the
// k-step's fragments and issues this wave's share of the k-step S - 1 ahead,
// M issues its MFMAs.  A small tile's k-step is short, so the loads need
// several k-steps of lead: S stages fill the LDS.
//
// K-step t is read by group 0 in slot 2t and by group 1 in slot 2t + 1, both
// retired before the barrier that ends the slot; its stage is refilled from
// slot 2t + 2 on.  Each wave waits for its own share of k-step t + 1 at the
// end of its L(t), so both groups' shares have landed before slot 2t + 2.
// ---------------------------------------------------------------------------

// One operand's [ROWS x 64] tile: per-wave loads and fragment addresses.
template <int ROWS, int F, int S, bool TRANS>
struct RingTile {
  static constexpr int BK = 64, KS = 2;
  static constexpr int BYTES = ROWS * BK * 2, WB = BYTES / 8, NI = WB / 1024;  // per wave: whole 1 KB loads
  static constexpr int G = 65536 / BYTES < S ? 65536 / BYTES : S;  // stages one address register reaches
  static constexpr int NG = (S + G - 1) / G, NOFF = TRANS ? F : KS;
  static_assert(ROWS % 64 == 0 && G >= 1, "tile shape");
  uint32_t voff[NI];
  u32x4_t rsrc;
  int off[NG][NOFF];

  // 128-byte multiples alternate between the halves of a 256-byte bank line
  // from k-row to k-row, so one XOR bit less spreads the eight k-rows
  __device__ static __forceinline__ int swz(int k) {
    return ROWS % 128 == 0 ? t_swz(k) : ((((k >> 1) & 1) | (((k >> 3) & 1) << 1)) << 1);
  }
  __device__ __forceinline__ void init(const bf16_t *base, uint32_t nbytes, int ld, int r0, int w, int wid, int lane,
                                       int lds_base) {
    rsrc = make_rsrc(base, nbytes);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int o = wid * WB + i * 1024 + lane * 16;
      if constexpr (!TRANS) {
        using T = NtTile<BK>;
        const int r = o / T::RB, pch = (o % T::RB) >> 4;
        const int c = pch ^ ((r / T::RP) % T::CPR);
        voff[i] = static_cast<uint32_t>(((r0 + r) * static_cast<long>(ld) + c * 8) * 2);
      } else {
        const int k = o / (ROWS * 2), pch = (o % (ROWS * 2)) >> 4;
        const int c = (pch ^ swz(k)) * 8;
        voff[i] = static_cast<uint32_t>((k * static_cast<long>(ld) + r0 + c) * 2);
      }
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int gb = lds_base + g * G * BYTES;
      if constexpr (!TRANS) {
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
          off[g][kk] = gb + NtTile<BK>::off(w * F * 16 + (lane & 15), kk * 4 + (lane >> 4));
      } else {
        const int k = 8 * (lane >> 4) + ((lane & 15) >> 2);
#pragma unroll
        for (int f = 0; f < F; ++f) {
          const int n = w * F * 16 + f * 16 + 4 * (lane & 3);
          off[g][f] = gb + k * (ROWS * 2) + (((n >> 3) ^ swz(k)) << 4) + (n & 7) * 2;
        }
      }
#pragma unroll
      for (int i = 0; i < NOFF; ++i) asm volatile("" : "+v"(off[g][i]));
    }
  }
  template <int OFF, int I = 0>
  __device__ __forceinline__ void issue(uint32_t wbase, uint32_t soff) const {
    if constexpr (I < NI) {
      issue_lds16<OFF + I * 1024>(rsrc, wbase, voff[I], soff);
      issue<OFF, I + 1>(wbase, soff);
    }
  }
  template <int ST>
  __device__ __forceinline__ bf16x8_t get(const lds_char *smem, int f, int kk) const {
    const lds_char *q = smem + (ST % G) * BYTES;
    if constexpr (!TRANS) {
      return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8_t *>(q + off[ST / G][kk] +
                                                                                     f * 16 * BK * 2);
    } else {
      q += off[ST / G][f] + kk * 32 * ROWS * 2;
      return lds_read_tr(q, q + 4 * ROWS * 2);
    }
  }
};

// f(cnt<0>, cnt<1>, ...).
template <class F, int... I>
__device__ __forceinline__ void with_counts(F f, std::integer_sequence<int, I...>) {
  f(cnt<I>()...);
}

// Wait until at most r k-steps of PS loads each are in flight.
template <int PS, int R>
__device__ __forceinline__ void wait_ksteps(int r) {
  if constexpr (R > 0) {
    if (r >= R)
      wait_vmcnt<R * PS, 0>();
    else
      wait_ksteps<PS, R - 1>(r);
  } else {
    wait_vmcnt<0, 0>();
  }
}

template <int WM, int WN, int FM, int FN, int S, int WGS, bool STAG, bool AT, bool BT, Epi EPI>
__global__ __launch_bounds__(512, 2 * WGS) void gemm_ring_kernel(GemmArgs p, uint32_t a_bytes, uint32_t b_bytes) {
  static_assert(WM * WN == 8 && S >= 2, "eight waves, two per SIMD");
  constexpr int BM = WM * FM * 16, BN = WN * FN * 16, BK = 64, KS = 2, D = S - 1;
  using TA = RingTile<BM, FM, S, AT>;
  using TB = RingTile<BN, FN, S, BT>;
  constexpr int PS = TA::NI + TB::NI, B_BASE = S * TA::BYTES;
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
  const lds_char *smem = (const lds_char *)(smem_raw);

  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wid >> 2;
  const int wm = wid / WN, wn = wid % WN;
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
  int tm, tn, kbeg, klen;
  const int split = split_of<8>(p, tiles_m, tiles_n, tm, tn, kbeg, klen);
  const int m0 = tm * BM, n0 = tn * BN;

  TA la;
  TB lb;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  la.init(p.A, a_bytes, p.lda, m0, wm, wid, lane, 0);
  lb.init(p.B, b_bytes, p.ldb, n0, wn, wid, lane, B_BASE);
  const uint32_t a_step = AT ? static_cast<uint32_t>(BK) * p.lda * 2 : BK * 2;
  const uint32_t b_step = BT ? static_cast<uint32_t>(BK) * p.ldb * 2 : BK * 2;
  uint32_t so_a = AT ? static_cast<uint32_t>(kbeg) * p.lda * 2 : static_cast<uint32_t>(kbeg) * 2;
  uint32_t so_b = BT ? static_cast<uint32_t>(kbeg) * p.ldb * 2 : static_cast<uint32_t>(kbeg) * 2;
  const uint32_t wa = __builtin_amdgcn_readfirstlane(lds0 + wid * TA::WB);
  const uint32_t wb = __builtin_amdgcn_readfirstlane(lds0 + B_BASE + wid * TB::WB);

  f32x4_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  constexpr bool kDb = (EPI == Epi::kF32) && AT;  // fused bias gradient, as above
  constexpr int DBF = (FM + WN - 1) / WN;
  const bool do_db = kDb && p.db != nullptr && tn == 0;
  float dbacc[DBF];
#pragma unroll
  for (int i = 0; i < DBF; ++i) dbacc[i] = 0.f;

  const int nk = (klen + BK - 1) / BK;
  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};
  auto issue = [&](auto st) {
    la.template issue<st.value * TA::BYTES>(wa, so_a);
    lb.template issue<st.value * TB::BYTES>(wb, so_b);
    so_a += a_step;
    so_b += b_step;
  };
  auto barrier = [] {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  bf16x8_t a[KS][FM], b[KS][FN];
  auto step = [&](auto st, auto full, auto db, int t) {
    constexpr bool FULL = decltype(full)::value;
    constexpr int ST = st.value;
    // ---- L (without stagger: the k-step's only barrier precedes it)
    if constexpr (!STAG) {
      if constexpr (FULL)
        wait_vmcnt<(D - 1) * PS>();
      else
        wait_ksteps<PS, D - 1>(min(t + D - 1, nk - 1) - t);
      barrier();
    }
    if (FULL || t + D < nk) issue(cnt<(ST + D) % S>());
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
#pragma unroll
      for (int j = 0; j < FN; ++j) b[kk][j] = lb.template get<ST>(smem, j, kk);
#pragma unroll
      for (int i = 0; i < FM; ++i) a[kk][i] = la.template get<ST>(smem, i, kk);
    }
    if constexpr (STAG) {
      if constexpr (FULL)
        wait_vmcnt<(D - 1) * PS, 0>();
      else
        wait_ksteps<PS, D - 1>(min(t + D, nk - 1) - (t + 1));
      barrier();
    }
    // ---- M
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = mfma16(b[kk][j], a[kk][i], acc[i][j]);
    if constexpr (decltype(db)::value) {
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        if (i % WN != wn) continue;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
          const u32x4_t w = __builtin_bit_cast(u32x4_t, a[kk][i]);
#pragma unroll
          for (int e = 0; e < 4; ++e) dbacc[i / WN] = add_pair(w[e], dbacc[i / WN]);
        }
      }
    }
    if constexpr (STAG)
      barrier();
    else
      wait_vmcnt<63, 0>();  // this k-step's reads retired before the next barrier
  };

  // the first D k-steps
  with_counts([&](auto... i) { ((i.value < nk ? issue(i) : void()), ...); }, std::make_integer_sequence<int, D>{});
  if constexpr (STAG) {
    wait_ksteps<PS, D - 1>(min(D, nk) - 1);
    barrier();
    if (grp == 1) barrier();  // group 1 runs one slot behind
  }

  auto k_loop = [&](auto db) {
    int t = 0;
    for (; t + S - 1 + D < nk; t += S)
      with_counts([&](auto... i) { (step(i, c1, db, t + i.value), ...); }, std::make_integer_sequence<int, S>{});
    while (t < nk)
      with_counts([&](auto... i) { ((t < nk ? (step(i, c0, db, t), void(++t)) : void()), ...); },
                  std::make_integer_sequence<int, S>{});
  };
  if constexpr (kDb) {
    if (do_db)
      k_loop(c1);
    else
      k_loop(c0);
  } else {
    k_loop(c0);
  }
  if (STAG && grp == 0) barrier();  // match group 1's extra barrier

  const GemmArgs q = split_outputs(p, split);
  store_tile_lds<EPI, BM, BN, WM, WN>(q, acc, m0, n0, wm, wn, lane, reinterpret_cast<float *>(smem_raw));
  if constexpr (kDb) {
    if (do_db) {
#pragma unroll
      for (int i = 0; i < DBF; ++i) {
        float tot = dbacc[i] + __shfl_xor(dbacc[i], 16, kWave);
        tot += __shfl_xor(tot, 32, kWave);
        const int f = i * WN + wn;
        const int row = m0 + (wm * FM + f) * 16 + (lane & 15);
        if (f < FM && lane < 16 && row < q.M) q.db[row] = q.accumulate ? q.db[row] + tot : tot;
      }
    }
  }
}

template <int WM, int WN, int FM, int FN, int S, int WGS, bool STAG, bool AT, bool BT, Epi EPI>
bool launch_ring_cfg(const GemmArgs &a, uint32_t a_bytes, uint32_t b_bytes, hipStream_t s) {
  constexpr int BM = WM * FM * 16, BN = WN * FN * 16;
  constexpr size_t pipe = static_cast<size_t>(S) * (RingTile<BM, FM, S, AT>::BYTES + RingTile<BN, FN, S, BT>::BYTES);
  constexpr size_t epi = static_cast<size_t>(kEpiRows) * (BN + 4) * sizeof(float);
  constexpr size_t lds = pipe > epi ? pipe : epi;
  static_assert(lds * WGS <= 160 * 1024, "LDS budget");
  const int tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN) * (a.splits > 1 ? a.splits : 1);
  hipLaunchKernelGGL((gemm_ring_kernel<WM, WN, FM, FN, S, WGS, STAG, AT, BT, EPI>), dim3(tiles), dim3(512), lds, s, a,
                     a_bytes, b_bytes);
  return true;
}

// Direct-to-LDS path on tile t (of kTiles): 256-row tiles run gemm_half_kernel,
// the others gemm_ring_kernel.
// Returns false when the operands do not fit the path's constraints.  Only the
// tiles that the cost table offers these products are compiled (forward and
// input-gradient products write fp32 as partials of a split only).
template <bool AT, bool BT, Epi EPI>
bool launch_lds(const GemmArgs &a, hipStream_t s, TileShape t) {
  constexpr bool gelu = EPI == Epi::kBiasGelu || EPI == Epi::kGeluGrad;
  constexpr GemmLayout row = !AT && EPI == Epi::kF32 ? kSplit : gemm_layout(AT, BT, gelu);
  if (!lds_fits(a.M, a.N, a.K, a.lda, a.ldb, AT, BT)) return false;
  // operand extents (bytes) bound the buffer loads
  const uint32_t ab = static_cast<uint32_t>(static_cast<uint64_t>(AT ? a.K : a.M) * a.lda * 2);
  const uint32_t bb = static_cast<uint32_t>(static_cast<uint64_t>(BT ? a.K : a.N) * a.ldb * 2);
  // Staggered groups pay where a k-step has enough MFMAs to cover the other
  // group's reads: 128x192 tiles 56.8 against 63.5 us on the ViT-22B shard's
  // QKV forward; without them 192x128 tiles (two per CU) 31.4 against 39.1 on
  // the ViT-Base QKV input gradient, 64x128 13.4 against 14.6 at a quarter of
  // its tokens.  64-row tiles with two strided operands are even or better
  // with them.
  if constexpr (tile_offered(256, 256, row))
    if (t.bm == 256 && t.bn == 256) return launch_half_cfg<2, 4, 4, 2, AT, BT, EPI>(a, ab, bb, s);
  if constexpr (tile_offered(256, 192, row))
    if (t.bm == 256 && t.bn == 192) return launch_half_cfg<4, 2, 2, 3, AT, BT, EPI>(a, ab, bb, s);
  if constexpr (tile_offered(128, 256, row))
    if (t.bm == 128 && t.bn == 256) return launch_ring_cfg<2, 4, 4, 4, 3, 1, true, AT, BT, EPI>(a, ab, bb, s);
  if constexpr (tile_offered(128, 192, row))
    if (t.bm == 128 && t.bn == 192) return launch_ring_cfg<2, 4, 4, 3, 4, 1, true, AT, BT, EPI>(a, ab, bb, s);
  if constexpr (tile_offered(192, 128, row))
    if (t.bm == 192 && t.bn == 128) return launch_ring_cfg<4, 2, 3, 4, 2, 2, false, AT, BT, EPI>(a, ab, bb, s);
  if constexpr (tile_offered(128, 128, row))
    if (t.bm == 128 && t.bn == 128) return launch_ring_cfg<2, 4, 4, 2, 2, 2, false, AT, BT, EPI>(a, ab, bb, s);
  if constexpr (tile_offered(64, 192, row))
    if (t.bm == 64 && t.bn == 192) return launch_ring_cfg<2, 4, 2, 3, 4, 1, AT, AT, BT, EPI>(a, ab, bb, s);
  if constexpr (tile_offered(64, 128, row))
    if (t.bm == 64 && t.bn == 128) return launch_ring_cfg<2, 4, 2, 2, 3, 2, AT, AT, BT, EPI>(a, ab, bb, s);
  if constexpr (tile_offered(64, 64, row))
    if (t.bm == 64 && t.bn == 64) return launch_ring_cfg<2, 4, 2, 1, 4, 2, false, AT, BT, EPI>(a, ab, bb, s);
  return false;
}

template <bool AT, bool BT, Epi EPI>
bool launch_lds(const GemmArgs &a, hipStream_t s) {
  constexpr bool gelu = EPI == Epi::kBiasGelu || EPI == Epi::kGeluGrad;
  return launch_lds<AT, BT, EPI>(a, s, choose_tile(a.M, a.N, a.K, gemm_layout(AT, BT, gelu)));
}

}  // namespace

namespace {

// Sum of the fp32 partials [S][M][N] in split order, then the epilogue of
// the unsplit kernel: bias, residual, GELU (writing u and g) or GELU' (from
// the saved u in R), rounded once to bf16.  Eight outputs per thread and
// iteration (N is a multiple of 8).
template <Epi EPI>
__global__ __launch_bounds__(256) void splitk_epilogue_kernel(const float *__restrict__ part, int splits,
                                                              size_t stride, int M, int N,
                                                              const bf16_t *__restrict__ bias,
                                                              const bf16_t *__restrict__ R, bf16_t *__restrict__ Y,
                                                              bf16_t *__restrict__ Y2) {
  const long n8 = static_cast<long>(M) * N / 8;
  for (long i = blockIdx.x * 256L + threadIdx.x; i < n8; i += static_cast<long>(gridDim.x) * 256) {
    const size_t e0 = static_cast<size_t>(i) * 8;
    f32x4_t lo = *reinterpret_cast<const f32x4_t *>(part + e0);
    f32x4_t hi = *reinterpret_cast<const f32x4_t *>(part + e0 + 4);
    for (int sp = 1; sp < splits; ++sp) {
      lo += *reinterpret_cast<const f32x4_t *>(part + sp * stride + e0);
      hi += *reinterpret_cast<const f32x4_t *>(part + sp * stride + e0 + 4);
    }
    float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    if constexpr (EPI == Epi::kBias || EPI == Epi::kBiasResid || EPI == Epi::kBiasGelu) {
      const u32x4_t bw = ldg16(bias + e0 % N);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[2 * e] += lo_bf(bw[e]);
        v[2 * e + 1] += hi_bf(bw[e]);
      }
    }
    if constexpr (EPI == Epi::kBiasResid || EPI == Epi::kResid) {
      const u32x4_t rw = ldg16(R + e0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[2 * e] += lo_bf(rw[e]);
        v[2 * e + 1] += hi_bf(rw[e]);
      }
    }
    if constexpr (EPI == Epi::kGeluGrad) {
      const u32x4_t uw = ldg16(R + e0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[2 * e] *= gelu_grad_f(lo_bf(uw[e]));
        v[2 * e + 1] *= gelu_grad_f(hi_bf(uw[e]));
      }
    }
    u32x4_t o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = pack2(v[2 * e], v[2 * e + 1]);
    stg16_nt(Y + e0, o);
    if constexpr (EPI == Epi::kBiasGelu) {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = pack2(gelu_f(v[2 * e]), gelu_f(v[2 * e + 1]));
      stg16_nt(Y2 + e0, o);
    }
  }
}

// Split launch of a forward (AT = false, BT = false) or input-gradient
// (BT = true) product: fp32 partials into ws, then the epilogue kernel.
// Returns false (nothing launched) when the plan does not split or ws is
// missing or too small.
template <bool BT, Epi EPI>
bool launch_split(const GemmArgs &a, void *ws, size_t ws_bytes, hipStream_t s) {
  const SplitPlan sp = gemm_split_plan(a.M, a.N, a.K);
  if (sp.splits <= 1 || ws == nullptr || ws_bytes < gemm_ws_bytes(a.M, a.N, a.K) || a.ldy != a.N || a.N % 8)
    return false;
  GemmArgs b = a;
  b.splits = sp.splits;
  b.k_chunk = sp.k_chunk;
  b.split_stride = static_cast<size_t>(a.M) * a.N;
  b.Wf = static_cast<float *>(ws);
  b.db = nullptr;
  b.accumulate = 0;
  if (!launch_lds<false, BT, Epi::kF32>(b, s, sp.tile)) return false;
  const long n8 = static_cast<long>(a.M) * a.N / 8;
  const int blocks = static_cast<int>(std::min<long>((n8 + 255) / 256, 2048));
  hipLaunchKernelGGL((splitk_epilogue_kernel<EPI>), dim3(blocks), dim3(256), 0, s, b.Wf, sp.splits, b.split_stride,
                     a.M, a.N, a.bias, a.R, a.Y, a.Y2);
  return true;
}

template <Epi EPI>
bool fwd_any(const GemmArgs &a, void *ws, size_t ws_bytes, hipStream_t s) {
  return launch_split<false, EPI>(a, ws, ws_bytes, s) || launch_lds<false, false, EPI>(a, s) ||
         launch_any<false, false, EPI>(a, s);
}

template <Epi EPI>
bool dgrad_any(const GemmArgs &a, void *ws, size_t ws_bytes, hipStream_t s) {
  return launch_split<true, EPI>(a, ws, ws_bytes, s) || launch_lds<false, true, EPI>(a, s) ||
         launch_any<false, true, EPI>(a, s);
}

}  // namespace

bool launch_gemm_fwd(const GemmArgs &a, Epi epi, void *ws, size_t ws_bytes, hipStream_t s) {
  switch (epi) {
    case Epi::kBias: return fwd_any<Epi::kBias>(a, ws, ws_bytes, s);
    case Epi::kBiasResid: return fwd_any<Epi::kBiasResid>(a, ws, ws_bytes, s);
    case Epi::kBiasGelu: return fwd_any<Epi::kBiasGelu>(a, ws, ws_bytes, s);
    case Epi::kPlain: return fwd_any<Epi::kPlain>(a, ws, ws_bytes, s);
    default: return false;
  }
}

bool launch_gemm_dgrad(const GemmArgs &a, Epi epi, void *ws, size_t ws_bytes, hipStream_t s) {
  switch (epi) {
    case Epi::kPlain: return dgrad_any<Epi::kPlain>(a, ws, ws_bytes, s);
    case Epi::kGeluGrad: return dgrad_any<Epi::kGeluGrad>(a, ws, ws_bytes, s);
    case Epi::kResid: return dgrad_any<Epi::kResid>(a, ws, ws_bytes, s);
    default: return false;
  }
}

namespace {

// The split sum of dW (blockIdx.y 0) or db (1), over n4 float4s.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(float *__restrict__ w, const float *__restrict__ wp,
                                                            long w4, float *__restrict__ b,
                                                            const float *__restrict__ bp, long b4, int splits,
                                                            int accumulate) {
  float *out = blockIdx.y == 0 ? w : b;
  const float *part = blockIdx.y == 0 ? wp : bp;
  const long n4 = blockIdx.y == 0 ? w4 : b4;
  for (long i = blockIdx.x * 256L + threadIdx.x; i < n4; i += static_cast<long>(gridDim.x) * 256)
    split_sum_at(i, n4, out, part, splits, accumulate);
}

}  // namespace

bool launch_gemm_wgrad(const GemmArgs &a, void *ws, size_t ws_bytes, hipStream_t s, FinishJobs *defer) {
  // both paths fuse the bias gradient into the weight-gradient kernel
  const SplitPlan sp = wgrad_split_plan(a.M, a.N, a.K);
  if (sp.splits > 1 && ws != nullptr && ws_bytes >= gemm_wgrad_ws_bytes(a.M, a.N, a.K) && a.ldy == a.N &&
      a.M % 4 == 0 && a.N % 4 == 0) {
    GemmArgs b = a;
    b.splits = sp.splits;
    b.k_chunk = sp.k_chunk;
    b.split_stride = static_cast<size_t>(a.M) * a.N;
    b.Wf = static_cast<float *>(ws);
    b.db = a.db ? b.Wf + ws_round256(static_cast<size_t>(sp.splits) * a.M * a.N * sizeof(float)) / sizeof(float)
                : nullptr;
    b.accumulate = 0;
    if (launch_lds<true, true, Epi::kF32>(b, s, sp.tile)) {
      const long w4 = static_cast<long>(a.M) * a.N / 4, b4 = a.db ? a.M / 4 : 0;
      if (defer)
        return defer->add_split(a.Wf, b.Wf, w4, sp.splits, a.accumulate) &&
               (!a.db || defer->add_split(a.db, b.db, b4, sp.splits, a.accumulate));
      const int blocks = static_cast<int>(std::min<long>((w4 + 255) / 256, 2048));
      hipLaunchKernelGGL(splitk_reduce_kernel, dim3(blocks, a.db ? 2 : 1), dim3(256), 0, s, a.Wf, b.Wf, w4, a.db,
                         b.db, b4, sp.splits, a.accumulate);
      return true;
    }
  }
  return launch_lds<true, true, Epi::kF32>(a, s) || launch_any<true, true, Epi::kF32>(a, s);
}

}  // namespace optimus
