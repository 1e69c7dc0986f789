// Reference kernels for the measured ceilings: an MFMA-only loop and a
// device copy (see enc_calib_mfma / enc_calib_copy).
#include "common.hpp"
#include "kernels.hpp"

namespace optimus {

namespace {

// Every wave: iters x 32 16x16x32 bf16 MFMAs (the instruction of the GEMMs'
// loops), two into each of 16 accumulators.  Operands are bf16 pairs in [1, 2) (exponent fixed, so no
// overflow) whose mantissa bits are re-drawn every iteration: a matrix core fed
// constant operands switches less and runs at a higher clock than one fed real
// data.
constexpr int kCalibFrags = 16;

__global__ __launch_bounds__(256, 4) void calib_mfma_kernel(int iters, float *__restrict__ out) {
  const uint32_t t = blockIdx.x * 256 + threadIdx.x;
  u32x4_t ua, ub;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    ua[e] = 0x3F803F80u ^ ((t * 0x9E3779B9u + e * 0x85EBCA6Bu) & 0x007F007Fu);
    ub[e] = 0x3F803F80u ^ ((t * 0xC2B2AE35u + e * 0x27D4EB2Fu) & 0x007F007Fu);
  }
  f32x4_t acc[kCalibFrags];
#pragma unroll
  for (int i = 0; i < kCalibFrags; ++i) acc[i] = f32x4_t{};
  for (int it = 0; it < iters; ++it) {
    const uint32_t m = (static_cast<uint32_t>(it) * 0x9E3779B9u) & 0x007F007Fu;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      ua[e] ^= m;
      ub[e] ^= (m << 1) & 0x007F007Fu;
    }
    const bf16x8_t a = as_bf16x8(ua), b = as_bf16x8(ub);
#pragma unroll
    for (int i = 0; i < 2 * kCalibFrags; ++i) acc[i % kCalibFrags] = mfma16(a, b, acc[i % kCalibFrags]);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < kCalibFrags; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) s += acc[i][e];
  out[t] = s;
}

// Grid-stride copy: eight independent 16-byte loads in flight per thread,
// non-temporal so that the stream does not evict the caches' contents.
constexpr int kCopyUnroll = 8;

__global__ __launch_bounds__(256) void calib_copy_kernel(const u32x4_t *__restrict__ src, u32x4_t *__restrict__ dst,
                                                         size_t n) {
  const size_t stride = static_cast<size_t>(gridDim.x) * 256;
  size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
  for (; i + (kCopyUnroll - 1) * stride < n; i += kCopyUnroll * stride) {
    u32x4_t v[kCopyUnroll];
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) v[u] = __builtin_nontemporal_load(src + i + u * stride);
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) __builtin_nontemporal_store(v[u], dst + i + u * stride);
  }
  for (; i < n; i += stride) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

}  // namespace

bool launch_calib_mfma(int blocks, int iters, float *out, hipStream_t s) {
  hipLaunchKernelGGL(calib_mfma_kernel, dim3(blocks), dim3(256), 0, s, iters, out);
  return true;
}

bool launch_calib_copy(const void *src, void *dst, size_t bytes, hipStream_t s) {
  const size_t n = bytes / 16;
  const size_t want = (n + kCopyUnroll * 256 - 1) / (kCopyUnroll * 256);
  const int blocks = static_cast<int>(want < 4096 ? (want > 0 ? want : 1) : 4096);
  hipLaunchKernelGGL(calib_copy_kernel, dim3(blocks), dim3(256), 0, s, static_cast<const u32x4_t *>(src),
                     static_cast<u32x4_t *>(dst), n);
  return true;
}

}  // namespace optimus
