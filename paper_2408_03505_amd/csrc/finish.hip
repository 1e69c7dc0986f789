// The last launch of a layer's backward: every pending fixed-order reduction
// of the layer in one grid (LayerNorm scales and biases, split weight and bias
// gradients).  Each is a few microseconds of memory traffic, and launched one
// by one each paid its own launch and its own ramp at the end.
#include "kernels.hpp"
#include "reduce.hpp"

namespace optimus {

namespace {

__global__ __launch_bounds__(256) void finish_kernel(FinishJobs jobs) {
  __shared__ float red[kRedGroups][kRedCols + 1];
  int j = 0;
  while (j + 1 < jobs.n && static_cast<int>(blockIdx.x) >= jobs.job[j + 1].first_block) ++j;
  const FinishJob &job = jobs.job[j];
  const int b = static_cast<int>(blockIdx.x) - job.first_block;
  if (job.cols > 0) {
    column_sum_block(b, job.parts, job.cols, job.part, job.out, job.accumulate, red);
  } else {
    const long i = b * 256L + threadIdx.x;
    if (i < job.n4) split_sum_at(i, job.n4, job.out, job.part, job.parts, job.accumulate);
  }
}

}  // namespace

bool FinishJobs::add_split(float *out, const float *part, long n4, int splits, int accumulate) {
  if (n >= kMax) return false;
  job[n++] = {out, part, n4, splits, 0, accumulate, blocks};
  blocks += static_cast<int>((n4 + 255) / 256);
  return true;
}

bool FinishJobs::add_columns(float *out, const float *part, int rows, int cols, int accumulate) {
  if (n >= kMax) return false;
  job[n++] = {out, part, 0, rows, cols, accumulate, blocks};
  blocks += (cols + kRedCols - 1) / kRedCols;
  return true;
}

bool launch_finish(const FinishJobs &jobs, hipStream_t s) {
  if (jobs.n > 0) hipLaunchKernelGGL(finish_kernel, dim3(jobs.blocks), dim3(256), 0, s, jobs);
  return true;
}

}  // namespace optimus
