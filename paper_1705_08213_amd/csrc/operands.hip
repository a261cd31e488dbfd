// operands.hip -- the pre-pass of the one-shot fp4 MFMA kernels (layout and
// device code in operands.h).
#include "operands.h"

namespace ccc {

namespace {

// One workgroup per block of 16 rows and share of the fields.
__global__ __launch_bounds__(1024) void operands_kernel(OperandJob job, int64_t base) {
  const int64_t b = base + blockIdx.x;
  if (job.zero && b == 0 && threadIdx.x == 0) *job.zero = 0ull;
  const bool second = b >= job.set[0].blocks;
  const OperandSet& s = job.set[second ? 1 : 0];
  const int64_t block = b - (second ? job.set[0].blocks : 0);
  __shared__ int part[16][16][2];
  if (block >= s.first)  // uniform
    operand_block<true>(job, s, block, blockIdx.y, part);
  else
    operand_block<false>(job, s, block, blockIdx.y, part);
}

// The counts of a pass in several shares.
__global__ __launch_bounds__(64) void share_counts_kernel(OperandJob job) {
  const int64_t r = (int64_t)blockIdx.x * 64 + threadIdx.x, n = job.set[0].n;
  if (r >= n) return;
  int a = 0, m = 0;
  for (int k = 0; k < job.shares; ++k) {
    const int2 x = job.part[k * n + r];
    a += x.x;
    m += x.y;
  }
  put_counts(job, job.set[0], r, a, m);
}

}  // namespace

hipError_t launch_operands(OperandJob job, hipStream_t stream) {
  if (job.shares < 1 || !job.part || job.set[1].blocks) job.shares = 1;
  const int64_t blocks = (int64_t)job.set[0].blocks + job.set[1].blocks;
  if (blocks <= 0) return hipSuccess;
  // a wave per super-step up to sixteen: few blocks leave the chip idle
  const int waves = job.steps > 8 ? 16 : 4;
  timing_begin("count1", stream);
  hipError_t e = launch_slices(blocks, 64 * waves, [&](int64_t base, dim3 grid) {
    grid.y = (unsigned)job.shares;
    hipLaunchKernelGGL(operands_kernel, grid, dim3(64 * waves), 0, stream, job, base);
  });
  if (e == hipSuccess && job.shares > 1) {
    hipLaunchKernelGGL(share_counts_kernel, dim3((unsigned)((job.set[0].n + 63) / 64)), dim3(64), 0,
                       stream, job);
    e = hipGetLastError();
  }
  timing_end(stream);
  return e;
}

}  // namespace ccc
