// The batched kernel of 256 threads for batches without a dense or factored Q.
// Its phases are chains of memory round trips, so what counts is how many waves
// a CU has to switch between.  The dense products of batch_kernels.hip take 248
// registers; without them nothing needs more than 168, and three workgroups fit
// on a CU instead of two (the chunk of LDS that stages a dense operand goes
// too).  600 linear-MPC members, T = 50 (n = 1500, m = 5000, FP64, to 1e-4):
// 233 ms at two waves per SIMD, 172 at three, 174 at four (128 registers, where
// the phases spill).
#define PDHCG_BLOCK_SIZE 256
#include "solver.hpp"

namespace pdhcg {

__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3)))
pdhcg_batch_kernel_sparse(BatchParams BP) {
  batch_solve<false>(BP);
}

hipError_t launch_batch_sparse(const BatchParams& p, int count, hipStream_t s) {
  hipLaunchKernelGGL(pdhcg_batch_kernel_sparse, dim3(count), dim3(kBlock), 0, s, p);
  return hipGetLastError();
}

}  // namespace pdhcg
