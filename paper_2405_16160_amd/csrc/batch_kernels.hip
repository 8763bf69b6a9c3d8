// The batched kernel: many independent QPs in one launch, one workgroup per QP
// (the same restarted PDHCG loop as the cooperative kernel, Alg. 1 with the
// rules of Sec. 4; the loop itself is batch_solve in solver.hpp).  This
// translation unit compiles the shared device code for workgroups of 256
// threads, the default: two instances then share a CU, so the fixed latency
// of a small instance's iteration (a few dependent memory round trips per
// phase, tens of microseconds in all) is overlapped with another instance's
// work.  batch_kernels_512.hip holds the same kernel at 512 threads.
#define PDHCG_BLOCK_SIZE 256
#include "solver.hpp"

namespace pdhcg {

// Launched with kBlock threads but declared for 512: that bound holds the
// kernel and every function it calls to two waves per SIMD (256 registers),
// the budget at which two workgroups fit on a CU; with the bound of the
// launch size alone the compiler takes the whole register file.
__global__ void __launch_bounds__(kSolveBlock) pdhcg_batch_kernel(BatchParams BP) { batch_solve<true>(BP); }

__global__ void batch_clock_kernel(uint64_t* t0, uint64_t* bars, int64_t nbars, uint32_t* queue, uint32_t first,
                                   double* norm) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0 && t0) *t0 = wall_clock64();
  if (i == 0 && queue) *queue = first;
  if (i == 0 && norm) *norm = -1.0;
  for (int64_t k = i; k < nbars; k += (int64_t)gridDim.x * blockDim.x) bars[k] = 0;
}

hipError_t launch_batch_clock(uint64_t* t0, uint64_t* bars, int64_t nbars, uint32_t* queue, uint32_t first,
                              double* norm, hipStream_t s) {
  const int grid = nbars > 0 ? (int)((nbars + 255) / 256 < 256 ? (nbars + 255) / 256 : 256) : 1;
  hipLaunchKernelGGL(batch_clock_kernel, dim3(grid), dim3(256), 0, s, t0, bars, nbars, queue, first, norm);
  return hipGetLastError();
}

hipError_t launch_batch_256(const BatchParams& p, int count, hipStream_t s) {
  hipLaunchKernelGGL(pdhcg_batch_kernel, dim3(count), dim3(kBlock), 0, s, p);
  return hipGetLastError();
}

}  // namespace pdhcg
