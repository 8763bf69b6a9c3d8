// The batched kernel with teams of workgroups, 256 threads each, for batches that
// hold dense or factored Q; batch_kernels_sparse_team.hip is its form for sparse
// ones.  They are kernels of their own because the others know at compile time
// that an instance has one workgroup (half the code; 3 % of the time of 600 MPC
// QPs).  When they run and what they gain stands at team_sizes (api.cpp).
#define PDHCG_BLOCK_SIZE 256
#include "solver.hpp"

namespace pdhcg {

__global__ void __launch_bounds__(kSolveBlock) pdhcg_batch_kernel_team(BatchParams BP) { batch_team_solve<true>(BP); }

const void* batch_kernel_sparse_team();

static const void* team_kernel(bool dense) {
  return dense ? (const void*)pdhcg_batch_kernel_team : batch_kernel_sparse_team();
}

hipError_t launch_batch_teams(bool dense, const BatchParams& p, int grid, hipStream_t s) {
  BatchParams pc = p;
  void* args[] = {&pc};
  return hipLaunchCooperativeKernel(team_kernel(dense), dim3(grid), dim3(kBlock), args, 0, s);
}

hipError_t batch_resident(bool dense, int* grid, int* cus) {
  int dev = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, team_kernel(dense), kBlock, 0);
  *grid = e == hipSuccess ? *cus * per_cu : 0;
  return e;
}

}  // namespace pdhcg
