// The batched kernel with teams of workgroups for batches without a dense or
// factored Q (batch_kernels_team.hip), at the registers of
// batch_kernels_sparse.hip.
#define PDHCG_BLOCK_SIZE 256
#include "solver.hpp"

namespace pdhcg {

__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3)))
pdhcg_batch_kernel_sparse_team(BatchParams BP) {
  batch_team_solve<false>(BP);
}

const void* batch_kernel_sparse_team() { return (const void*)pdhcg_batch_kernel_sparse_team; }

}  // namespace pdhcg
