// The 256-thread kernels of solve_kernels_256.hip with their matrices streamed past
// the caches (non-temporal loads of the entries), which leaves the L2 to the gathered
// vectors.  It pays once those outgrow the L2 well (api.cpp, streamed_matrices, has
// the line); for smaller QPs the matrices are better kept in the last-level cache.
#define PDHCG_BLOCK_SIZE 256
#define PDHCG_STREAMED 1
#include "solver.hpp"

namespace pdhcg {

__global__ void __launch_bounds__(kSolveBlock) pdhcg_solve_kernel_wg256_streamed(const SolveParams* __restrict__ Pg) {
  solve_body(Pg);
}

__global__ void __launch_bounds__(kSolveBlock) pdhcg_power_kernel_wg256_streamed(PowerParams P) { power_body(P); }

const void* solve_kernel_256_streamed() { return (const void*)pdhcg_solve_kernel_wg256_streamed; }
const void* power_kernel_256_streamed() { return (const void*)pdhcg_power_kernel_wg256_streamed; }

}  // namespace pdhcg
