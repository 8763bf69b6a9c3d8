// Host stand-in for the HIP runtime header, used only by the CPU tests: the
// library's own sources compiled for the host, every lane of a workgroup a fiber
// (simt.cpp).  What waits for other lanes, waves or workgroups on the device ends
// the lane's turn here, so the order in which waves and workgroups run is the
// scheduler's choice and a missing barrier shows the same way on every run.
#pragma once
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>
#include <hip/hip_vector_types.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <functional>

#undef __device__
#undef __host__
#undef __global__
#undef __shared__
#undef __forceinline__
#undef __launch_bounds__
#undef __align__
#define __device__
#define __host__
#define __global__
#define __shared__ static thread_local  // one workgroup per thread at a time
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))

namespace simt {
struct Index {
  unsigned x, y, z;
};
extern thread_local Index lane_index, block_index, grid_dim, block_dim;
enum Kind { kDpp, kReadLane, kBallot, kShflXor, kWaveBarrier };
uint64_t collective(Kind kind, uint64_t v, int a, int b);
void sync_threads();
void yield_block();
uint64_t clock_ticks();
uint32_t xcd();
char* dynamic_lds();
hipError_t launch(dim3 grid, dim3 block, const std::function<void()>& body);
}  // namespace simt

#define threadIdx simt::lane_index
#define blockIdx simt::block_index
#define gridDim simt::grid_dim
#define blockDim simt::block_dim
#define hipLaunchKernelGGL(k, g, b, lds, stream, ...) (void)simt::launch((g), (b), [&] { (k)(__VA_ARGS__); })
#undef HIP_SYMBOL
#define HIP_SYMBOL(x) (x)

#define __syncthreads() simt::sync_threads()
#define wall_clock64() simt::clock_ticks()
#undef __HIP_MEMORY_SCOPE_AGENT
#undef __HIP_MEMORY_SCOPE_WORKGROUP
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __hip_atomic_load(p, o, s) __atomic_load_n((p), __ATOMIC_SEQ_CST)
#define __hip_atomic_store(p, v, o, s) __atomic_store_n((p), (v), __ATOMIC_SEQ_CST)
#define __hip_atomic_fetch_add(p, v, o, s) __atomic_fetch_add((p), (v), __ATOMIC_SEQ_CST)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_s_sleep(n) simt::yield_block()
#define __builtin_amdgcn_wave_barrier() ((void)simt::collective(simt::kWaveBarrier, 0, 0, 0))
// (the sources apply it to values that are equal in all lanes only)
#define __builtin_amdgcn_readfirstlane(v) ((int)(v))
#define __builtin_amdgcn_readlane(v, lane) ((int)simt::collective(simt::kReadLane, (uint32_t)(v), (lane), 0))
#define __builtin_amdgcn_update_dpp(old, v, ctrl, rows, banks, bound) \
  ((int)simt::collective(simt::kDpp, (uint32_t)(v), (ctrl), (rows)))
#define __ballot(p) simt::collective(simt::kBallot, (p) ? 1 : 0, 0, 0)

inline double simt_double(uint64_t b) {
  double d;
  memcpy(&d, &b, 8);
  return d;
}
inline uint64_t simt_bits(double d) {
  uint64_t b;
  memcpy(&b, &d, 8);
  return b;
}
inline double __shfl_xor(double v, int off, int width) {
  return simt_double(simt::collective(simt::kShflXor, simt_bits(v), off, width));
}
inline int __double2loint(double v) { return (int)(uint32_t)simt_bits(v); }
inline int __double2hiint(double v) { return (int)(uint32_t)(simt_bits(v) >> 32); }
inline double __hiloint2double(int hi, int lo) { return simt_double((uint64_t)(uint32_t)hi << 32 | (uint32_t)lo); }
inline long long __double_as_longlong(double v) { return (long long)simt_bits(v); }
inline int __clz(int v) { return v ? __builtin_clz((unsigned)v) : 32; }
inline int atomicAdd(int* p, int v) { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
using std::max;
using std::min;
