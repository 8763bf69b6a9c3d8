// Device building blocks: NaN-propagating max, wavefront/workgroup
// reductions, a grid barrier for cooperative launches, and the row-split CSR
// row reduction used by every sparse product of the solver.
#pragma once
#include <type_traits>

#include "internal.hpp"

namespace pdhcg {
// internal linkage: the workgroup size (kBlock) differs between the
// translation units that include this header
namespace {

// max of two values that are >= +0 or NaN, propagating NaN (the hardware max
// returns the non-NaN operand, which would hide a diverged iterate from the
// termination test).  As unsigned integers the bit patterns of such doubles
// are in the order of their values with every NaN above infinity, so one
// 64-bit integer compare decides; the FP64 form of this test (two compares for
// NaN, a compare, an add) made the maxima of a phase its largest cost: an
// n-side phase of the n = 1000 QP 7.1 us with it.
__device__ __forceinline__ double maxp(double a, double b) {
  return (uint64_t)__double_as_longlong(a) > (uint64_t)__double_as_longlong(b) ? a : b;
}

// A value that every lane of the wave holds equal, marked as such for the
// compiler (it then keeps it in scalar registers instead of 64 vector lanes,
// which matters for the solver's scalar state that stays live across phases).
__device__ __forceinline__ double uniform(double v) {
  const int lo = __builtin_amdgcn_readfirstlane(__double2loint(v));
  const int hi = __builtin_amdgcn_readfirstlane(__double2hiint(v));
  return __hiloint2double(hi, lo);
}

// Data-parallel-primitive (DPP) lane moves of a double: each half moves with
// v_mov_b32_dpp inside the VALU, far cheaper than a shuffle through the LDS
// crossbar.  Lanes whose source lies outside the row, or whose row is masked
// off, read +0.0.
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ double dpp(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROW_MASK, 0xF, true);
  return __hiloint2double(hi, lo);
}

// Reduction over aligned groups of G lanes (G a power of two <= 64) with the
// result in the group's last lane (lane G-1 of each group): row shifts by 1,
// 2, 4, 8 make lane i hold the combination of lanes i-2^s+1 .. i of its row;
// row_bcast15 / row_bcast31 then carry row totals across the rows of a wave.
// op must have +0.0 as identity on its inputs (sums; maxima of values >= 0).
template <typename Op>
__device__ __forceinline__ double group_reduce_last(double v, int G, Op op) {
  if (G >= 2) v = op(v, dpp<0x111>(v));       // row_shr:1
  if (G >= 4) v = op(v, dpp<0x112>(v));       // row_shr:2
  if (G >= 8) v = op(v, dpp<0x114>(v));       // row_shr:4
  if (G >= 16) v = op(v, dpp<0x118>(v));      // row_shr:8
  if (G >= 32) v = op(v, dpp<0x142, 0xA>(v));  // row_bcast:15 into rows 1 and 3
  if (G >= 64) v = op(v, dpp<0x143, 0xC>(v));  // row_bcast:31 into rows 2 and 3
  return v;
}

struct AddOp {
  __device__ __forceinline__ double operator()(double a, double b) const { return a + b; }
};
struct MaxOp {
  __device__ __forceinline__ double operator()(double a, double b) const { return maxp(a, b); }
};

// sum over the aligned group of G lanes, valid in the group's last lane
__device__ __forceinline__ double group_sum_last(double v, int G) { return group_reduce_last(v, G, AddOp{}); }

// N such sums, the steps of one in the shadow of the others'
template <int N>
__device__ __forceinline__ void group_sums_last(double* v, int G) {
  auto step = [&](auto move) {
    double t[N];
#pragma unroll
    for (int j = 0; j < N; ++j) t[j] = move(v[j]);
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] += t[j];
  };
  if (G >= 2) step([](double x) { return dpp<0x111>(x); });
  if (G >= 4) step([](double x) { return dpp<0x112>(x); });
  if (G >= 8) step([](double x) { return dpp<0x114>(x); });
  if (G >= 16) step([](double x) { return dpp<0x118>(x); });
  if (G >= 32) step([](double x) { return dpp<0x142, 0xA>(x); });
  if (G >= 64) step([](double x) { return dpp<0x143, 0xC>(x); });
}

// Workgroup reduction of NS sums and NM maxima at once.  Every thread ends
// with the results; the combination order is fixed, so equal inputs give
// bit-equal outputs in every workgroup.  lds must hold kWaves*(NS+NM) doubles.
template <int NS, int NM>
__device__ __forceinline__ void block_reduce(double* s, double* mx, double* lds) {
  constexpr int W = NS + NM;
#pragma unroll
  for (int k = 0; k < NS; ++k) s[k] = group_reduce_last(s[k], kWave, AddOp{});
#pragma unroll
  for (int k = 0; k < NM; ++k) mx[k] = group_reduce_last(mx[k], kWave, MaxOp{});
  const int w = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == kWave - 1) {
#pragma unroll
    for (int k = 0; k < NS; ++k) lds[w * W + k] = s[k];
#pragma unroll
    for (int k = 0; k < NM; ++k) lds[w * W + NS + k] = mx[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    double a = lds[k];
    for (int j = 1; j < kWaves; ++j) a += lds[j * W + k];
    s[k] = uniform(a);
  }
#pragma unroll
  for (int k = 0; k < NM; ++k) {
    double a = lds[NS + k];
    for (int j = 1; j < kWaves; ++j) a = maxp(a, lds[j * W + NS + k]);
    mx[k] = uniform(a);
  }
  __syncthreads();
}

// The workgroup's partial results of a phase: NS sums and NM maxima reduced
// over the workgroup and stored as its partials part[slot(k) * nb + b], sums
// first.  Only the stored values are needed, so the combination over the waves
// is done by one lane per value (the waves' results side by side in LDS, read
// once for all values), not by every thread for every value.  There is no barrier
// behind that read: the one of the grid barrier that ends a phase serves, and a
// phase that uses lds again before it has to synchronise first.  lds holds
// kWaves * (NS + NM) doubles.
template <int NS, int NM, typename Slot>
__device__ __forceinline__ void store_partials(double* s, double* mx, const Slot& slot, double* part, int nb, int b,
                                               double* lds) {
  constexpr int W = NS + NM;
#pragma unroll
  for (int k = 0; k < NS; ++k) s[k] = group_reduce_last(s[k], kWave, AddOp{});
#pragma unroll
  for (int k = 0; k < NM; ++k) mx[k] = group_reduce_last(mx[k], kWave, MaxOp{});
  const int w = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == kWave - 1) {
#pragma unroll
    for (int k = 0; k < NS; ++k) lds[w * W + k] = s[k];
#pragma unroll
    for (int k = 0; k < NM; ++k) lds[w * W + NS + k] = mx[k];
  }
  __syncthreads();
  if (threadIdx.x < W) {
    const int k = (int)threadIdx.x;
    double v[kWaves];
#pragma unroll
    for (int j = 0; j < kWaves; ++j) v[j] = lds[j * W + k];
    double a = v[0], m = v[0];
#pragma unroll
    for (int j = 1; j < kWaves; ++j) {
      a += v[j];
      m = maxp(m, v[j]);
    }
    part[slot(k) * nb + b] = k < NS ? a : m;
  }
}

// N slots' partials part[j][0 .. nb), each lane combining those of its own index
// modulo the wave (a fixed order); the loads of all N are issued first, and only
// one value per slot is left to move between the lanes.
template <int N, typename Op>
__device__ __forceinline__ void lane_partials(const double* const* part, int nb, const Op& op, double* a) {
  constexpr int U = 4;
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
  for (int k = 0; k < N; ++k) a[k] = 0.0;
  for (int j0 = 0; j0 < nb; j0 += U * kWave) {
    double v[N][U];
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = j0 + u * kWave + lane;
        v[k][u] = j < nb ? part[k][j] : 0.0;
      }
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int u = 0; u < U; ++u) a[k] = op(k, a[k], v[k][u]);
  }
}

// the value that a lane of the wave holds, for every lane
__device__ __forceinline__ double lane_value(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// NS sums of the per-workgroup partials part[slot * nb + j], j < nb, for every
// thread: each wave combines them itself from the partials (a few loads and
// lane moves, no exchange through LDS and no workgroup barrier; at most four
// values), in the same order in every wave and workgroup.
template <int... SLOTS>
__device__ __forceinline__ void reduce_sums(const double* part, int nb, double* s) {
  constexpr int NS = sizeof...(SLOTS);
  constexpr int slots[NS] = {SLOTS...};
  if (nb == 1) {  // one workgroup: its own partial is the total
#pragma unroll
    for (int k = 0; k < NS; ++k) s[k] = part[slots[k]];
    return;
  }
  const double* p[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k) p[k] = part + slots[k] * nb;
  lane_partials<NS>(p, nb, [](int, double x, double y) { return x + y; }, s);
  group_sums_last<NS>(s, kWave);
#pragma unroll
  for (int k = 0; k < NS; ++k) s[k] = lane_value(s[k], kWave - 1);
}

// NS sums and NM maxima of the partials into out[0 .. NS + NM) (LDS), sums
// first: the waves of the workgroup take two values each in turn, in one loop
// (the ten values of relKKT unrolled were 13 KB of code).  The caller
// synchronises the workgroup before reading out.  With 256 workgroups, lanes moved
// per 64 partials and one value after the other took 5.1 us, this takes 3.5 (n = 1e5
// QP, 60 iterations: 3.57 -> 3.34 ms; MPC QP re-solved: 11.63 -> 11.08).
template <int NS, int NM, typename Slot>
__device__ __forceinline__ void reduce_to_lds(const double* part, int nb, const Slot& slot, double* out) {
  constexpr int N = NS + NM;
  if (nb == 1) {
    if (threadIdx.x < N) out[threadIdx.x] = part[slot((int)threadIdx.x)];
    return;
  }
  for (int k = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave); k < N; k += 2 * kWaves) {
    const int k2 = k + kWaves < N ? k + kWaves : k;
    const double* const p[2] = {part + (int64_t)slot(k) * nb, part + (int64_t)slot(k2) * nb};
    const bool sum[2] = {k < NS, k2 < NS};
    double a[2];
    lane_partials<2>(p, nb, [&](int j, double x, double y) { return sum[j] ? x + y : maxp(x, y); }, a);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      a[j] = sum[j] ? group_reduce_last(a[j], kWave, AddOp{}) : group_reduce_last(a[j], kWave, MaxOp{});
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) {
      out[k] = a[0];
      if (k2 != k) out[k2] = a[1];
    }
  }
}

// ------------------------------------------------------------ grid barrier
//
// Arrival is counted per XCD, in that XCD's L2: the CUs of one XCD share its
// L2, so a counter there needs no device-scope traffic.  Before arriving,
// every wave of the workgroup waits until its stores are complete (written to
// the L2); the last workgroup of an XCD to arrive then writes that L2 back to
// memory once, for the whole XCD, and arrives on the device-scope counter; the
// last XCD publishes the new generation, one copy per XCD on a line of its own.
// Waiters poll their XCD's copy with relaxed device-scope loads and take one
// acquire fence (invalidating their L1 and the XCD's L2).  The XCD of a workgroup is read from the hardware
// register that names it, and the number of the grid's workgroups on each XCD
// is counted once per launch (init), so the barrier holds for any placement of
// workgroups on XCDs.  Counters grow monotonically within a launch (64-bit),
// so no reset race exists.  Every wait is bounded by a wall-clock limit: on
// expiry the workgroup raises the abort word and returns false, and every
// other waiter then returns false too.
//
// When all of the barrier's workgroups are on one XCD (a team of a batch), its L2
// is all that they have to agree on: stores are there once they complete, so
// nothing is written back, and the counter is polled there; the acquire fence
// then drops the L1's lines.  Writing an L2 back that others are using costs
// more than the barrier: with 64 teams of 4 among 500 QPs, 10 us and 1.2 us.
namespace bar {
constexpr int kMaxXcd = 16;
constexpr int kCount = 0, kAbort = kBarAbortWord, kSetup = 96;  // word offsets (256 bytes apart)
constexpr int kXcdArrive = 128;                     // + 32 x: arrivals of XCD x (in its L2)
constexpr int kXcdCount = kXcdArrive + 32 * kMaxXcd;  // + 32 x: workgroups on XCD x
constexpr int kXcdGen = kXcdCount + 32 * kMaxXcd;     // + 32 x: the generation, one copy per XCD
constexpr int kWords = kXcdGen + 32 * kMaxXcd;
static_assert(kWords <= kBarWords, "barrier words");
}  // namespace bar

#define PDHCG_LD(p) __hip_atomic_load((p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
#define PDHCG_ST(p, v) __hip_atomic_store((p), (v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
#define PDHCG_ADD(p, v) __hip_atomic_fetch_add((p), (v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)

// the XCD (accelerator complex die) this wave runs on
__device__ __forceinline__ uint32_t xcd_id() {
  uint32_t v;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
  return v & (uint32_t)(bar::kMaxXcd - 1);
}

// wait until this wave's outstanding memory operations are complete (stores
// written to the L2)
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

struct GridSync {
  uint64_t* w;
  uint32_t nb;
  uint64_t epoch;
  uint32_t xcd = 0, xsize = 1, nxcd = 1;  // this workgroup's XCD, workgroups on it, XCDs in use
  static constexpr uint64_t kTimeoutTicks = 500000000ull;  // 5 s of the 100 MHz wall clock

  __device__ bool wait_word(int k, uint64_t target, int& ok) {
    const uint64_t t0 = wall_clock64();
    while (PDHCG_LD(&w[k]) < target) {
      if (PDHCG_LD(&w[bar::kAbort]) != 0ull) { ok = 0; return false; }
      if (wall_clock64() - t0 > kTimeoutTicks) {
        PDHCG_ST(&w[bar::kAbort], 1ull);
        ok = 0;
        return false;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    return true;
  }

  // the same for this XCD's arrival counter, read where it is counted (an atomic
  // that adds an opaque zero: it is not turned into a load, which the L1 could
  // answer)
  __device__ bool wait_arrivals(uint64_t target, int& ok) {
    const uint64_t t0 = wall_clock64();
    uint32_t zero = 0, polls = 0;
    asm volatile("" : "+v"(zero));
    while (__hip_atomic_fetch_add(&w[bar::kXcdArrive + 32 * xcd], (uint64_t)zero, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_WORKGROUP) < target) {
      __builtin_amdgcn_s_sleep(1);
      if ((++polls & 63u) != 0) continue;
      if (PDHCG_LD(&w[bar::kAbort]) != 0ull || wall_clock64() - t0 > kTimeoutTicks) {
        PDHCG_ST(&w[bar::kAbort], 1ull);
        ok = 0;
        return false;
      }
    }
    return true;
  }

  // Once per launch, before the first sync: count the workgroups per XCD.
  __device__ bool init() {
    __shared__ uint32_t sx[3];
    __shared__ int ok_s;
    if (threadIdx.x == 0) {
      int ok = 1;
      sx[0] = 0;
      sx[1] = 1;
      sx[2] = 1;
      if (nb > 1) {
        const uint32_t x = xcd_id();
        PDHCG_ADD(&w[bar::kXcdCount + 32 * x], 1ull);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        PDHCG_ADD(&w[bar::kSetup], 1ull);
        if (wait_word(bar::kSetup, nb, ok)) {
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
          uint32_t used = 0;
          for (int j = 0; j < bar::kMaxXcd; ++j) used += PDHCG_LD(&w[bar::kXcdCount + 32 * j]) > 0ull;
          sx[0] = x;
          sx[1] = (uint32_t)PDHCG_LD(&w[bar::kXcdCount + 32 * x]);
          sx[2] = used;
        }
      }
      ok_s = ok;
    }
    __syncthreads();
    xcd = sx[0];
    xsize = sx[1];
    nxcd = sx[2];
    return ok_s != 0;
  }

  __device__ bool sync() {
    __shared__ int ok_s;
    if (nb > 1) wait_stores();
    __syncthreads();
    ++epoch;
    if (threadIdx.x == 0) {
      int ok = 1;
      if (nb > 1) {
        const uint64_t a = __hip_atomic_fetch_add(&w[bar::kXcdArrive + 32 * xcd], 1ull, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_WORKGROUP);
        if (nxcd == 1) {
          wait_arrivals((uint64_t)xsize * epoch, ok);
        } else if (a == (uint64_t)xsize * epoch - 1) {  // last of its XCD: write the XCD's L2 back once
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
          const uint64_t t = PDHCG_ADD(&w[bar::kCount], 1ull);
          if (t == (uint64_t)nxcd * epoch - 1) {  // publish to every XCD's own line
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            for (int x = 0; x < bar::kMaxXcd; ++x) PDHCG_ST(&w[bar::kXcdGen + 32 * x], epoch);
          }
        }
        if (nxcd > 1) wait_word(bar::kXcdGen + 32 * xcd, epoch, ok);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      }
      ok_s = ok;
    }
    __syncthreads();
    return ok_s != 0;
  }
};

// ------------------------------------------------------- row-split products

// FP64 or FP32 matrix values, FP64 or FP32 gathered vectors; products are
// accumulated in FP64.

// Load through a global-address-space pointer (the solver's arrays all live
// in device memory; a generic pointer would make the compiler emit flat loads,
// which also count against the LDS counter and force wider waits).
template <typename T>
__device__ __forceinline__ T gld(const T* p) {
  return *(const __attribute__((address_space(1))) T*)p;
}

// The same with the non-temporal hint, for a matrix streamed once per
// product: its lines should not displace the reused vectors and index data
// (of this workgroup and of the others on the XCD) from the L2 and the MALL.
template <typename T>
__device__ __forceinline__ T gld_nt(const T* p) {
  return __builtin_nontemporal_load((const __attribute__((address_space(1))) T*)p);
}

// Four consecutive FP32 values from a 4-byte aligned address in one
// global_load_dwordx4 (gfx950 takes dword-aligned 16-byte accesses), plain
// or with the non-temporal hint.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ f32x4u gld4(const float* p) {
  return *(const __attribute__((address_space(1))) f32x4u*)p;
}
__device__ __forceinline__ f32x4u gld4_nt(const float* p) {
  return __builtin_nontemporal_load((const __attribute__((address_space(1))) f32x4u*)p);
}

// an (r, p) record of the textbook CG: one 8-byte load or store
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f32x2 gld2(const float2* p) {
  return *(const __attribute__((address_space(1))) f32x2*)p;
}
__device__ __forceinline__ void gst2(float2* p, float a, float b) {
  *(__attribute__((address_space(1))) f32x2*)p = f32x2{a, b};
}

template <typename T>
__device__ __forceinline__ void gst(T* p, T v) {
  *(__attribute__((address_space(1))) T*)p = v;
}

// float4 rows move as one 16-byte access (through the clang vector type: the
// HIP vector class has no constructors for address-space-qualified operands)
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <>
__device__ __forceinline__ float4 gld<float4>(const float4* p) {
  const f32x4 v = *(const __attribute__((address_space(1))) f32x4*)p;
  return make_float4(v.x, v.y, v.z, v.w);
}

template <>
__device__ __forceinline__ void gst<float4>(float4* p, float4 v) {
  f32x4 w;
  w.x = v.x;
  w.y = v.y;
  w.z = v.z;
  w.w = v.w;
  *(__attribute__((address_space(1))) f32x4*)p = w;
}

// sum_k M[i,k] * g(col[k]) for the entries [beg, end) of one row, computed by
// `width` lanes starting at lane `lane` (partial sums; reduced by the caller)
// Loads go in batches of 8 per lane, unconditional (indices clamped into the
// row): 8 index/value loads, then 8 gathers, instead of one dependent pair at
// a time.
template <typename V, typename Gather>
__device__ __forceinline__ double row_partial(const int32_t* col, const V* val, int beg, int end, int lane,
                                              int width, const Gather& g) {
  constexpr int U = 8;
  double s = 0.0;
  for (int base = beg + lane; base < end; base += U * width) {
    int c[U];
    V v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min(base + u * width, end - 1);
      c[u] = gld(col + k);
      v[u] = gld(val + k);
    }
    double gv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) gv[u] = g(c[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (base + u * width < end) s += (double)v[u] * gv[u];
  }
  return s;
}

template <typename T>
struct GatherVec {
  const T* v;
  __device__ __forceinline__ double operator()(int j) const { return (double)gld(v + j); }
};

// p_j = r_j + beta p_prev_j, formed at gather time (the CG direction update is
// folded into the next product, which saves a grid barrier per CG step)
template <typename T>
struct GatherDir {
  const T* r;
  const T* pp;
  double beta;
  int first;
  // both loads are unconditional (pp is always a valid buffer; when first is
  // set its contents are not used), so a tile's gathers issue together
  __device__ __forceinline__ double operator()(int j) const {
    const double rj = (double)gld(r + j), pj = (double)gld(pp + j);
    return first ? rj : rj + beta * pj;
  }
};

// The same from the interleaved FP32 records (r_j, p_prev_j): one 8-byte
// load, one cache line, per gathered entry
struct GatherDir2 {
  const float2* rp;
  double beta;
  int first;
  __device__ __forceinline__ double operator()(int j) const {
    const f32x2 w = gld2(rp + j);
    const double rj = (double)w.x, pj = (double)w.y;
    return first ? rj : rj + beta * pj;
  }
};

// ------------------------------------------------------------- wave tiles
//
// A sparse product is cut on the host into tiles of whole rows that one wave
// processes alone: at most kTileNnz entries (8 per lane) and kTileRows rows (one
// per lane), sized so that the waves of a workgroup get equal shares.  The wave
// loads the tile's row offsets, the rows' own inputs and its entries in one
// burst, gathers, parks the products in its own stretch of LDS and sums the
// rows from there.  A wave's LDS accesses complete in order, so no workgroup
// barrier is needed anywhere in a tile, and the waves drift apart: one gathers
// while another sums.  Bound by the latency of that chain (two dependent round
// trips, then LDS).  Against tiles of the whole workgroup (8 entries per thread
// always loaded, five workgroup barriers, descriptors by flat loads): n = 1000
// QP 8.2 -> 6.7 ms for 200 iterations, 600 MPC members in a batch 326 -> 233 ms,
// the low-rank QP n = 1e5 10.5 -> 8.4 ms for 60 iterations.

// the wave's number in the workgroup and lane, the former in a scalar register
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave); }
__device__ __forceinline__ int lane_id() { return (int)threadIdx.x & (kWave - 1); }

// element k of an array whose start is uniform over the wave and whose byte
// offset 8 k fits 32 bits (entries and rows of one tile): base in scalar
// registers, one 32-bit offset per lane
template <typename T>
__device__ __forceinline__ T gld_at(const T* base, int k) {
  return *(const __attribute__((address_space(1))) T*)((const __attribute__((address_space(1))) char*)base +
                                                       (uint32_t)k * (uint32_t)sizeof(T));
}

// An entry of a matrix.  Where the gathered vectors outgrow the L2 well
// (solve_kernels_256_streamed.hip), the load carries the non-temporal hint, which
// leaves the L2 to them: power-law QP n = 2e6, 7 TB/s of L2 misses, 32.0 -> 31.4 ms
// for 40 iterations.
#ifndef PDHCG_STREAMED
#define PDHCG_STREAMED 0
#endif
template <typename T>
__device__ __forceinline__ T gld_entry(const T* p) {
  return PDHCG_STREAMED ? gld_nt(p) : gld(p);
}
template <typename T>
__device__ __forceinline__ T gld_entry_at(const T* base, int k) {
  const auto* p = (const __attribute__((address_space(1))) T*)((const __attribute__((address_space(1))) char*)base +
                                                               (uint32_t)k * (uint32_t)sizeof(T));
  return PDHCG_STREAMED ? __builtin_nontemporal_load(p) : *p;
}

// a pointer or integer that is equal in all lanes, in scalar registers
template <typename T>
__device__ __forceinline__ T* uni(T* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return (T*)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// order this wave's LDS stores before its following loads by other lanes (the
// hardware keeps the order; this keeps the compiler from changing it)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// the row sums read up to prod[kTileNnz + 3 * kWave], that one included (lane_row_sums)
constexpr int kReadAhead = 3 * kWave + 1;
struct TileLds {
  double prod[kWaves][kTileNnz];
  double ahead[kReadAhead];  // read, and dropped, behind the last wave's stretch
};

// the workgroup's staging area
__device__ __forceinline__ TileLds& tile_lds() {
  __shared__ TileLds L;
  return L;
}

// Load through a pointer known to address LDS (ds_read rather than a flat load)
template <typename T>
__device__ __forceinline__ T lld(const T* p) {
  return *(const __attribute__((address_space(3))) T*)p;
}

// store through a generic pointer known to point into LDS
template <typename T>
__device__ __forceinline__ void lst(T* p, T v) {
  *(__attribute__((address_space(3))) T*)p = v;
}

// One tile: rows [ra, ra + nr), entries [z0, z0 + nz) of the first matrix and
// [w0, w0 + nw) of the second (scalars of the wave)
struct Tile {
  int ra, nr, z0, nz, w0, nw;
};

// the six descriptor words of tile t, one per lane (not waited for)
__device__ __forceinline__ int tile_words(const WgPart& pt, int t) {
  const int q = min(lane_id(), 5), k = t - pt.t0;
  return k < kCacheTiles ? lld(pt.tl + 6 * k + q) : gld(pt.tiles + 6 * (int64_t)t + q);
}

__device__ __forceinline__ Tile tile_of(int words) {
  const auto w = [&](int k) { return __builtin_amdgcn_readlane(words, k); };
  const int ra = w(0), z0 = w(2), w0 = w(4);
  return Tile{ra, w(1) - ra, z0, w(3) - z0, w0, w(5) - w0};
}

// run(tile) for this wave's tiles of the workgroup's share (tiles wave,
// wave + kWaves, ...); the next descriptor is on its way while one runs
template <typename Run>
__device__ __forceinline__ void for_wave_tiles(const WgPart& pt, const Run& run) {
  const int t1 = uni(pt.t1);
  int t = uni(pt.t0) + wave_id();
  if (t >= t1) return;
  int words = tile_words(pt, t);
  for (;;) {
    const Tile d = tile_of(words);
    t += kWaves;
    const bool more = t < t1;
    if (more) words = tile_words(pt, t);
    run(d);
    if (!more) return;
  }
}

// Where a tile's row offsets and entries come from: device memory, or the
// workgroup's rows held in LDS (lrp[j] = rowptr[r0 + j], entries from e0).
template <typename V_>
struct MemRows {
  using V = V_;
  const int32_t* rowptr;
  const int32_t* cols;
  const V* vals;
  // row offset ra + i, entries z0 + k (ra and z0 uniform, i and k small)
  __device__ __forceinline__ int rp(int ra, int i) const { return gld_at(rowptr + ra, i); }
  __device__ __forceinline__ int col(int z0, int k) const { return gld_entry_at(cols + z0, k); }
  __device__ __forceinline__ V val(int z0, int k) const { return gld_entry_at(vals + z0, k); }
};

template <typename V_>
struct LdsRows {
  using V = V_;
  const int32_t* lrp;
  const int32_t* lcol;
  const V* lval;
  int r0, e0;
  __device__ __forceinline__ int rp(int ra, int i) const { return lld(lrp + (ra - r0) + i); }
  __device__ __forceinline__ int col(int z0, int k) const { return lld(lcol + (z0 - e0) + k); }
  __device__ __forceinline__ V val(int z0, int k) const { return lld(lval + (z0 - e0) + k); }
};

// gathers in flight per lane: 8, or what a gather of several vectors declares
template <typename G, typename = void>
struct burst_of {
  static constexpr int value = 8;
};
template <typename G>
struct burst_of<G, std::void_t<decltype(G::kBurst)>> {
  static constexpr int value = G::kBurst;
};

// Products val * g(col) of the entries z0 .. z0 + nz - 1 into prod[0 .. nz),
// nz <= kTileNnz.  Loads are unconditional within a step of two entries per
// lane (indices clamped into the tile, surplus lanes repeat the last entry and
// store nothing) and steps beyond the tile's entries are skipped by the whole
// wave, so the index and value loads all issue before the first wait, then the
// gathers, and a small tile issues none for entries that it does not have.
constexpr int kLaneNnz = kTileNnz / kWave;
template <typename Src, typename G>
__device__ __forceinline__ void stage(const Src& src, const G& g, int z0, int nz, double* prod) {
  constexpr int B = burst_of<G>::value;
  const int lane = lane_id();
  int c[kLaneNnz];
  typename Src::V v[kLaneNnz];
#pragma unroll
  for (int u = 0; u < kLaneNnz; u += 2) {
    if (u * kWave >= nz) break;
#pragma unroll
    for (int q = u; q < u + 2; ++q) {
      const int k = min(q * kWave + lane, nz - 1);
      c[q] = src.col(z0, k);
      v[q] = src.val(z0, k);
    }
  }
#pragma unroll
  for (int u0 = 0; u0 < kLaneNnz; u0 += B) {
    double gv[B];
#pragma unroll
    for (int u = 0; u < B; u += 2) {
      if ((u0 + u) * kWave >= nz) break;
      gv[u] = g(c[u0 + u]);
      gv[u + 1] = g(c[u0 + u + 1]);
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      if ((u & 1) == 0 && (u0 + u) * kWave >= nz) break;
      const int k = (u0 + u) * kWave + lane;
      if (k < nz) prod[k] = (double)v[u0 + u] * gv[u];
    }
  }
}

// The same for two matrices over the same rows: entries [z0, z0 + nz) of the
// first, then [w0, w0 + nw) of the second, nz + nw <= kTileNnz, in one burst.
template <typename S, typename G>
__device__ __forceinline__ void stage2(const S& s1, const G& g1, int z0, int nz, const S& s2, const G& g2, int w0,
                                       int nw, double* prod) {
  const int lane = lane_id(), ntot = nz + nw;
  const int32_t* const c1 = s1.cols + z0;
  const int32_t* const c2 = s2.cols + ((int64_t)w0 - nz);
  const auto* const v1 = s1.vals + z0;
  const auto* const v2 = s2.vals + ((int64_t)w0 - nz);
  int c[kLaneNnz];
  typename S::V v[kLaneNnz];
#pragma unroll
  for (int u = 0; u < kLaneNnz; u += 2) {
    if (u * kWave >= ntot) break;
#pragma unroll
    for (int q = u; q < u + 2; ++q) {
      const int k = min(q * kWave + lane, ntot - 1);
      c[q] = gld_entry((k < nz ? c1 : c2) + k);
      v[q] = gld_entry((k < nz ? v1 : v2) + k);
    }
  }
  double gv[kLaneNnz];
#pragma unroll
  for (int u = 0; u < kLaneNnz; u += 2) {
    if (u * kWave >= ntot) break;
#pragma unroll
    for (int q = u; q < u + 2; ++q) {
      const int k = min(q * kWave + lane, ntot - 1);
      gv[q] = gld((k < nz ? g1.v : g2.v) + c[q]);
    }
  }
#pragma unroll
  for (int u = 0; u < kLaneNnz; ++u) {
    if ((u & 1) == 0 && u * kWave >= ntot) break;
    const int k = u * kWave + lane;
    if (k < ntot) prod[k] = (double)v[u] * gv[u];
  }
}

// a[j] = sum of prod[k] for k = beg[j] + lane, beg[j] + lane + G, ... < end[j],
// j < N, each in two chains.  Four entries of every sum are read at a time,
// whether a lane has them or not (reads stay within kReadAhead behind the staging
// area, surplus values are dropped): one LDS round trip per step instead of two.
// n = 1000 QP, 200 iterations: 6.67 -> 6.44 ms with the two matrices' sums
// interleaved; n = 1e5, FP32, 60 iterations: 3.70 -> 3.57 ms.
template <int N>
__device__ __forceinline__ void lane_row_sums(const double* prod, const int* beg, const int* end, int lane, int G,
                                              double* a) {
  double a0[N], a1[N];
  int k[N];
  bool more = false;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    a0[j] = a1[j] = 0.0;
    k[j] = min(beg[j] + lane, kTileNnz);
    more = more || k[j] < end[j];
  }
  while (more) {
    double v[N][4];
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) v[j][q] = lld(prod + k[j] + q * G);
    more = false;
#pragma unroll
    for (int j = 0; j < N; ++j) {
#pragma unroll
      for (int q = 0; q < 4; q += 2) {
        const double t0 = a0[j] + v[j][q], t1 = a1[j] + v[j][q + 1];
        a0[j] = k[j] + q * G < end[j] ? t0 : a0[j];
        a1[j] = k[j] + (q + 1) * G < end[j] ? t1 : a1[j];
      }
      k[j] = min(k[j] + 4 * G, kTileNnz);
      more = more || k[j] < end[j];
    }
  }
#pragma unroll
  for (int j = 0; j < N; ++j) a[j] = a0[j] + a1[j];
}

// A row longer than this many entries per lane of its group is summed by the
// whole wave instead (skewed tiles: one long row among many short ones)
constexpr int kLaneEntries = 8;
__device__ __forceinline__ int wide_row_len(int G) { return kLaneEntries * G > kWave ? kLaneEntries * G : kWave; }

// Lanes per row of a tile: the partition's group size G, at most what lets the
// wave sum all of the tile's rows at once.
__device__ __forceinline__ int tile_group(int G, int nr) {
  const int f = kWave >> (32 - __clz(nr - 1));  // 64 over the power of two at or above nr
  return f < G ? f : G;
}

// Row sums of a staged tile: lane group `lane / Gt` sums prod[beg[j] .. end[j]),
// j < N, of its row; the sums are valid in the group's last lane.  act: the group
// has a row.
template <int N>
__device__ __forceinline__ void wave_row_sums(const double* prod, const int* beg, const int* end, bool act, int Gt,
                                              double* s) {
  const int lane = lane_id(), sub = lane & (Gt - 1), limit = wide_row_len(Gt);
  bool wide[N];
  int e[N];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    wide[j] = act && end[j] - beg[j] > limit;
    e[j] = act && !wide[j] ? end[j] : beg[j];
  }
  lane_row_sums<N>(prod, beg, e, sub, Gt, s);
  group_sums_last<N>(s, Gt);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    uint64_t todo = __ballot(wide[j] && sub == Gt - 1);
    while (todo) {  // wide rows: the whole wave, one after another
      const int L = __builtin_ctzll(todo);
      todo &= todo - 1;
      const int wb = __builtin_amdgcn_readlane(beg[j], L), we = __builtin_amdgcn_readlane(end[j], L);
      double t;
      lane_row_sums<1>(prod, &wb, &we, lane, kWave, &t);
      t = lane_value(group_sum_last(t, kWave), kWave - 1);
      if (lane == L) s[j] = t;
    }
  }
}

// One tile: epi(row, s1, s2, pre(row)) for its rows, each in one lane, s1 and
// s2 the row's sums over the entries of the first and of the second matrix
// (TWO; else s2 = 0).  pre(row) loads the row's own inputs (rows of the tile,
// indices clamped into it) and is issued with the tile's loads, so those inputs
// cost no memory round trip of their own.  stage_in(prod) parks the products,
// the first matrix's in prod[0 .. nz), the second's behind them.
template <bool TWO, typename S1, typename S2, typename Stage, typename Pre, typename Epi>
__device__ __forceinline__ void tile_rows_staged(const Tile& t, int G, const S1& m1, const S2& m2,
                                                 const Stage& stage_in, const Pre& pre, Epi& epi) {
  double* const prod = tile_lds().prod[wave_id()];
  const int lane = lane_id();
  const int Gt = tile_group(G, t.nr), lg = 31 - __clz(Gt);
  const int i = min(lane >> lg, t.nr - 1);
  const bool act = (lane >> lg) < t.nr;
  constexpr int N = TWO ? 2 : 1;
  int beg[N], end[N];
  beg[0] = m1.rp(t.ra, i) - t.z0;
  end[0] = m1.rp(t.ra, i + 1) - t.z0;
  if constexpr (TWO) {
    beg[1] = m2.rp(t.ra, i) - t.w0 + t.nz;
    end[1] = m2.rp(t.ra, i + 1) - t.w0 + t.nz;
  }
  const auto pv = pre(t.ra, i);
  stage_in(prod);
  wave_sync();
  double s[N];
  wave_row_sums<N>(prod, beg, end, act, Gt, s);
  if (act && (lane & (Gt - 1)) == Gt - 1) epi(t.ra + i, s[0], TWO ? s[N - 1] : 0.0, pv);
  wave_sync();
}

// A tile that is one row of more than kTileNnz entries (at most kLongRow):
// summed straight from memory by the wave; its last lane ends with the row.
template <typename V, typename Gather>
__device__ __forceinline__ double wave_long_row(const MemRows<V>& m, int z0, int nz, const Gather& g) {
  return group_sum_last(row_partial(m.cols, m.vals, z0, z0 + nz, lane_id(), kWave, g), kWave);
}
template <typename V, typename Gather>
__device__ __forceinline__ double wave_long_row(const LdsRows<V>& m, int z0, int nz, const Gather& g) {
  double s = 0.0;
  for (int k = z0 + lane_id(); k < z0 + nz; k += kWave) s += (double)m.val(0, k) * g(m.col(0, k));
  return group_sum_last(s, kWave);
}

// the rows of the workgroup's tiles of a single matrix, the partition's first or
// (SECOND: the A' of a partition cut for a dense Q) its second
template <bool SECOND = false, typename Src, typename Gather, typename Pre, typename Epi>
__device__ __forceinline__ void part_rows(const WgPart& pt, const Src& src, const Gather& g, const Pre& pre, Epi epi) {
  const int G = uni(pt.group);
  for_wave_tiles(pt, [&](const Tile& d) {
    const Tile t = SECOND ? Tile{d.ra, d.nr, d.w0, d.nw, 0, 0} : d;
    if (t.nz > kTileNnz) {
      const auto pv = pre(t.ra, 0);
      const double s = wave_long_row(src, t.z0, t.nz, g);
      if (lane_id() == kWave - 1) epi(t.ra, s, pv);
      return;
    }
    auto put = [&](double* prod) {
      if (t.nz > 0) stage(src, g, t.z0, t.nz, prod);
    };
    auto one = [&](int i, double s, double, const auto& pv) { epi(i, s, pv); };
    tile_rows_staged<false>(t, G, src, src, put, pre, one);
  });
}

// The no-op prefetch.
struct NoPre {
  __device__ __forceinline__ int operator()(int, int) const { return 0; }
};

template <typename V, typename Gather, typename Epi>
__device__ __forceinline__ void part_rows(const WgPart& pt, const int32_t* rowptr, const int32_t* col, const V* val,
                                          const Gather& g, Epi epi) {
  part_rows(pt, MemRows<V>{uni(rowptr), uni(col), uni(val)}, g, NoPre{}, [&](int i, double s, int) { epi(i, s); });
}

// The rows of the workgroup's tiles of two matrices over the same rows (the
// stacked [Q | A'] pass): epi(row, sum1, sum2, pre(row)).
template <typename Pre, typename Epi>
__device__ __forceinline__ void part_rows2(const WgPart& pt, const MemRows<double>& m1, const GatherVec<double>& g1,
                                           const MemRows<double>& m2, const GatherVec<double>& g2, const Pre& pre,
                                           Epi epi) {
  const int G = uni(pt.group);
  for_wave_tiles(pt, [&](const Tile& t) {
    if (t.nz + t.nw > kTileNnz) {
      const auto pv = pre(t.ra, 0);
      const double a = wave_long_row(m1, t.z0, t.nz, g1);
      const double b = wave_long_row(m2, t.w0, t.nw, g2);
      if (lane_id() == kWave - 1) epi(t.ra, a, b, pv);
      return;
    }
    auto put = [&](double* prod) {
      if (t.nz + t.nw > 0) stage2(m1, g1, t.z0, t.nz, m2, g2, t.w0, t.nw, prod);
    };
    tile_rows_staged<true>(t, G, m1, m2, put, pre, epi);
  });
}

}  // namespace
}  // namespace pdhcg
