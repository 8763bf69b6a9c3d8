// Scheduler and HIP runtime of the host build (hip/hip_runtime.h beside this
// file).  A workgroup's lanes are fibers of one thread; a wave runs until each of
// its lanes waits for the others (a lane move, a wave or workgroup barrier), the
// waves in the order that simt_wave_order sets.  The workgroups of a cooperative
// launch are threads of which one runs at a time, until it sleeps in a wait.
#include "hip/hip_runtime.h"

#include <sys/mman.h>

#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <thread>
#include <vector>

#include "internal.hpp"

namespace simt {

thread_local Index lane_index, block_index, grid_dim, block_dim;

namespace {

constexpr size_t kStack = 256 << 10;
int g_descending = 0;              // waves from the last to the first
int g_refuse = 0, g_late = 0;      // cooperative launches to refuse; to run with waits that are over at once
uint64_t g_tick = 1, g_clock = 0;  // ticks per reading of the clock
int g_coop = 0, g_plain = 0;       // launches that ran
int g_cus = 64, g_per_cu = 2, g_l2 = 4 << 20;

__attribute__((naked, noinline)) void switch_to(void**, void*) {
  asm("pushq %rbp; pushq %rbx; pushq %r12; pushq %r13; pushq %r14; pushq %r15\n"
      "movq %rsp, (%rdi); movq %rsi, %rsp\n"
      "popq %r15; popq %r14; popq %r13; popq %r12; popq %rbx; popq %rbp; ret");
}

enum State { kRun, kAtCollective, kAtSync, kAsleep, kDone };
struct Lane {
  void* sp;
  State state;
  Index index;
  Kind kind;
  uint64_t v, out;
  int a, b;
};

struct Stacks {
  char* base = nullptr;
  int n = 0;
  ~Stacks() {
    if (base) munmap(base, kStack * n);
  }
};

struct Turns {  // whose turn it is among the workgroups of a cooperative launch
  std::mutex mu;
  std::condition_variable cv;
  std::vector<char> alive;
  int now = 0;
  void pass(int me, bool end) {
    std::unique_lock<std::mutex> lock(mu);
    if (end) alive[me] = 0;
    for (size_t k = 1; k <= alive.size(); ++k) {
      const int q = (int)((me + k) % alive.size());
      if (alive[q]) {
        now = q;
        break;
      }
    }
    cv.notify_all();
    if (!end) cv.wait(lock, [&] { return now == me; });
  }
  void first(int me) {
    std::unique_lock<std::mutex> lock(mu);
    cv.wait(lock, [&] { return now == me; });
  }
};

struct Workgroup {
  std::vector<Lane> lanes;
  const std::function<void()>* body = nullptr;
  Turns* turns = nullptr;
  int id = 0;
  void* sched = nullptr;
  Lane* cur = nullptr;
};
thread_local Workgroup* wg = nullptr;
thread_local Stacks stacks;
thread_local std::vector<double> dyn;

void enter() {
  (*wg->body)();
  wg->cur->state = kDone;
  void* dead;
  switch_to(&dead, wg->sched);
}

void wait_as(State s) {
  Lane* me = wg->cur;
  me->state = s;
  switch_to(&me->sp, wg->sched);
}

void exchange(Lane* w, int n) {
  for (int i = 0; i < n; ++i) {
    Lane& l = w[i];
    if (l.state == kDone) continue;
    uint64_t r = 0;
    switch (l.kind) {
      case kDpp: {
        int src = -1;
        const int row = i / 16;
        if ((l.a & ~0xF) == 0x110) src = i % 16 >= (l.a & 0xF) ? i - (l.a & 0xF) : -1;  // row_shr
        else if (l.a == 0x142) src = row > 0 ? 16 * row - 1 : -1;                        // row_bcast:15
        else if (l.a == 0x143) src = i >= 32 ? 31 : -1;                                  // row_bcast:31
        if (!(l.b >> row & 1)) src = -1;
        r = src >= 0 ? w[src].v : 0;
        break;
      }
      case kReadLane: r = w[l.a].v; break;
      case kShflXor: r = w[(i & ~(l.b - 1)) + ((i ^ l.a) & (l.b - 1))].v; break;
      case kBallot:
        for (int j = 0; j < n; ++j) r |= (w[j].state != kDone ? w[j].v : 0) << j;
        break;
      case kWaveBarrier: break;
    }
    l.out = r;
  }
}

// one workgroup from start to end; false if its lanes wait for one another for ever
bool run_workgroup(Workgroup& W, int nlanes) {
  wg = &W;
  if (stacks.n < nlanes) {
    if (stacks.base) munmap(stacks.base, kStack * stacks.n);
    stacks.base = (char*)mmap(nullptr, kStack * nlanes, PROT_READ | PROT_WRITE,
                              MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    stacks.n = nlanes;
  }
  W.lanes.assign(nlanes, Lane{});
  for (int i = 0; i < nlanes; ++i) {
    void** top = (void**)(stacks.base + kStack * (i + 1));
    top[-2] = (void*)enter;
    W.lanes[i].sp = top - 8;
    W.lanes[i].index = Index{(unsigned)i, 0, 0};
  }
  const int nw = (nlanes + 63) / 64;
  for (;;) {
    bool moved = false;
    int sync = 0, asleep = 0, done = 0;
    for (int k = 0; k < nw; ++k) {
      const int w = g_descending ? nw - 1 - k : k;
      Lane* L = &W.lanes[64 * w];
      const int n = std::min(64, nlanes - 64 * w);
      for (;;) {
        int at[5] = {0, 0, 0, 0, 0};
        for (int i = 0; i < n; ++i) {
          if (L[i].state == kRun) {
            W.cur = &L[i];
            lane_index = L[i].index;
            switch_to(&W.sched, L[i].sp);
            moved = true;
          }
          ++at[L[i].state];
        }
        if (at[kAtCollective] > 0 && at[kAtCollective] + at[kDone] == n) {
          exchange(L, n);
          for (int i = 0; i < n; ++i)
            if (L[i].state == kAtCollective) L[i].state = kRun;
          continue;
        }
        sync += at[kAtSync];
        asleep += at[kAsleep];
        done += at[kDone];
        break;
      }
    }
    if (done == nlanes) return true;
    if (sync + done == nlanes) {
      for (Lane& l : W.lanes)
        if (l.state == kAtSync) l.state = kRun;
      continue;
    }
    if (moved) continue;
    if (asleep == 0) {
      fprintf(stderr, "simt: workgroup %d: lanes wait for one another\n", W.id);
      return false;
    }
    if (W.turns) W.turns->pass(W.id, false);
    for (Lane& l : W.lanes)
      if (l.state == kAsleep) l.state = kRun;
  }
}

void place(int b, dim3 grid, dim3 block) {
  block_index = Index{b % grid.x, b / grid.x % grid.y, b / grid.x / grid.y};
  grid_dim = Index{grid.x, grid.y, grid.z};
  block_dim = Index{block.x, block.y, block.z};
}

hipError_t launch_cooperative(dim3 grid, dim3 block, unsigned lds, const std::function<void()>& body) {
  const int nb = (int)grid.x;
  if (g_refuse > 0) {
    --g_refuse;
    return hipErrorCooperativeLaunchTooLarge;
  }
  if (nb > g_cus * g_per_cu) return hipErrorCooperativeLaunchTooLarge;
  ++g_coop;
  const uint64_t tick = g_tick;
  if (g_late > 0) {
    --g_late;
    g_tick = 600000000;  // (6 s)
  }
  Turns turns;
  turns.alive.assign(nb, 1);
  std::vector<char> ok(nb, 0);
  std::vector<std::thread> threads;
  for (int b = 0; b < nb; ++b)
    threads.emplace_back([&, b] {
      place(b, grid, block);
      dyn.assign(lds / sizeof(double) + 1, 0.0);
      Workgroup W;
      W.body = &body;
      W.turns = &turns;
      W.id = b;
      turns.first(b);
      ok[b] = run_workgroup(W, (int)block.x);
      turns.pass(b, true);
    });
  for (std::thread& t : threads) t.join();
  g_tick = tick;
  for (char o : ok)
    if (!o) return hipErrorLaunchFailure;
  return hipSuccess;
}

}  // namespace

uint64_t collective(Kind kind, uint64_t v, int a, int b) {
  Lane* me = wg->cur;
  me->kind = kind;
  me->v = v;
  me->a = a;
  me->b = b;
  wait_as(kAtCollective);
  return me->out;
}
void sync_threads() { wait_as(kAtSync); }
void yield_block() { wait_as(kAsleep); }
uint64_t clock_ticks() { return __atomic_add_fetch(&g_clock, g_tick, __ATOMIC_SEQ_CST); }
uint32_t xcd() { return block_index.x % 8; }
char* dynamic_lds() { return (char*)dyn.data(); }

hipError_t launch(dim3 grid, dim3 block, const std::function<void()>& body) {
  bool ok = true;
  ++g_plain;
  // (on a thread of its own: a workgroup's LDS is thread-local)
  std::thread([&] {
    for (int b = 0; b < (int)(grid.x * grid.y * grid.z) && ok; ++b) {
      place(b, grid, block);
      Workgroup W;
      W.body = &body;
      W.id = b;
      ok = run_workgroup(W, (int)block.x);
    }
  }).join();
  if (!ok) abort();
  return hipSuccess;
}

}  // namespace simt

namespace pdhcg {
void pdhcg_solve_kernel(const SolveParams*);
void pdhcg_solve_kernel_wg256(const SolveParams*);
void pdhcg_solve_kernel_wg256_streamed(const SolveParams*);
void pdhcg_power_kernel_wg256_streamed(PowerParams);
void pdhcg_power_kernel(PowerParams);
void pdhcg_power_kernel_wg256(PowerParams);
void pdhcg_batch_kernel_team(BatchParams);
void pdhcg_batch_kernel_sparse_team(BatchParams);
}  // namespace pdhcg

using namespace pdhcg;

extern "C" {

void simt_wave_order(int descending) { simt::g_descending = descending; }
void simt_refuse(int launches) { simt::g_refuse = launches; }
void simt_late(int launches) { simt::g_late = launches; }
void simt_tick(uint64_t ticks) { simt::g_tick = ticks; }
void simt_l2(int bytes) { simt::g_l2 = bytes; }
// launches since the last call: cooperative ones * 1000 + the others
int simt_launches() {
  const int n = simt::g_coop * 1000 + simt::g_plain;
  simt::g_coop = simt::g_plain = 0;
  return n;
}

hipError_t hipLaunchCooperativeKernel(const void* f, dim3 grid, dim3 block, void** args, unsigned lds, hipStream_t) {
  std::function<void()> body;
  auto bind = [&](auto* k, auto* arg) {
    if (f == (const void*)k) body = [k, arg] { k(*arg); };
  };
  bind(pdhcg_solve_kernel, (const SolveParams**)args[0]);
  bind(pdhcg_solve_kernel_wg256, (const SolveParams**)args[0]);
  bind(pdhcg_solve_kernel_wg256_streamed, (const SolveParams**)args[0]);
  bind(pdhcg_power_kernel_wg256_streamed, (PowerParams*)args[0]);
  bind(pdhcg_power_kernel, (PowerParams*)args[0]);
  bind(pdhcg_power_kernel_wg256, (PowerParams*)args[0]);
  bind(pdhcg_batch_kernel_team, (BatchParams*)args[0]);
  bind(pdhcg_batch_kernel_sparse_team, (BatchParams*)args[0]);
  return simt::launch_cooperative(grid, block, lds, body);
}

hipError_t hipMalloc(void** p, size_t n) {
  *p = aligned_alloc(256, (n + 511) / 256 * 256);
  memset(*p, 0xFF, std::min<size_t>(n, 16 << 20));  // (NaN: what is read before it is written shows)
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  memmove(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "host build"; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeL2CacheSize ? simt::g_l2 : a == hipDeviceAttributeMultiprocessorCount ? simt::g_cus : 160 << 10;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) {
  *a = hipFuncAttributes{};
  a->sharedSizeBytes = 60 << 10;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = simt::g_per_cu;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* s) {
  *p = const_cast<void*>(s);
  return hipSuccess;
}
// events: readings of the kernels' clock (100 MHz)
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = (hipEvent_t) new uint64_t;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  delete (uint64_t*)e;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  *(uint64_t*)e = simt::g_clock;
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  *ms = 1e-5f * (float)(*(uint64_t*)b - *(uint64_t*)a);
  return hipSuccess;
}

}  // extern "C"
