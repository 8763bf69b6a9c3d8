// The row sums of a staged tile, with the staging area against a protected page.
#include <sys/mman.h>
#include <sys/wait.h>
#include <unistd.h>

#include "solver.hpp"

// the two sums of a row of n1 + n2 entries by a whole wave, in a child process:
// 0, or the signal that ended it
extern "C" int simt_row_sums(int n1, int n2, double* out) {
  const size_t page = (size_t)sysconf(_SC_PAGESIZE), room = (sizeof(pdhcg::TileLds) + page - 1) / page * page;
  char* base = (char*)mmap(nullptr, room + page, PROT_READ | PROT_WRITE, MAP_SHARED | MAP_ANONYMOUS, -1, 0);
  mprotect(base + room, page, PROT_NONE);
  auto* tile = (pdhcg::TileLds*)(base + room - sizeof(pdhcg::TileLds));
  double* const prod = tile->prod[pdhcg::kWaves - 1];
  for (int k = 0; k < n1 + n2; ++k) prod[k] = k < n1 ? 1.0 : 1024.0;
  double* sums = (double*)base;  // (below the area: the child's results)
  const pid_t pid = fork();
  if (pid == 0) {
    const int beg[2] = {0, n1}, end[2] = {n1, n1 + n2};
    double total[2] = {0.0, 0.0};
    for (int lane = 0; lane < 64; ++lane) {
      double a[2];
      pdhcg::lane_row_sums<2>(prod, beg, end, lane, 64, a);
      total[0] += a[0];
      total[1] += a[1];
    }
    sums[0] = total[0];
    sums[1] = total[1];
    _exit(0);
  }
  int status = 0;
  waitpid(pid, &status, 0);
  out[0] = sums[0];
  out[1] = sums[1];
  munmap(base, room + page);
  return WIFSIGNALED(status) ? WTERMSIG(status) : 0;
}
