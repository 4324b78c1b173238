// Eight lanes of a wavefront run on the host in lockstep: a fiber per lane,
// switched at the cross-lane operations.  Every lane reaches the same
// operations in the same order (the condition the device code meets as well);
// a lane stores what it contributes, yields until all eight have, reads, and
// yields until all eight have read.
#pragma once
#include <stdio.h>
#include <stdlib.h>
#include <ucontext.h>
#include <functional>
#include <vector>

struct LaneId {
  unsigned x;
};
static LaneId threadIdx;

namespace lanes {
constexpr int N = 8;
static ucontext_t home, ctx[N];
static bool done[N];
static double slot[N];
static std::function<void(int)> body;

static void enter(int lane) {
  body(lane);
  done[lane] = true;
  swapcontext(&ctx[lane], &home);
}
static void yield() {
  const int lane = (int)threadIdx.x;
  swapcontext(&ctx[lane], &home);
}
static void run(std::function<void(int)> f) {
  static std::vector<char> stacks(N * (1 << 18));
  body = f;
  for (int l = 0; l < N; l++) {
    done[l] = false;
    getcontext(&ctx[l]);
    ctx[l].uc_stack.ss_sp = &stacks[(size_t)l << 18];
    ctx[l].uc_stack.ss_size = 1 << 18;
    ctx[l].uc_link = nullptr;
    makecontext(&ctx[l], (void (*)())enter, 1, l);
  }
  for (int left = N; left > 0;) {
    const int before = left;
    left = 0;
    for (int l = 0; l < N; l++)
      if (!done[l]) {
        threadIdx.x = (unsigned)l;
        swapcontext(&home, &ctx[l]);
        left += !done[l];
      }
    if (left != 0 && left != before) {   // one lane returned while another waits for it
      fprintf(stderr, "lanes diverged\n");
      exit(3);
    }
  }
}
}  // namespace lanes

static inline double __shfl(double x, int from, int width) {
  if (width != lanes::N) exit(4);
  lanes::slot[threadIdx.x] = x;
  lanes::yield();
  const double y = lanes::slot[from];
  lanes::yield();
  return y;
}
static inline unsigned long long __ballot(bool p) {
  lanes::slot[threadIdx.x] = p ? 1.0 : 0.0;
  lanes::yield();
  unsigned long long m = 0;
  for (int l = 0; l < lanes::N; l++) m |= (unsigned long long)(lanes::slot[l] != 0.0) << l;
  lanes::yield();
  return m;
}
static inline int __ffs(unsigned x) { return __builtin_ffs((int)x); }
