// Launches of kernels the timer may sample, and the sizes they are launched with.
#pragma once

#include <hip/hip_ext.h>

#include "common.h"

// Launch of a kernel the timer may sample: a sampled launch carries the
// timer's start and stop events in its dispatch (they then hold the times the
// dispatch began and completed, which include the command processor's
// per-dispatch work around the kernel); while a graph is being captured, the
// kernel node is handed to the timer instead.
#define LAUNCH_TIMED(fam, kernel, grid, block, shm, st, ...)                              \
  do {                                                                                     \
    hipEvent_t ev0_ = nullptr, ev1_ = nullptr;                                             \
    if (timer_events((fam), &ev0_, &ev1_))                                                 \
      hipExtLaunchKernelGGL(kernel, grid, block, shm, st, ev0_, ev1_, 0, __VA_ARGS__);    \
    else                                                                                   \
      hipLaunchKernelGGL(kernel, grid, block, shm, st, __VA_ARGS__);                       \
    timer_captured((fam), st);                                                             \
  } while (0)

namespace lddmm {
inline unsigned nblk(long long n, int t) { return (unsigned)((n + t - 1) / t); }
constexpr int tiles16(int n) { return (n + 15) / 16; }
}  // namespace lddmm
