// Side streams for launches that touch disjoint problems.
#pragma once

#include "internal.hpp"

namespace tebd {

// The size classes of one batched factorisation touch disjoint problems and
// each fills only a few waves per CU, so they run side by side: the first
// class on the caller's stream, the others on side streams (default
// priority) forked from it and joined back with events.  Side streams and
// events are per host thread and device, created on first use.
constexpr int kSide = 3;
struct SideStreams {
  bool ready = false;
  hipStream_t st[kSide];
  hipEvent_t fork, join[kSide];
};

inline hipError_t side_streams(SideStreams*& out) {
  static thread_local SideStreams tab[16];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 16) {
    out = nullptr;
    return hipSuccess;
  }
  SideStreams& ss = tab[dev];
  if (!ss.ready) {
    e = hipEventCreateWithFlags(&ss.fork, hipEventDisableTiming);
    for (int i = 0; i < kSide && e == hipSuccess; ++i) {
      e = hipStreamCreateWithFlags(&ss.st[i], hipStreamNonBlocking);
      if (e == hipSuccess) e = hipEventCreateWithFlags(&ss.join[i], hipEventDisableTiming);
    }
    if (e != hipSuccess) return e;
    ss.ready = true;
  }
  out = &ss;
  return hipSuccess;
}

// Run launches[0..n) (each a callable taking a stream) concurrently after
// everything already enqueued on s; s continues after all of them.  Small
// batches, and the second pass of the adaptive rank (which re-runs only the
// few rejected problems), run them in order on s: there the fork and join
// cost more than the overlap gains.
constexpr int kForkMinProblems = 64;

template <class L>
hipError_t fork_join(hipStream_t s, L* launches, int n, const Common& c) {
  if (n == 0) return hipSuccess;
  SideStreams* ss = nullptr;
  const bool fork = n > 1 && c.nprob >= kForkMinProblems && !c.pass2 && !c.serial;
  hipError_t e = fork ? side_streams(ss) : hipSuccess;
  if (e != hipSuccess) return e;
  if (n == 1 || !ss) {
    for (int i = 0; i < n; ++i) {
      launches[i](s);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  e = hipEventRecord(ss->fork, s);
  if (e != hipSuccess) return e;
  const int side = n - 1 < kSide ? n - 1 : kSide;
  for (int i = 0; i < side; ++i) {
    e = hipStreamWaitEvent(ss->st[i], ss->fork, 0);
    if (e != hipSuccess) return e;
  }
  for (int i = 0; i < n; ++i) {
    hipStream_t t = i == 0 ? s : ss->st[(i - 1) % side];
    launches[i](t);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  for (int i = 0; i < side; ++i) {
    e = hipEventRecord(ss->join[i], ss->st[i]);
    if (e == hipSuccess) e = hipStreamWaitEvent(s, ss->join[i], 0);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace tebd
