// Replay of captured CG steps, shared by the CG paths.
#pragma once

#include <algorithm>
#include <cstdlib>

#include "common.h"

namespace mbl {

// Runs step(stream) m - it times: from a hipGraph captured on a private
// non-blocking stream (forked from and joined back to s by events) when at
// least 8 steps remain, else launch by launch.  The legacy default stream
// cannot be captured, and a capture on a caller's blocking stream would forbid
// legacy-stream work in every other thread of the process meanwhile.
// With a stop check the replays are issued in chunks of kStopChunk, one chunk
// queued ahead of the one running, and no further chunk is issued once the
// check triggers.  Returns the number of steps run.
constexpr int kStopChunk = 32;

template <class F>
int replay_steps(F&& step, int it, int m, hipStream_t s, const StopCheck* stop) {
  const char* env = std::getenv("MBL_PCG_GRAPH");
  const bool graph_on = env == nullptr || std::atoi(env) != 0;
  if (graph_on && m - it >= 8) {
    hipStream_t own = nullptr;
    hipEvent_t fork = nullptr, join = nullptr, mark[2] = {nullptr, nullptr};
    MBL_HIP(hipStreamCreateWithFlags(&own, hipStreamNonBlocking));
    hipError_t err = hipEventCreateWithFlags(&fork, hipEventDisableTiming);
    if (err == hipSuccess) err = hipEventCreateWithFlags(&join, hipEventDisableTiming);
    for (int k = 0; k < 2 && err == hipSuccess; ++k)
      err = hipEventCreateWithFlags(&mark[k], hipEventDisableTiming);
    if (err == hipSuccess) err = hipEventRecord(fork, s);
    if (err == hipSuccess) err = hipStreamWaitEvent(own, fork, 0);
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    if (err == hipSuccess) err = hipStreamBeginCapture(own, hipStreamCaptureModeThreadLocal);
    if (err == hipSuccess) {
      try {
        step(own);
      } catch (...) {
        hipGraph_t dropped = nullptr;
        (void)hipStreamEndCapture(own, &dropped);
        if (dropped) (void)hipGraphDestroy(dropped);
        (void)hipStreamSynchronize(own);
        (void)hipStreamDestroy(own);
        (void)hipEventDestroy(fork);
        (void)hipEventDestroy(join);
        for (hipEvent_t e : mark)
          if (e) (void)hipEventDestroy(e);
        throw;
      }
      err = hipStreamEndCapture(own, &graph);
    }
    if (err == hipSuccess) err = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    int chunk = 0;
    while (err == hipSuccess && it < m) {
      const int end = stop ? std::min(m, it + kStopChunk) : m;
      for (; err == hipSuccess && it < end; ++it) err = hipGraphLaunch(exec, own);
      if (!stop || err != hipSuccess || it >= m) continue;
      // wait for the chunk before this one, then decide whether to go on
      err = hipEventRecord(mark[chunk & 1], own);
      if (err == hipSuccess && chunk > 0) err = hipEventSynchronize(mark[(chunk - 1) & 1]);
      ++chunk;
      if (err == hipSuccess && stop->triggered()) break;
    }
    if (err == hipSuccess) err = hipEventRecord(join, own);
    if (err == hipSuccess) err = hipStreamWaitEvent(s, join, 0);
    // the graph and its stream are torn down only after the replays finished
    const hipError_t se = hipStreamSynchronize(own);
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    (void)hipStreamDestroy(own);
    if (fork) (void)hipEventDestroy(fork);
    if (join) (void)hipEventDestroy(join);
    for (hipEvent_t e : mark)
      if (e) (void)hipEventDestroy(e);
    MBL_HIP(err);
    MBL_HIP(se);
    return it;
  }
  for (; it < m; ++it) {
    if (stop && it % kStopChunk == 0 && stop->triggered()) break;
    step(s);
  }
  return it;
}

}  // namespace mbl
