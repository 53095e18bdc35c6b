// Replay of fixed launch sequences from HIP graphs.  A solver iteration is a fixed
// sequence of kernel launches whose arguments do not change between iterations, so it
// is captured once (on a private stream, nothing runs during capture) and replayed on
// the caller's stream: one launch per replay instead of one per kernel.  Only kernels
// are captured (no memset or copy nodes).
#pragma once

#include <hip/hip_runtime_api.h>

#include <atomic>

#include "capi.hpp"

namespace pafem {

// Process-wide switch (pafem_set_graph_mode): 1 = replay solver iterations from
// graphs (default), 0 = launch every kernel directly.
std::atomic<int>& graph_mode_flag();
inline bool graphs_enabled() { return graph_mode_flag().load(std::memory_order_relaxed) != 0; }

// Whether a solver should capture `kernels` launches that it will replay `replays` times at
// most.  The graphs live for one solve, capture and instantiation cost about 2 us a kernel, and
// a replay's own launch as much as several kernels'.  Jacobi-PCG, direct -> graph: batches of 5
// kernels (two iterations) 0.87 -> 1.10 ms a solve of 16 replays and 3.22 -> 3.80 of 64 (4913
// dofs), of 6 (0.5M dofs) 2.34 -> 2.56 and 8.96 -> 9.54; 9 kernels 1.57 -> 1.49 and 5.97 ->
// 5.36, 17 kernels 2.42 -> 2.31 and 9.28 -> 8.53, 41 kernels 4.88 -> 4.76 and 19.5 -> 18.2; 8
// kernels (element-vector scatter) 1.37 -> 1.24 and 5.22 -> 4.35; on 0.5M dofs, where the
// device is the slower side, equal to 2 % from 9 kernels on.  Pairs of multigrid FCG iterations
// of 38 to 58 kernels, replayed 6 to 13 times, 0.96 to 1.07 times as fast; of about 90 kernels
// (p = 3) 18.5 -> 19.0 ms; 200 CG iterations in 2D as one graph of 600 kernels, replayed once,
// 9.6 -> 10.9 ms.
inline bool graph_pays(int kernels, int replays) {
  return kernels >= 8 && kernels <= 64 && replays >= 16;
}

// graphs launched by all solves of the process (pafem_graph_replays)
std::atomic<int64_t>& graph_replay_count();

class CapturedGraph {
 public:
  CapturedGraph() = default;
  CapturedGraph(const CapturedGraph&) = delete;
  CapturedGraph& operator=(const CapturedGraph&) = delete;
  ~CapturedGraph() { reset(); }

  bool ready() const { return exec_ != nullptr; }

  // Records body(stream) into the graph; body must only launch kernels.
  template <typename F>
  void capture(F&& body) {
    reset();
    hip_check(hipStreamCreateWithFlags(&cs_, hipStreamNonBlocking), "capture stream");
    hip_check(hipStreamBeginCapture(cs_, hipStreamCaptureModeThreadLocal), "begin capture");
    try {
      body(cs_);
    } catch (...) {
      hipGraph_t g = nullptr;
      hipStreamEndCapture(cs_, &g);
      if (g) hipGraphDestroy(g);
      throw;
    }
    hip_check(hipStreamEndCapture(cs_, &graph_), "end capture");
    hip_check(hipGraphInstantiate(&exec_, graph_, nullptr, nullptr, 0), "graph instantiate");
  }

  void launch(hipStream_t st) {
    hip_check(hipGraphLaunch(exec_, st), "graph launch");
    graph_replay_count().fetch_add(1, std::memory_order_relaxed);
  }

  void reset() {
    if (exec_) hipGraphExecDestroy(exec_);
    if (graph_) hipGraphDestroy(graph_);
    if (cs_) hipStreamDestroy(cs_);
    exec_ = nullptr;
    graph_ = nullptr;
    cs_ = nullptr;
  }

 private:
  hipStream_t cs_ = nullptr;
  hipGraph_t graph_ = nullptr;
  hipGraphExec_t exec_ = nullptr;
};

}  // namespace pafem
