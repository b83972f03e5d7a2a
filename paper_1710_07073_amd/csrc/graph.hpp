// Capture of a fixed number of method steps into a HIP graph, replayed while the step inputs
// (bubble constants, bubble buffers, ping-pong parities) stay the same. The graph holds kernel
// launches only (buffers are cleared by fill kernels, never by memset nodes).
#pragma once

#include <hip/hip_runtime.h>
#include <string.h>

#include "../../include/lbm.h"

namespace lbm {

struct GraphKey {
  bubble_params p;
  bubble_soa s;
  int32_t nb, cur, flag, steps;
  uint32_t mode;  // the rest of the host step state and the launch configuration
  bool valid;

  static GraphKey of(const bubble_params* p, const bubble_soa* s, int32_t nb, int cur, int flag,
                     int steps, uint32_t mode) {
    GraphKey k;
    memset(&k, 0, sizeof(k));
    if (p) memcpy(&k.p, p, sizeof(*p));
    if (s) memcpy(&k.s, s, sizeof(*s));
    k.nb = nb;
    k.cur = cur;
    k.flag = flag;
    k.steps = steps;
    k.mode = mode;
    k.valid = true;
    return k;
  }
  bool same(const GraphKey& o) const {
    return valid && o.valid && memcmp(&p, &o.p, sizeof(p)) == 0 &&
           memcmp(&s, &o.s, sizeof(s)) == 0 && nb == o.nb && cur == o.cur && flag == o.flag &&
           steps == o.steps && mode == o.mode;
  }
};

// A captured graph and the end of its last replay. The runtime still walks a graph it replays, one of several
// streams most of all: it may be destroyed only once that replay has ended.
struct GraphExec {
  hipGraphExec_t exec = nullptr;
  hipEvent_t done = nullptr;

  void destroy() {
    if (done) {
      (void)hipEventSynchronize(done);  // ended long ago as a rule
      (void)hipEventDestroy(done);
    }
    if (exec) (void)hipGraphExecDestroy(exec);
    exec = nullptr;
    done = nullptr;
  }
};

// A few captured graphs, each with the host step state its replay leaves behind (Post); a new
// key replaces the least recently used one. Replaced graphs wait for the end of their last replay among the old
// ones, of which a few are kept.
template <class Post, int N = 2>
class GraphCache {
 public:
  GraphCache() = default;
  ~GraphCache() {
    reset();
    for (int i = 0; i < nold_; ++i) old_[i].destroy();
  }
  GraphCache(const GraphCache&) = delete;
  GraphCache& operator=(const GraphCache&) = delete;

  // No graph is replayed any more; no call to the runtime, so also for a caller that captures.
  void reset() {
    for (Slot& s : slot_) retire(s);
  }

  // Capture `enqueue` on stream s unless a graph for the same key exists. forked: on a second stream too; such a
  // graph is captured once no other replays (a process that captured and replaced hundreds of them during
  // replays has ended in a segmentation fault inside the runtime, for a reason that was not found).
  template <class F>
  hipError_t ensure(const GraphKey& key, hipStream_t s, bool forked, F&& enqueue, bool* captured) {
    *captured = false;
    int k = -1;
    for (int i = 0; i < N; ++i)
      if (slot_[i].g.exec && slot_[i].key.same(key)) k = i;
    if (k >= 0) {
      cur_ = k;
      slot_[k].used = ++clock_;
      return hipSuccess;
    }
    k = 0;
    for (int i = 1; i < N; ++i)
      if (slot_[i].used < slot_[k].used) k = i;
    Slot& slot = slot_[k];
    cur_ = k;
    slot.used = ++clock_;
    retire(slot);
    if (forked) wait();
    clear_old();
    hipError_t e = hipEventCreateWithFlags(&slot.g.done, hipEventDisableTiming);
    if (e != hipSuccess) return e;
    hipGraph_t g = nullptr;
    e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
      const hipError_t ee = enqueue();
      e = hipStreamEndCapture(s, &g);
      if (ee != hipSuccess) {
        if (e == hipSuccess && g) (void)hipGraphDestroy(g);
        e = ee;
      } else if (e == hipSuccess) {
        e = hipGraphInstantiate(&slot.g.exec, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (e != hipSuccess) slot.g.exec = nullptr;
      }
    }
    if (e != hipSuccess) {
      slot.g.destroy();
      return e;
    }
    slot.key = key;
    *captured = true;
    return hipSuccess;
  }

  // Replays the graph of the last ensure().
  hipError_t launch(hipStream_t s) {
    GraphExec& g = slot_[cur_].g;
    const hipError_t e = hipGraphLaunch(g.exec, s);
    return e == hipSuccess ? hipEventRecord(g.done, s) : e;
  }
  Post& post() { return slot_[cur_].post; }

 private:
  struct Slot {
    GraphExec g;
    GraphKey key{};
    Post post{};
    unsigned long long used = 0;
  };
  static constexpr int kOldMax = 8;  // kept by clear_old(), before the next of which at most N more come

  void retire(Slot& s) {
    if (s.g.exec) old_[nold_++] = s.g;
    s.g = GraphExec{};
  }
  // Waits for the end of every replay.
  void wait() {
    for (Slot& s : slot_)
      if (s.g.exec) (void)hipEventSynchronize(s.g.done);
    for (int i = 0; i < nold_; ++i) (void)hipEventSynchronize(old_[i].done);
  }
  // Destroys the old graphs whose last replay has ended; waits for the oldest ones if there are many.
  void clear_old() {
    int kept = 0;
    for (int i = 0; i < nold_; ++i) {
      const hipError_t before = hipPeekAtLastError();
      const bool ended = hipEventQuery(old_[i].done) == hipSuccess;
      if (!ended && before == hipSuccess) (void)hipGetLastError();  // "not ready" is no error
      if (ended || nold_ - i > kOldMax)
        old_[i].destroy();
      else
        old_[kept++] = old_[i];
    }
    nold_ = kept;
  }

  Slot slot_[N];
  GraphExec old_[kOldMax + N];
  int nold_ = 0;
  int cur_ = 0;
  unsigned long long clock_ = 0;
};

}  // namespace lbm
