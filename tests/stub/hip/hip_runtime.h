// The part of the HIP runtime the graph cache calls, on the host: streams run nothing until the driver says that
// what was launched on them has ended. An executable graph destroyed before that is counted.
#pragma once
#include <vector>

enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorNotReady = 600 };
enum { hipStreamCaptureModeThreadLocal = 1, hipEventDisableTiming = 2 };

struct FakeGraph {
  int launches = 0, ended = 0;
};
struct FakeEvent {
  FakeGraph* graph = nullptr;  // the graph whose launches so far it stands behind
  int launches = 0;
  bool done() const { return !graph || graph->ended >= launches; }
};
using hipStream_t = void*;
using hipGraph_t = FakeGraph*;
using hipGraphExec_t = FakeGraph*;
using hipEvent_t = FakeEvent*;

struct FakeHip {
  int captures = 0, destroyed = 0, destroyed_running = 0, waits = 0, captured_during = 0;
  FakeGraph* last = nullptr;
  std::vector<FakeGraph*> live;
};
inline FakeHip fake;

inline hipError_t hipStreamBeginCapture(hipStream_t, int) { return hipSuccess; }
inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = new FakeGraph;
  return hipSuccess;
}
inline hipError_t hipGraphDestroy(hipGraph_t g) {
  delete g;
  return hipSuccess;
}
inline hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, void*, void*, size_t) {
  ++fake.captures;
  *e = new FakeGraph;
  fake.live.push_back(*e);
  return hipSuccess;
}
inline hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
  ++e->launches;
  fake.last = e;
  return hipSuccess;
}
inline hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  ++fake.destroyed;
  if (e->ended < e->launches) ++fake.destroyed_running;
  return hipSuccess;  // the graph itself stays, for the driver to end its launches
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, int) {
  *e = new FakeEvent;
  return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  e->graph = fake.last;
  e->launches = fake.last->launches;
  return hipSuccess;
}
inline hipError_t hipEventQuery(hipEvent_t e) { return e->done() ? hipSuccess : hipErrorNotReady; }
inline hipError_t hipEventSynchronize(hipEvent_t e) {
  ++fake.waits;
  if (e->graph) e->graph->ended = e->launches;  // the wait lasts until it has ended
  return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) {
  delete e;
  return hipSuccess;
}
inline hipError_t hipPeekAtLastError() { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
