// A second stream per device for work that can overlap the main chain of a
// training step (the weight-gradient GEMMs, the loss-term reduction), plus the
// events that fork it from and join it back into the caller's stream, inside
// captured graphs (the side stream joins the capture through the fork event).
// Created on first use per device, kept for the life of the process, at the
// default priority.  CPRA_OVERLAP=0 in the environment keeps all work on the
// caller's stream.
#include <cstdlib>
#include <map>
#include <mutex>

#include "common.hpp"

namespace cpra {

namespace {
std::mutex g_side_mu;
std::map<int, SideStream> g_side;

cpra_status get_side_stream(SideStream** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) CPRA_FAIL(CPRA_ERR_HIP, "side stream: hipGetDevice: %s", hipGetErrorString(e));
  std::lock_guard<std::mutex> lk(g_side_mu);
  auto it = g_side.find(dev);
  if (it == g_side.end()) {
    SideStream s{};
    e = hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking);
    if (e != hipSuccess) CPRA_FAIL(CPRA_ERR_HIP, "side stream: create: %s", hipGetErrorString(e));
    for (int i = 0; i < 2; ++i) {
      e = hipEventCreateWithFlags(&s.ev[i], hipEventDisableTiming);
      if (e != hipSuccess) CPRA_FAIL(CPRA_ERR_HIP, "side stream: event: %s", hipGetErrorString(e));
    }
    it = g_side.emplace(dev, s).first;
  }
  *out = &it->second;
  return CPRA_OK;
}
}  // namespace

// The side stream for work enqueued on `main`, or null: it forks in a captured graph,
// where a fork is an edge between nodes (a step of a 3-layer network, N = 100,000:
// 1.24 ms, on one stream 1.26; 10,000 nodes, 2x256: 0.214 and 0.225).  An eager fork and
// join cost 20 to 80 us of event traffic between the streams, which the overlap rarely
// pays for.  Eager steps, forked and on one stream, us: 3 layers of 128, N = 100,000 1,204
// and 1,173; 2x256, N = 10,000 209 and 206; 4 layers of 128, N = 50,000 638 and 618;
// 6 layers of 64, N = 20,000 372 and 316.  A backward alone: 637 and 593; 103 and 106;
// 284 and 308; 281 and 198; over 52 shapes of one to three layers 0.96 to 1.35 times as
// long with the fork, with no order in depth or size.  The environment is read at every
// call, so that a caller can capture either kind.
cpra_status side_stream_for(hipStream_t main, SideStream** out) {
  *out = nullptr;
  const char* e = getenv("CPRA_OVERLAP");
  if (e != nullptr && e[0] == '0') return CPRA_OK;
  SideStream* side = nullptr;
  CPRA_CHECK(get_side_stream(&side));  // created by the first step, eager or captured
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (main != nullptr && hipStreamIsCapturing(main, &cs) == hipSuccess && cs == hipStreamCaptureStatusActive)
    *out = side;  // (the null stream cannot be captured)
  return CPRA_OK;
}

cpra_status fork_mark(SideStream* s, hipStream_t main) {
  const hipError_t e = hipEventRecord(s->ev[0], main);
  if (e != hipSuccess) CPRA_FAIL(CPRA_ERR_HIP, "fork mark: %s", hipGetErrorString(e));
  return CPRA_OK;
}

cpra_status fork_wait(SideStream* s) {
  const hipError_t e = hipStreamWaitEvent(s->stream, s->ev[0], 0);
  if (e != hipSuccess) CPRA_FAIL(CPRA_ERR_HIP, "fork wait: %s", hipGetErrorString(e));
  return CPRA_OK;
}

cpra_status join_from(SideStream* s, hipStream_t main) {
  hipError_t e = hipEventRecord(s->ev[1], s->stream);
  if (e == hipSuccess) e = hipStreamWaitEvent(main, s->ev[1], 0);
  if (e != hipSuccess) CPRA_FAIL(CPRA_ERR_HIP, "join: %s", hipGetErrorString(e));
  return CPRA_OK;
}

}  // namespace cpra
