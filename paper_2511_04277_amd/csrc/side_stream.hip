// A second stream per device and host thread, for work that overlaps the
// caller's stream inside one call (fork and join through events), and the turns
// of resident grids, which an event per device hands on.
#include <unordered_map>

#include "common.h"

namespace rad {
namespace {
thread_local std::unordered_map<int, SideStream> g_side;

struct Turn {
  std::mutex mutex;
  hipEvent_t done = nullptr;  // of the last resident grid
  bool lost = false;          // a grid was enqueued without its event
};
Turn g_turns[64];
}

ResidentTurn::ResidentTurn(hipStream_t s) : s_(s) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    (void)hipGetLastError();
    return;
  }
  Turn& t = g_turns[dev];
  lock_ = std::unique_lock<std::mutex>(t.mutex);
  dev_ = dev;
  if (t.lost) return;
  if (!t.done) {
    if (hipEventCreateWithFlags(&t.done, hipEventDisableTiming) != hipSuccess) {
      (void)hipGetLastError();
      t.done = nullptr;
      return;
    }
    ok_ = true;
    return;
  }
  ok_ = hipStreamWaitEvent(s, t.done, 0) == hipSuccess;  // nothing to wait for on the grid's own stream
  if (!ok_) (void)hipGetLastError();
}

ResidentTurn::~ResidentTurn() {
  if (!ok_ || hipEventRecord(g_turns[dev_].done, s_) == hipSuccess) return;
  (void)hipGetLastError();
  g_turns[dev_].lost = true;
}

hipError_t side_stream(SideStream** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  auto it = g_side.find(dev);
  if (it == g_side.end()) {
    SideStream ss{};
    // default priority; no implicit ordering with the null stream (events order it)
    e = hipStreamCreateWithFlags(&ss.s2, hipStreamNonBlocking);
    if (e != hipSuccess) return e;
    for (hipEvent_t& ev : ss.ev) {
      e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
      if (e != hipSuccess) return e;
    }
    it = g_side.emplace(dev, ss).first;
  }
  *out = &it->second;
  return hipSuccess;
}

}  // namespace rad
