// When the memory of a compression plan may be used again (asc.hip).  No HIP header: the CPU test compiles it with
// events and queues of its own.
#pragma once

#include <cstddef>
#include <thread>

namespace reslim {

// The work that may still read a block: one event per queue that launched some, each recorded after the latest of it.
// Gpu has the types Event and Stream and the functions create, wait, record (false: failed), done, and per_thread,
// which says that a handle names another queue in every thread.
//
// A handle alone is not a queue: the per-thread handle is one value in all threads, and a destroyed stream's value may
// come back for a new one.  The first is told apart by the thread.  For the second the new queue waits for the old mark
// before the mark is overwritten, which the same queue has done anyway, being in order: whatever the handle stands for by now,
// an event that has happened says that all work marked under it is finished.
template <class Gpu>
struct UseMarks {
  static constexpr int kMost = 4;
  typename Gpu::Event ev[kMost] = {};      // kept from use to use
  typename Gpu::Stream stream[kMost] = {};
  std::thread::id thread[kMost];
  int n = 0;

  // the work on `st` so far reads the block; false: that cannot be marked (too many queues, or an error)
  bool add(typename Gpu::Stream st) {
    const std::thread::id self = Gpu::per_thread(st) ? std::this_thread::get_id() : std::thread::id();
    int i = 0;
    while (i < n && !(stream[i] == st && thread[i] == self)) ++i;
    if (i == kMost) return false;
    if (i < n ? !Gpu::wait(st, ev[i]) : !ev[i] && !Gpu::create(&ev[i])) return false;
    if (!Gpu::record(ev[i], st)) return false;
    stream[i] = st;
    thread[i] = self;
    n = i < n ? n : i + 1;
    return true;
  }
  bool done() const {
    for (int i = 0; i < n; ++i)
      if (!Gpu::done(ev[i])) return false;
    return true;
  }
};

// Which of the n kept blocks (oldest first) a plan of `bytes` takes, -1: none, it gets a new one.  A new block or one too
// small costs an allocation, a block given up also a wait for the whole device: the smallest finished block that is large
// enough; else a new one while fewer than `most` are kept; else the smallest finished one, which is replaced; with all
// of them still in use the oldest that is large enough, or the oldest, is waited for.
struct KeptBlock {
  size_t cap;
  bool done;
};
inline int choose_block(const KeptBlock *b, int n, int most, size_t bytes) {
  int fit = -1, least = -1, busy = -1;
  for (int i = 0; i < n; ++i) {
    const bool fits = b[i].cap >= bytes;
    if (b[i].done) {
      if (fits && (fit < 0 || b[i].cap < b[fit].cap)) fit = i;
      if (least < 0 || b[i].cap < b[least].cap) least = i;
    } else if (fits && busy < 0) {
      busy = i;
    }
  }
  if (fit >= 0) return fit;
  if (n < most) return -1;
  return least >= 0 ? least : busy >= 0 ? busy : 0;
}

}  // namespace reslim
