// Pinned host buffers that the tables of a layout go to the device from, and the list of those that released layouts
// leave for the next ones.  The HIP calls it makes are those of Runtime (abi.hip), so that its rules can be tested on the
// CPU.
#pragma once
#include <cstddef>
#include <mutex>
#include <new>

template <class Runtime>
struct UploadStaging {
  void* buffer[2] = {nullptr, nullptr};   // pinned host memory
  size_t capacity[2] = {0, 0};
  typename Runtime::Event done[2] = {};   // recorded behind the copy that reads the buffer
  int device[2] = {-1, -1};               // ... which each was created on: streams of another one refuse it
  bool in_use[2] = {false, false};
  int next = 0;
  bool unrecorded = false;                // a buffer may be read by a copy that its event does not stand behind: a replay, or one refused an event

  ~UploadStaging() {
    for (int i = 0; i < 2; ++i) {
      if (in_use[i]) Runtime::wait(done[i]);
      if (done[i]) Runtime::destroy(done[i]);
      if (buffer[i]) Runtime::free_host(buffer[i]);
    }
  }
  // both events, where made, belong to `d`
  bool belongs_to(int d) const { return (!done[0] || device[0] == d) && (!done[1] || device[1] == d); }
};

// Staging of released layouts, kept for the next ones: taking and giving back pinned memory costs more (some 150 us a
// layout: a turn of eight steps over sixteen contexts, laid out and released, takes 1.6 ms) than laying a batch out.
// At most kKept of them with buffers of at most kBytes are kept; all are given back when the last block pool is
// destroyed.  The list is an array: giving one back happens where a layout is destroyed and must not allocate.
template <class Staging, class Runtime>
class StagingPool {
 public:
  static constexpr size_t kKept = 4, kBytes = size_t(1) << 20;

  void give(Staging* s) {
    const bool one_device = s->done[0] ? s->belongs_to(s->device[0]) : true;
    if (s->capacity[0] <= kBytes && s->capacity[1] <= kBytes && one_device && !s->unrecorded) {
      const std::lock_guard<std::mutex> hold(lock_);
      if (count_ < kKept) {
        kept_[count_++] = s;   // a copy may still be reading a buffer: its event goes along
        return;
      }
    }
    delete s;
  }

  // One for uploads on `device` whose copies are done (so that its new owner never waits for another layout's stream),
  // or a new one; null if there is no memory for that.
  Staging* take(int device) {
    {
      const std::lock_guard<std::mutex> hold(lock_);
      for (size_t k = 0; k < count_; ++k) {
        Staging* s = kept_[k];
        bool idle = s->belongs_to(device);
        for (int i = 0; i < 2 && idle; ++i) {
          if (s->in_use[i]) {
            // (whatever else the answer is -- not ready, or an event that cannot be asked -- is no error of the launches to come)
            if (Runtime::query(s->done[i])) s->in_use[i] = false;
            else Runtime::forget_error();
          }
          idle = !s->in_use[i];
        }
        if (!idle) continue;
        kept_[k] = kept_[--count_];
        return s;
      }
    }
    return new (std::nothrow) Staging();
  }

  void drain() {
    Staging* all[kKept];
    size_t n = 0;
    {
      const std::lock_guard<std::mutex> hold(lock_);
      for (; count_; ++n) all[n] = kept_[--count_];
    }
    for (size_t k = 0; k < n; ++k) delete all[k];
  }

 private:
  std::mutex lock_;
  Staging* kept_[kKept] = {};
  size_t count_ = 0;
};
