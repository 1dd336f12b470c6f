// Device buffers that overlapping calls, each on a stream of its own, use in turn.
#pragma once

#include <hip/hip_runtime.h>

#include <mutex>

namespace scan {

struct TurnState {
  std::mutex lock;
  int inflight = 0;         // calls that have not left
  hipEvent_t ev = nullptr;  // after the work of the last call to come
};

// One call's turn: work enqueued on s between the constructor and enqueued()
// starts after the work of the calls that came before.  Each call records the
// event on its own stream, from its own thread, and the next one waits for the
// event: a stream handle of another call's means nothing by then (its stream may
// be destroyed, and hipStreamPerThread is another stream in each thread).
// hold: a call that finds no other there keeps the lock until it leaves, and the
// event is not recorded (of 123 us a clustering of 2,000 vertices takes, 3); the
// call that had to wait for the lock records, so that calls which go on
// overlapping queue on the device.
class Turn {
 public:
  Turn(TurnState& t, hipStream_t s, bool hold) : t_(t), s_(s), lk_(t.lock, std::try_to_lock), hold_(hold) {
    if (!lk_.owns_lock()) {
      lk_.lock();
      hold_ = false;
    }
    if (t_.inflight > 0) {
      hold_ = false;
      err_ = hipStreamWaitEvent(s_, t_.ev, 0);
    }
    ++t_.inflight;
  }
  Turn(const Turn&) = delete;
  Turn& operator=(const Turn&) = delete;

  hipError_t error() const { return err_; }

  // Everything is on the stream.
  hipError_t enqueued() {
    if (hold_) return hipSuccess;
    err_ = hipEventRecord(t_.ev, s_);
    if (err_ == hipSuccess) lk_.unlock();
    return err_;
  }

  // The stream has been waited for since.
  void done() { done_ = true; }

  // (A call that failed on the way may have left work on its stream.)
  ~Turn() {
    if (!done_) (void)hipStreamSynchronize(s_);
    if (!lk_.owns_lock()) lk_.lock();
    --t_.inflight;
  }

 private:
  TurnState& t_;
  hipStream_t s_;
  std::unique_lock<std::mutex> lk_;
  bool hold_;
  hipError_t err_ = hipSuccess;
  bool done_ = false;
};

}  // namespace scan
