// What becomes of signals whose copy fails (plain C++: nothing of HIP or HSA).
#pragma once

#include <stdint.h>

#include <atomic>
#include <chrono>
#include <condition_variable>
#include <mutex>
#include <thread>
#include <vector>

namespace hmy {

// A signal is a 64-bit word, 1 until what it stands for has happened, then 0: written by a copy engine at the end of a
// copy, by k_signal (engine.hip) where a stream reaches it; waited for by copy engines, streams (hipStreamWaitValue64)
// and the host.  A copy that fails leaves a negative value.
typedef uint64_t *Signal;

// Copy engines and streams wait for exactly 0, so whatever waits for a failed copy would wait for good, and with it, in the
// end, the host thread that enqueues.  So a thread of its own looks at the signals in use every millisecond: where it finds
// a negative value it notes the failure and then stores the 0 itself, so that all that has been queued behind runs to its
// end (on data nobody uses: whoever sees that 0 sees the failure too).
class SignalWatch {
 public:
  // store: puts a value into a signal and wakes those that wait for it
  explicit SignalWatch(void (*store)(Signal, int64_t)) : store_(store) {}
  ~SignalWatch() {
    {
      std::lock_guard<std::mutex> lk(mu_);
      stop_ = true;
    }
    wake_.notify_one();
    if (thread_.joinable()) thread_.join();
  }
  SignalWatch(const SignalWatch &) = delete;
  SignalWatch &operator=(const SignalWatch &) = delete;

  void add(Signal s) {   // watched until clear()
    bool idle;
    {
      std::lock_guard<std::mutex> lk(mu_);
      idle = first_ == in_use_.size();
      in_use_.push_back(s);
      if (!thread_.joinable()) thread_ = std::thread([this] { run(); });   // only where there is something to watch
    }
    if (idle) wake_.notify_one();
  }
  // forgets signals and failures; nothing may wait for or will set any of them
  void clear() {
    std::lock_guard<std::mutex> lk(mu_);
    in_use_.clear();
    first_ = 0;
    failed_.store(false);
  }
  // whether what the signal stands for is over, well or not
  bool over(Signal s) {
    const int64_t v = value(s);
    if (v < 0) give_up(s);
    return v < 1;
  }
  // looks at every signal now; true: no copy has failed
  bool settle() {
    std::lock_guard<std::mutex> lk(mu_);
    look();
    return !failed();
  }
  bool failed() const { return failed_.load(std::memory_order_acquire); }

 private:
  static int64_t value(Signal s) { return int64_t(__atomic_load_n(s, __ATOMIC_ACQUIRE)); }
  void give_up(Signal s) {
    failed_.store(true, std::memory_order_release);   // before the 0: see above
    store_(s, 0);
  }
  void look() {
    for (size_t i = first_; i < in_use_.size(); ++i) {
      const int64_t v = value(in_use_[i]);
      if (v < 0) give_up(in_use_[i]);
      if (v < 1 && i == first_) ++first_;   // they are over in about the order they were taken
    }
  }
  void run() {
    std::unique_lock<std::mutex> lk(mu_);
    while (!stop_) {
      look();
      if (first_ == in_use_.size()) wake_.wait(lk, [&] { return stop_ || first_ != in_use_.size(); });
      else wake_.wait_for(lk, std::chrono::milliseconds(1), [&] { return stop_; });
    }
  }

  void (*store_)(Signal, int64_t);
  std::mutex mu_;
  std::condition_variable wake_;
  std::vector<Signal> in_use_;
  size_t first_ = 0;   // everything before it is over
  bool stop_ = false;
  std::atomic<bool> failed_{false};
  std::thread thread_;
};

}  // namespace hmy
