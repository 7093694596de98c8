// Host-link copies on copy engines that the library names itself, ordered by signals.
#pragma once

#include <stdint.h>

#include <vector>

#include "signal_watch.h"

namespace hmy {

// Logical queues: the copies of one run in the order they were submitted.
enum CopyQueue { COPY_IN = 0, COPY_STATE_IN = 1, COPY_OUT = 2, COPY_QUEUES = 3 };

class CopyEngines {
 public:
  // For copies between the device allocation `dev` lies in (current device) and page-locked host memory; nullptr where the
  // runtime does not offer them (the caller then copies through streams).
  static CopyEngines *create(void *dev);
  ~CopyEngines();
  CopyEngines(const CopyEngines &) = delete;
  CopyEngines &operator=(const CopyEngines &) = delete;
  // whether [p, p + bytes) is page-locked host memory these engines reach under its host address
  bool reaches(const void *p, uint64_t bytes) const;
  // A signal at 1, owned by this object; all signals are taken back by recycle(), which the caller may only do when nothing
  // waits for or will set any of them.  nullptr: out of memory.
  Signal take();
  void recycle();
  // Queue a copy that starts once every signal of `deps` has happened and then sets `done`.  False: refused, nothing queued.
  bool copy(CopyQueue q, void *dst, const void *src, uint64_t bytes, const std::vector<Signal> &deps, Signal done);
  static void set(Signal s);            // by the host, in place of a copy
  bool happened(Signal s);              // also where its copy, or one it waited for, has failed: failed() then says so
  bool wait(Signal s);                  // blocks the calling thread; false: a copy has failed
  bool failed();                        // whether any copy since the last recycle() has
  // copies submitted from now on are timed (process-wide, cannot be taken back)
  static void time_copies();
  // seconds on the device's clock of a finished, timed copy; false if it was not timed
  static bool times(Signal s, double *begin, double *end);

 private:
  CopyEngines() {}
  struct Impl;
  Impl *p = nullptr;
};

}  // namespace hmy
