// Pinned host memory that kernels write records into and the host reads, and
// when such memory may be asked for another record.  Host code only.
#pragma once

#include <stdint.h>

#include <chrono>

namespace spg {

// A kernel writes the words of its record and then the token of the request,
// which the host waits for.  A call may end without that wait (an allocation
// or a launch failed meanwhile), and its kernel may still be queued: the
// next request, possibly on a stream that nothing orders behind it, must not
// get the same memory until that kernel's token has come.
struct Mailbox {
  uint64_t *token = nullptr;  // in pinned memory, 0 at first
  uint64_t asked = 0;         // token of the latest request

  // no kernel is still to write here: the record of the latest request came
  bool idle() const { return __atomic_load_n(token, __ATOMIC_ACQUIRE) == asked; }
  uint64_t request() { return ++asked; }
  // the kernel of the latest request was never launched
  void drop() { asked = __atomic_load_n(token, __ATOMIC_ACQUIRE); }
};

// Waits for the record of the latest request (0: it came).  A wait beyond a
// few milliseconds is left to sync(), which waits for the stream and reports
// its errors.  Where the token is missing even then, its kernel was not
// launched: the answer is why(), the error of that launch, which is thereby
// not left behind for a later call.
template <typename Sync, typename Why> int wait_mailbox(Mailbox &box, Sync sync, Why why) {
  const auto t0 = std::chrono::steady_clock::now();
  for (int spin = 0; !box.idle(); ++spin) {
    __builtin_ia32_pause();
    if ((spin & 255) == 255 && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(5)) {
      const int e = sync();
      if (e != 0) return e;
      if (box.idle()) return 0;
      box.drop();
      return why();
    }
  }
  return 0;
}

}  // namespace spg
