// Pinned host memory that kernels write records into and the host reads, and
// when such memory may be asked for another record.  Host code only.
#pragma once

#include <stdint.h>

namespace spg {

// A kernel writes the words of its record and then the token of the request,
// which the host waits for.  A call may end without that wait (an allocation
// or a launch failed meanwhile), and its kernel may still be queued: the
// next request, possibly on a stream that nothing orders behind it, must not
// get the same memory until that kernel's token has come.
struct Mailbox {
  uint64_t *token = nullptr;  // in pinned memory, 0 at first
  uint64_t asked = 0;         // token of the latest request

  bool arrived(uint64_t t) const { return __atomic_load_n(token, __ATOMIC_ACQUIRE) == t; }
  // no kernel is still to write here
  bool idle() const { return arrived(asked); }
  uint64_t request() { return ++asked; }
};

}  // namespace spg
