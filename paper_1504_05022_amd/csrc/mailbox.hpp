// Pinned host memory that kernels write records into and the host reads, and
// when such memory may be asked for another record.  Host code only.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <chrono>
#include <mutex>
#include <new>

namespace spg {

// A kernel writes the words of its record and then the token of the request,
// which the host waits for.  A call may end without that wait (an allocation
// or a launch failed meanwhile), and its kernel may still be queued: the
// next request, possibly on a stream that nothing orders behind it, must not
// get the same memory until that kernel's token has come.
struct Mailbox {
  void *mem = nullptr;        // pinned memory, zeroed at first
  uint64_t *token = nullptr;  // in it
  uint64_t asked = 0;         // token of the latest request
  Mailbox *next = nullptr;    // in its pool

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

// Mailboxes for the calls of every thread, given back when the call or its
// thread ends, so that threads leave nothing behind (allocating pinned memory
// is far too slow to do it per call).  At most kKeep idle ones are kept; of
// those left by failed calls, whose kernels or copies may yet write, at most
// kLeft are replaced: take() then gives none, and records go by copy.
class MailboxPool {
 public:
  static constexpr int kKeep = 64, kLeft = 16;

  // token_at: offset of the token in the memory of a mailbox; alloc: zeroed
  // pinned memory, nullptr if there is none
  MailboxPool(size_t bytes, size_t token_at, void *(*alloc)(size_t), void (*release)(void *))
      : bytes_(bytes), token_at_(token_at), alloc_(alloc), release_(release) {}

  Mailbox *take() {
    {
      std::lock_guard<std::mutex> lk(mu_);
      for (Mailbox **at = &free_; *at; at = &(*at)->next) {
        Mailbox *b = *at;
        if (!b->idle()) continue;
        *at = b->next;
        --count_;
        return b;
      }
      if (count_ >= kLeft) return nullptr;  // none of them idle
    }
    Mailbox *b = new (std::nothrow) Mailbox();
    if (b) b->mem = alloc_(bytes_);
    if (b && !b->mem) {
      delete b;
      b = nullptr;
    }
    if (b) b->token = reinterpret_cast<uint64_t *>(static_cast<char *>(b->mem) + token_at_);
    return b;
  }

  void give(Mailbox *b) {
    if (!b) return;
    {
      std::lock_guard<std::mutex> lk(mu_);
      if (count_ < kKeep || !b->idle()) {
        b->next = free_;
        free_ = b;
        ++count_;
        return;
      }
    }
    release_(b->mem);
    delete b;
  }

 private:
  const size_t bytes_, token_at_;
  void *(*const alloc_)(size_t);
  void (*const release_)(void *);
  std::mutex mu_;
  Mailbox *free_ = nullptr;
  int count_ = 0;
};

// The mailbox that stays with a thread from one of its calls to the next
// (taking it from the pool in every call: 54 instead of 51 us for a product of
// two reads and seven launches).
struct KeptMailbox {
  MailboxPool &pool;
  Mailbox *box = nullptr;
  bool lent = false;  // to a call of the thread that has not ended
  explicit KeptMailbox(MailboxPool &p) : pool(p) {}
  ~KeptMailbox() { pool.give(box); }
};

// A mailbox for the length of a call: the thread's own, or another while
// that one is taken or an earlier kernel may still write to it.
class MailboxLease {
 public:
  explicit MailboxLease(MailboxPool &pool, KeptMailbox *kept = nullptr)
      : box(nullptr), pool_(pool), kept_(kept && !kept->lent ? kept : nullptr) {
    if (kept_) {
      kept_->lent = true;
      box = kept_->box;
      if (box && !box->idle()) {
        pool.give(box);
        box = nullptr;
      }
    }
    if (!box) box = pool.take();
  }
  ~MailboxLease() {
    if (!kept_) {
      pool_.give(box);
      return;
    }
    kept_->box = box;
    kept_->lent = false;
  }
  MailboxLease(const MailboxLease &) = delete;
  MailboxLease &operator=(const MailboxLease &) = delete;

  Mailbox *box;  // nullptr: none to be had

 private:
  MailboxPool &pool_;
  KeptMailbox *kept_;
};

}  // namespace spg
