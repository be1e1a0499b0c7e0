"""Host-side rules of the library's sources, compiled with the host compiler:
pinned memory that kernels write, when it may be asked for another record and
who holds it, and the sizes of launches."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1504_05022_amd", "csrc")

HEAD = r"""
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); exit(1); } } while (0)
"""


def run_cpp(tmp_path, includes, body, *flags):
    """Compile and run a program that checks `body`; fails with what it printed."""
    src = tmp_path / "check.cpp"
    lines = ['#include "%s"\n' % i if i.endswith(".hpp") else "#include <%s>\n" % i for i in includes]
    src.write_text(HEAD + "".join(lines) + body)
    exe = tmp_path / "check"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, *flags, str(src),
                           "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_mailbox_is_not_asked_again_before_its_token(tmp_path):
    """A call that returned without waiting leaves a kernel that may still
    write: its memory is asked again only after that kernel's token."""
    run_cpp(tmp_path, ["mailbox.hpp"], r"""
int main() {
  uint64_t word = 0;
  spg::Mailbox b;
  b.token = &word;
  CHECK(b.idle());
  const uint64_t t1 = b.request();
  CHECK(t1 != 0 && !b.idle());
  word = t1;  // the kernel writes
  CHECK(b.idle());
  const uint64_t t2 = b.request();  // left without a wait
  CHECK(t2 != t1 && !b.idle());
  CHECK(!b.idle());
  word = t2;  // late
  CHECK(b.idle());
}
""")


def test_record_of_a_kernel_that_was_not_launched(tmp_path):
    """The wait reports the launch's error, and takes it away: the thread's
    next call must not find it.  Errors of the stream come first, a record
    that arrives during the wait for the stream is taken."""
    run_cpp(tmp_path, ["mailbox.hpp"], r"""
int main() {
  uint64_t word = 0;
  spg::Mailbox b;
  b.token = &word;
  int last = 9, syncs = 0;  // as left by the failed launch
  auto why = [&] { const int e = last; last = 0; return e; };
  b.request();
  CHECK(spg::wait_mailbox(b, [&] { ++syncs; return 0; }, why) == 9);
  CHECK(syncs == 1 && last == 0 && b.idle());
  b.request();
  CHECK(spg::wait_mailbox(b, [&] { return 7; }, why) == 7 && !b.idle());
  CHECK(spg::wait_mailbox(b, [&] { word = b.asked; return 0; }, why) == 0 && b.idle());
  word = b.request();
  CHECK(spg::wait_mailbox(b, [&] { return 7; }, why) == 0);
}
""")


def test_mailboxes_outlive_threads_and_are_bounded(tmp_path):
    """Threads that end leave their pinned memory to the next ones; a mailbox
    left by a failed call is not handed out before its token and at most a few
    are replaced; beyond what is kept, memory is released."""
    run_cpp(tmp_path, ["mailbox.hpp", "thread", "vector"], r"""
static int made = 0, freed = 0;
static bool full = false;
static void *get(size_t n) { if (full) return nullptr; ++made; return calloc(1, n); }
static void put(void *p) { ++freed; free(p); }
int main() {
  using spg::Mailbox; using spg::MailboxPool;
  MailboxPool pool(512, 504, get, put);
  for (int i = 0; i < 100; ++i)  // one thread after another
    std::thread([&] {
      Mailbox *b = pool.take();
      *b->token = b->request();
      pool.give(b);
    }).join();
  CHECK(made == 1);
  std::vector<Mailbox *> v;  // many calls at once
  for (int i = 0; i < 100; ++i) v.push_back(pool.take());
  CHECK(made == 100);
  for (Mailbox *b : v) pool.give(b);
  CHECK(freed == 100 - MailboxPool::kKeep);
  MailboxPool late(512, 504, get, put);
  made = 0;
  v.clear();
  for (int i = 0; i < MailboxPool::kLeft; ++i) {
    Mailbox *b = late.take();
    for (Mailbox *o : v) CHECK(b != o);
    b->request();  // its kernel has not written when the call ends
    v.push_back(b);
    late.give(b);
  }
  CHECK(made == MailboxPool::kLeft && late.take() == nullptr);
  *v[3]->token = v[3]->asked;  // one kernel writes
  CHECK(late.take() == v[3]);
  *v[3]->token = v[3]->request();
  late.give(v[3]);
  CHECK(late.take() == v[3]);
  made = 0;
  MailboxPool own(512, 504, get, put);
  for (int t = 0; t < 3; ++t)  // a thread keeps its mailbox between calls
    std::thread([&] {
      spg::KeptMailbox kept(own);
      Mailbox *first = nullptr;
      for (int call = 0; call < 3; ++call) {
        spg::MailboxLease lease(own, &kept);
        if (!call) first = lease.box;
        CHECK(lease.box == first);
        spg::MailboxLease inner(own, &kept);  // a call inside this one
        CHECK(inner.box && inner.box != first);
        *first->token = first->request();
      }
    }).join();
  CHECK(made == 2);
  {
    spg::KeptMailbox kept(own);
    Mailbox *a = nullptr;
    {
      spg::MailboxLease lease(own, &kept);
      a = lease.box;
      a->request();  // left without a wait
    }
    spg::MailboxLease lease(own, &kept);
    CHECK(lease.box != a);
  }
  MailboxPool none(512, 504, get, put);
  full = true;
  CHECK(none.take() == nullptr);
}
""", "-pthread")


def test_copy_rows_stay_within_a_launch(tmp_path):
    """Rows per wavefront of the copy into C: as measured up to sizes where
    the launch would reach 2^32 threads, more of them beyond."""
    run_cpp(tmp_path, ["launch_rules.hpp", "initializer_list"], r"""
using spg::copy_rows; using spg::copy_threads;
int main() {
  CHECK(copy_rows(300000, 300000 * 9ll) == 32 && copy_rows(300000, 300000 * 200ll) == 2);
  CHECK(copy_rows(1000, 5000) == 2 && copy_rows(0, 0) == 2);
  for (int64_t rows = 1; rows < (int64_t(1) << 31) - 256; rows = rows * 5 / 4 + 1)
    for (int64_t each : {0ll, 1ll, 9ll, 11ll, 30ll, 81ll, 500ll, 100000ll}) {
      const int r = copy_rows(rows, rows * each);
      CHECK(r == 2 || r == 4 || r == 8 || r == 16 || r == 32);
      CHECK(copy_threads(rows, r) <= 0xffffffffll);
      CHECK(r == 2 || copy_threads(rows, r / 2) > 0xffffffffll || (r * each <= 320 && rows >= 4096ll * r));
    }
  CHECK(copy_rows(1ll << 27, (1ll << 27) * 100) == 4);  // 2: 2^32 threads
}
""")


def test_batch_copy_work_groups(tmp_path):
    """Work-groups per tile of the batch's copy: every place of a full tile,
    one for problems of a few rows, and never 2^32 threads in a launch."""
    run_cpp(tmp_path, ["launch_rules.hpp", "initializer_list"], r"""
using spg::copy_parts;
int main() {
  CHECK(copy_parts(400, 400 * 256, 2, 256) == 32 && copy_parts(400, 400 * 256, 32, 256) == 2);
  CHECK(copy_parts(10000, 10000 * 5, 2, 256) == 1 && copy_parts(10000, 10000, 32, 256) == 1);
  CHECK(copy_parts(1, 0, 2, 256) == 1);
  for (int64_t tiles = 1; tiles < (1 << 24); tiles = tiles * 3 + 1)
    for (int64_t each : {0, 1, 9, 100, 255, 256})
      for (int r : {2, 4, 8, 16, 32}) {
        const int parts = copy_parts(tiles, tiles * each, r, 256);
        CHECK(parts >= 1 && parts * 4 * r <= 256);
        CHECK(tiles * parts * 256 <= 0xffffffffll);
        CHECK(parts == 1 || (parts - 1) * 4 * r < each);
      }
  CHECK(copy_parts(1 << 20, 256ll << 20, 2, 256) == 15);  // 32: beyond a launch
}
""")


def test_gradient_chunks(tmp_path):
    """Entries of A per wavefront: all of a chunk for a large A, fewer for a
    small one as long as they have products to fill a wavefront."""
    run_cpp(tmp_path, ["launch_rules.hpp", "initializer_list"], r"""
using spg::grad_chunk;
int main() {
  CHECK(grad_chunk(128, 6000000, 192000000) == 128 && grad_chunk(64, 600000, 7200000) == 64);
  CHECK(grad_chunk(128, 100, 10000) == 4 && grad_chunk(128, 100, 1000) == 64);
  CHECK(grad_chunk(64, 1, 1000000) == 1 && grad_chunk(64, 1000, 0) == 64);
  for (int64_t nnz = 1; nnz < (int64_t(1) << 31); nnz = nnz * 3 + 1)
    for (int64_t each : {0ll, 1ll, 5ll, 100ll, 100000ll}) {
      const int ch = grad_chunk(128, nnz, nnz * each);
      CHECK(ch >= 1 && ch <= 128 && (ch == 128 || (nnz < 4096ll * ch && ch * each >= 384)));
    }
}
""")


def test_joined_capacity_classes(tmp_path):
    """Classes with few rows join the next one with rows within eight times
    their capacity, in chains; a kernel takes neighbouring classes only, and
    at most 2048 rows below its own capacity."""
    run_cpp(tmp_path, ["launch_rules.hpp", "stdlib.h"], r"""
using spg::join_classes;
int main() {
  const int cap[11] = {1, 2, 4, 8, 16, 32, 64, 128, 256, 512, 1024};
  int to[11];
  int64_t chain[11] = {100, 0, 0, 100, 0, 0, 100, 0, 0, 100, 0};
  join_classes(11, chain, cap, to);
  CHECK(to[0] == 9 && to[3] == 9 && to[6] == 9 && to[9] == 9);
  int64_t gap[11] = {100, 0, 0, 0, 100, 0, 0, 0, 0, 0, 5};
  join_classes(11, gap, cap, to);
  CHECK(to[0] == 0 && to[4] == 4 && to[10] == 10);
  int64_t many[11] = {2000, 100, 100, 3000, 0, 0, 0, 0, 0, 0, 0};
  join_classes(11, many, cap, to);
  CHECK(to[0] == 1 && to[1] == 1 && to[2] == 3 && to[3] == 3);
  for (int r = 0; r < 20000; ++r) {
    int64_t rows[11];
    for (auto &x : rows) x = rand() % 3 ? rand() % 1500 : rand() % 2 * 5000;
    join_classes(11, rows, cap, to);
    for (int d = 0; d < 11; ++d) {
      int64_t below = 0;
      int first = d;
      for (int c = d - 1; c >= 0; --c)
        if (to[c] == d) {
          below += rows[c];
          first = c;
        }
      CHECK(below <= spg::kFewRows && (below == 0 || to[d] == d) && to[d] >= d);
      for (int c = first; c < d; ++c) CHECK(to[c] == d || rows[c] == 0);
    }
  }
}
""")
