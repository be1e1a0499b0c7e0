"""Host-side rules of the library's sources, compiled with the host compiler:
when pinned memory that a kernel writes may be asked for another record."""
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
    src.write_text(HEAD + "".join('#include "%s"\n' % i for i in includes) + body)
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
