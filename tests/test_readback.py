"""The host's side of the counters' readbacks (csrc/readback.hpp), with the
device played by a thread of the host: a readback left behind by a wait that
failed, or by an enqueueing that reported an error, is never taken for the one
that is waited for."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <atomic>
#include <cstdio>
#include <thread>
#include "readback.hpp"
using namespace lt;
using std::chrono::milliseconds;

// The mirror: one word of counters in front of the number, as k_publish writes them.
struct Mirror { uint64_t value; ReadSeq r; };
static Mirror m;
static uint64_t device_reads = 0;

static void arrive(uint64_t value) {   // one readback ends on the device
  __atomic_store_n(&m.value, value, __ATOMIC_RELAXED);
  __atomic_store_n(&m.r.seq, ++device_reads, __ATOMIC_RELEASE);
}
static uint64_t value() { return __atomic_load_n(&m.value, __ATOMIC_RELAXED); }

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main() {
  const auto never = [] { return false; };
  const auto unused = [] { std::printf("synchronized\n"); return false; };
  // at once, while it is watched for, and after the watching (by the wait)
  ReadTicket t = read_expect(&m.r);
  arrive(10);
  CHECK(read_await(&m.r, t, milliseconds(1), unused) == ReadEnd::arrived && value() == 10);
  t = read_expect(&m.r);
  std::thread later([] { std::this_thread::sleep_for(milliseconds(5)); arrive(11); });
  CHECK(read_await(&m.r, t, milliseconds(5000), unused) == ReadEnd::arrived && value() == 11);
  later.join();
  t = read_expect(&m.r);
  CHECK(read_await(&m.r, t, milliseconds(0), [] { arrive(12); return true; }) == ReadEnd::arrived && value() == 12);
  // a wait that fails; its readback arrives while the next one is watched for
  t = read_expect(&m.r);
  CHECK(read_await(&m.r, t, milliseconds(0), never) == ReadEnd::failed);
  t = read_expect(&m.r);
  std::atomic<bool> both{false};
  std::thread dev([&] {
    arrive(13);
    std::this_thread::sleep_for(milliseconds(20));
    both = true;
    arrive(14);
  });
  ReadEnd e = read_await(&m.r, t, milliseconds(5000), unused);
  const bool early = !both;
  const uint64_t got = value();
  dev.join();
  CHECK(e == ReadEnd::arrived && !early && got == 14);
  // an enqueueing that reports an error and arrives all the same
  read_expect(&m.r);
  arrive(15);
  t = read_expect(&m.r);
  CHECK(read_await(&m.r, t, milliseconds(0), [] { arrive(16); return true; }) == ReadEnd::arrived && value() == 16);
  // one that was never enqueued (a capture given up): the next two arrive, the
  // second without a synchronization
  read_expect(&m.r);
  t = read_expect(&m.r);
  arrive(17);
  CHECK(read_await(&m.r, t, milliseconds(0), [] { return true; }) == ReadEnd::arrived && value() == 17);
  t = read_expect(&m.r);
  arrive(18);
  CHECK(read_await(&m.r, t, milliseconds(1), unused) == ReadEnd::arrived && value() == 18);
  // the device came to rest without it
  t = read_expect(&m.r);
  CHECK(read_await(&m.r, t, milliseconds(0), [] { return true; }) == ReadEnd::missing);
  std::printf("ok\n");
  return 0;
}
"""


def test_readbacks_are_told_apart(tmp_path):
    src, exe = tmp_path / "readback.cpp", tmp_path / "readback"
    src.write_text(SRC)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-pthread", "-I",
                    os.path.join(ROOT, "paper_2306_06744_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
