// readback.hpp -- the host's side of the counters' readbacks (k_publish): every
// readback has a number, which arrives in pinned memory after its words.  No
// HIP in here: the wait for the device is the caller's.
#pragma once
#include <stdint.h>

#include <chrono>

namespace lt {

struct ReadSeq {
  uint64_t seq;    // number of the last readback that arrived (written by the device)
  uint64_t asked;  // number of the last one enqueued (the host's)
};

struct ReadTicket {
  uint64_t seen, want;
};

enum class ReadEnd { arrived, failed, missing };

inline uint64_t read_seq(const ReadSeq* r) { return __atomic_load_n(&r->seq, __ATOMIC_ACQUIRE); }

// To be called before a readback is enqueued, whether that succeeds or not: one
// that was enqueued after all, or whose wait failed, may still arrive later and
// must not be taken for the next one.
inline ReadTicket read_expect(ReadSeq* r) { return ReadTicket{read_seq(r), ++r->asked}; }

// Waits for that readback.  A short wait watches for its number; a long one, or
// one that cannot end (a stream being captured, a device error), is sync's
// (returns true once all work enqueued so far has ended).  sync also sets the
// count right where a number was asked for and never enqueued.
template <class Sync>
ReadEnd read_await(ReadSeq* r, ReadTicket t, std::chrono::nanoseconds watch, Sync&& sync) {
  const auto start = std::chrono::steady_clock::now();
  do {
    for (int i = 0; i < 64; ++i)
      if (read_seq(r) == t.want) return ReadEnd::arrived;
  } while (std::chrono::steady_clock::now() - start <= watch);
  if (!sync()) return ReadEnd::failed;
  const uint64_t now = read_seq(r);
  if (now == t.seen) return ReadEnd::missing;
  r->asked = now;
  return ReadEnd::arrived;
}

}  // namespace lt
