// The host's side of a one-kernel PCG solve: plain C++, so that it can be
// driven by a model of the device (tests/sanitize/solve_loop_driver.cpp).
#pragma once

namespace bfal {

// How a one-kernel solve ended; the first two are the values of PcgScalars::done.
enum : int { kEndConverged = 1, kEndMaxIter = 2, kEndBreakdown = 8, kEndAssembly = 16, kEndStuck = 32 };

// The words in pinned memory that the device reports into (PcgSystem::hstat):
// launches made << 32 | end code (0 while the solve runs), the iteration of the
// end, whether the resident kernel found its workgroups not all running, and
// whether one of them gave up waiting for the others (a word of its own: the
// launches queued behind go on reporting into the first).
enum : int { kWordState = 0, kWordIter = 1, kWordApart = 2, kWordStuck = 3, kSolveWords = 4 };

enum class StreamState { kBusy, kIdle, kError };
enum class SolveEnd {
  kEnded,     // the device reported an end: its code is in kWordState
  kStuck,     // a workgroup gave up: the vectors hold no state of the solve
  kError,     // a launch or the stream failed
  kLost,      // all launches are complete and no end was reported
};

// Launches are kept kAhead (kResidentAhead where the resident kernel makes the
// iterations) in front of what the device has reported, so that neither side
// waits and few launches follow the end.
constexpr int kAhead = 12, kResidentAhead = 4;
constexpr int kSpinsPerQuery = 4096;

// Follows a solve to its end.  The device: bool launch(long long number, bool
// resident) makes the next launch, false if it failed (what was to write the
// state that the next launch reads is then missing: no further one may follow);
// StreamState query() of the stream.  Every wait ends: a device that stays
// behind is asked for, and where its stream is idle on two askings with no
// report between that would let the host go on, the solve is lost.  kWordStuck
// is the caller's to clear and to look at once more when the stream has been
// waited for: a workgroup may give up after the solve's leader has gone on.
template <class Device>
SolveEnd follow_solve(Device& dev, volatile unsigned long long* word, bool resident) {
  word[kWordState] = word[kWordIter] = word[kWordApart] = 0;
  long long launched = 0, spins = 0;
  bool idle = false;
  for (;;) {
    const unsigned long long state = word[kWordState];
    const unsigned end = (unsigned)state;
    if (word[kWordStuck] || end == kEndStuck) return SolveEnd::kStuck;
    if (end) return SolveEnd::kEnded;
    if (resident && word[kWordApart]) resident = false;
    if (launched - (long long)(state >> 32) < (resident ? kResidentAhead : kAhead)) {
      if (!dev.launch(launched, resident)) return SolveEnd::kError;
      ++launched;
      spins = 0;
      idle = false;
    } else if (++spins % kSpinsPerQuery == 0) {
      switch (dev.query()) {
        case StreamState::kError: return SolveEnd::kError;
        case StreamState::kBusy: idle = false; break;
        case StreamState::kIdle:
          if (idle) return SolveEnd::kLost;
          idle = true;   // (the words are read once more)
      }
    }
  }
}

}  // namespace bfal
