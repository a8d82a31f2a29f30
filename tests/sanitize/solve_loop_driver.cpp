// The host's loop of a one-kernel solve (csrc/solve_loop.h) against a model of
// the device: launches that fail, a stream that fails, reports that never come,
// a device that answers only when it is asked, workgroups that do not all run.
// A loop that spins for ever is ended by the model.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "../../paper_2512_12151_amd/csrc/solve_loop.h"

using namespace bfal;

namespace {

int failures = 0;
#define EXPECT(cond)                                                          \
  do {                                                                        \
    if (!(cond)) {                                                            \
      std::printf("%s:%d: %s: %s\n", __FILE__, __LINE__, name, #cond);        \
      ++failures;                                                             \
    }                                                                         \
  } while (0)

constexpr long long kNever = 1LL << 40;

struct Model {
  volatile unsigned long long word[kSolveWords] = {7, 7, 7, 0};   // a solve before this one left them (the last is the caller's)
  long long end_at = kNever;      // the launch that ends the solve
  long long fail_at = kNever;     // the launch that fails
  long long silent_at = kNever;   // from this launch on nothing is reported
  long long stuck_at = kNever;    // the launch whose workgroups lose each other; those behind it report all the same
  long long apart_at = kNever;    // the launch that finds its workgroups not all running
  int query_error_after = 1 << 30;
  bool lazy = false;              // launches run when the stream is asked, and not before
  bool busy = false;              // the stream is never idle

  long long asked = 0, ran = 0, tried = 0;
  int queries = 0;
  bool failed = false, resident = false, resident_at_end = false;

  void run_queued() {
    for (; ran < asked; ++ran) {
      if (ran == apart_at) word[kWordApart] = 1;
      if (ran == stuck_at) {
        word[kWordStuck] = 1;
        continue;
      }
      if (ran >= silent_at) continue;
      if (ran == end_at) word[kWordIter] = 41;
      const int mask = resident ? 0 : 3;
      const bool end = ran >= end_at;
      if (end || !((ran + 1) & mask)) word[kWordState] = (unsigned long long)(ran + 1) << 32 | (end ? kEndConverged : 0);
    }
  }
  bool launch(long long number, bool res) {
    ++tried;
    resident = resident_at_end = res;
    if (number != asked || failed) std::abort();   // one after the other, and none after a failed one
    if (number == fail_at) {
      failed = true;
      return false;
    }
    ++asked;
    if (!lazy) run_queued();
    return true;
  }
  StreamState query() {
    if (++queries > 10000) {
      std::printf("the loop does not end\n");
      std::exit(1);
    }
    if (queries > query_error_after) return StreamState::kError;
    run_queued();
    return busy && queries < 1000 ? StreamState::kBusy : StreamState::kIdle;
  }
};

}  // namespace

int main() {
  for (bool resident : {false, true})
    for (bool lazy : {false, true}) {
      for (long long end_at : {0, 1, 2, 3, 4, 11, 12, 13, 40, 1000}) {
        const char* name = "end";
        Model m;
        m.end_at = end_at;
        m.lazy = lazy;
        EXPECT(follow_solve(m, m.word, resident) == SolveEnd::kEnded);
        EXPECT(m.word[kWordIter] == 41 && (unsigned)m.word[kWordState] == kEndConverged);
        EXPECT(m.asked >= end_at + 1 && m.asked <= end_at + 1 + (resident ? kResidentAhead : kAhead));
      }
      for (long long fail_at : {0, 1, 3, 4, 12, 57}) {
        const char* name = "failed launch";
        Model m;
        m.fail_at = fail_at;
        m.lazy = lazy;
        EXPECT(follow_solve(m, m.word, resident) == SolveEnd::kError);
        EXPECT(m.tried == fail_at + 1);
      }
      for (long long silent_at : {0, 1, 5, 100}) {
        const char* name = "no report";
        Model m;
        m.silent_at = silent_at;
        m.lazy = lazy;
        EXPECT(follow_solve(m, m.word, resident) == SolveEnd::kLost);
        EXPECT(m.queries < 1000);
      }
      {
        const char* name = "no report, busy for some time";
        Model m;
        m.silent_at = 20;
        m.lazy = lazy;
        m.busy = true;
        EXPECT(follow_solve(m, m.word, resident) == SolveEnd::kLost);
      }
      {
        const char* name = "stream error";
        Model m;
        m.silent_at = 9;
        m.lazy = lazy;
        m.query_error_after = 3;
        m.busy = true;
        EXPECT(follow_solve(m, m.word, resident) == SolveEnd::kError);
      }
    }
  for (bool lazy : {false, true})
    for (long long end_at : {kNever, 6LL, 7LL, 9LL}) {   // (a mixed state that seems to have converged, too)
      const char* name = "stuck";
      Model m;
      m.stuck_at = 5;   // (not the last of the launches that are queued together)
      m.end_at = end_at;
      m.lazy = lazy;
      EXPECT(follow_solve(m, m.word, true) == SolveEnd::kStuck);
      EXPECT(m.asked <= 6 + kResidentAhead);
    }
  for (bool lazy : {false, true}) {
    const char* name = "apart";
    Model m;
    m.apart_at = 5;
    m.end_at = 300;
    m.lazy = lazy;
    EXPECT(follow_solve(m, m.word, true) == SolveEnd::kEnded);
    EXPECT(!m.resident_at_end && m.asked >= 301);
  }
  if (failures) return 1;
  std::printf("all checks passed\n");
  return 0;
}
