// The steps of a rollout with a stop token, with looks at the stop flags in between.  Host code only.
#pragma once

#include <algorithm>

namespace mtmc {

// Steps 1 .. max_new - 1, `period` at a time, with a look behind each period that is read one period later, so that the GPU never
// waits for the host: the call ends when no row runs any more, and else can pack those that do.  With error codes, 0 if there is none:
//   steps(n)   queues n steps
//   look()     queues a look behind them
//   read(&n)   waits for the look and gives what it has seen: rows that run, an upper bound by then (rows only ever finish)
//   pack(n)    n rows are still running
// and settle() waits for the look without an answer.  The place that a look is written to is the next call's, on whatever stream:
// no look is left to be written when this returns.  One that nobody would read is not queued, and where an error ends
// the call the last one is waited for.
template <class Steps, class Look, class Read, class Pack, class Settle>
int run_with_looks(int max_new, int period, Steps steps, Look look, Read read, Pack pack, Settle settle) {
  struct Pending {
    Settle& settle;
    bool is;
    ~Pending() {
      if (is) settle();
    }
  } pending{settle, false};
  for (int i = 1; i < max_new;) {
    const int n = std::min(period, max_new - i);
    if (int rc = steps(n)) return rc;
    i += n;
    if (pending.is) {
      int live = 0;
      if (int rc = read(&live)) return rc;
      pending.is = false;
      if (live <= 0) return 0;
      if (int rc = pack(live)) return rc;
    }
    if (i + period < max_new) {
      pending.is = true;  // ahead of look(), which may fail with the look on its way
      if (int rc = look()) return rc;
    }
  }
  return 0;
}

}  // namespace mtmc
