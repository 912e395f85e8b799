// The looks at the stop flags of a rollout: where they lie, what is read of them, and that none is left to be written when the call
// returns, for its place is the next call's.  The device is made up: it comes to a look when somebody waits for it.
// Compiled and run by test_stop_looks.py; exits non-zero at the first call that does not hold.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "stop_looks.h"

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s (max_new %d, period %d, ends %d, fails %d)\n", __LINE__, #x, max_new, period, ends, fails); std::exit(1); } } while (0)

// Rows run before step `ends`; the operation number `fails` gives an error.  Number of operations.
static int check(int max_new, int period, int ends, int fails) {
  int queued = 1, ops = 0, looked = 0, looks = 0, reads = 0, packs = 0;
  bool under_way = false, ended = false;
  auto rc = [&] { return ++ops == fails ? -7 : 0; };
  auto steps = [&](int n) {
    CHECK(n >= 1 && n <= period);
    queued += n;
    return rc();
  };
  auto look = [&] {
    CHECK(!under_way);  // one place
    under_way = true;
    looked = queued;
    ++looks;
    return rc();
  };
  auto read = [&](int* live) {
    CHECK(under_way && queued > looked);  // the GPU has steps to go on with
    const int r = rc();
    if (r) return r;
    under_way = false;
    ++reads;
    *live = looked < ends ? 3 : 0;
    ended = *live == 0;
    return 0;
  };
  auto pack = [&](int live) {
    CHECK(live == 3 && !under_way);
    ++packs;
    return rc();
  };
  auto settle = [&] { under_way = false; };
  const int r = mtmc::run_with_looks(max_new, period, steps, look, read, pack, settle);
  CHECK(!under_way);
  CHECK(r == (fails >= 1 && fails <= ops ? -7 : 0));
  if (r == 0) {
    CHECK(looks == reads && packs == reads - ended);
    CHECK(ended ? queued - ends < 3 * period && queued < max_new : queued == max_new);
    // a period that a further one follows is looked behind, until one says that nobody runs
    int want = 0;
    for (int i = 1 + period; i + period < max_new; i += period) {
      ++want;
      if (i >= ends) break;
    }
    CHECK(looks == want);
  }
  return ops;
}

int main() {
  for (int max_new = 1; max_new <= 40; ++max_new)
    for (int period : {1, 2, 3, 4, 8, 19, 20, 32, 39, 40, 1 << 20})
      for (int ends = 1; ends <= max_new + 1; ++ends) {
        const int n = check(max_new, period, ends, 0);
        for (int fails = 1; fails <= n; ++fails) check(max_new, period, ends, fails);
      }
  std::printf("ok\n");
  return 0;
}
