// Sums of slices: each slice once, in order, all asked for before the first is added, whatever their number.
// Compiled and run by test_slices.py; exits non-zero at the first number that does not hold.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "slices.h"

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s (n %d)\n", __LINE__, #x, n); std::exit(1); } } while (0)

static int added;
struct Sum {
  float v;
  Sum operator+(const Sum& o) const {
    ++added;
    return {v + o.v};
  }
};

int main() {
  for (int n = 0; n <= mtmc::kMaxSlices; ++n) {
    // values of which every other order of the sums gives another result
    std::vector<float> slice;
    for (int s = 0; s < n; ++s) slice.push_back((s % 2 ? -1.f : 1.f) * (1.0e8f / (s + 1) + 0.37f * s));
    float want = 3.1f;
    for (int s = 0; s < n; ++s) want += slice[s];
    std::vector<int> asked;
    added = 0;
    const Sum got = mtmc::add_slices(Sum{3.1f}, n, [&](int s) {
      CHECK(added == 0);
      asked.push_back(s);
      return Sum{slice[s]};
    });
    CHECK(got.v == want && added == n && (int)asked.size() == n);
    for (int s = 0; s < n; ++s) CHECK(asked[s] == s);
  }
  std::printf("ok\n");
  return 0;
}
