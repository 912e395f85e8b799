// Threads as the workgroups of launches that wait for each other: some come late, any may lose patience at any time.  Compiled and
// run by test_persistent_turn.py; exits non-zero at the first claim that does not hold.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <thread>
#include <vector>

#include "roll_call.h"

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); std::exit(1); } } while (0)

struct Word {
  std::atomic<uint32_t>* p;
  uint32_t load() const { return p->load(std::memory_order_relaxed); }
  void store(uint32_t v) const { p->store(v, std::memory_order_relaxed); }
  uint32_t add(uint32_t v) const { return p->fetch_add(v, std::memory_order_relaxed); }
  uint32_t either(uint32_t v) const { return p->fetch_or(v, std::memory_order_relaxed); }
  bool swap(uint32_t& seen, uint32_t v) const { return p->compare_exchange_strong(seen, v, std::memory_order_relaxed); }
};

constexpr int kGroups = 4, kFull = 3, kAll = kGroups * kFull, kTops = 2;

struct Launch {
  std::atomic<uint32_t> group[kGroups] = {}, top[kTops] = {}, ended{0}, seats{0}, list{0};
  std::atomic<int> started{0};
  int late[kAll], patience[kAll];   // looks before it comes, looks before it gives up
  int went[kAll], id[kAll], n[kAll];
};

static void idle(int looks) {
  for (int i = 0; i < looks; ++i) std::this_thread::yield();
}
static void counted(Launch& L, int w) {
  if (mtmc::roll_call::count_in(Word{&L.group[w % kGroups]}, kFull, 1))
    for (auto& t : L.top) t.fetch_add(1);
  for (int i = 0;; ++i) {
    if (L.top[w % kTops] >= kGroups) break;
    if (L.ended) { L.went[w] = 0; return; }
    if (i > L.patience[w]) {
      if (mtmc::roll_call::close([&](int g) { return Word{&L.group[g]}; }, kGroups, kFull)) { L.ended = 1; L.went[w] = 0; return; }
      L.patience[w] = 1 << 30;
    }
    std::this_thread::yield();
  }
  L.went[w] = 1;
  // a second phase: the group counts again
  if (mtmc::roll_call::count_in(Word{&L.group[w % kGroups]}, kFull, 2))
    for (auto& t : L.top) t.fetch_add(1);
  while (L.top[w % kTops] < 2 * kGroups) std::this_thread::yield();
}
static void listed(Launch& L, int w) {
  int looks = 0;
  const mtmc::roll_call::Roster r = mtmc::roll_call::join(Word{&L.seats}, Word{&L.list}, kAll, [&] { std::this_thread::yield(); return ++looks > L.patience[w]; });
  L.id[w] = r.id;
  L.n[w] = r.n;
}

int main() {
  std::mt19937 rng(1);
  int ran = 0, given_up = 0, whole = 0, shorter = 0;
  for (int round = 0; round < 1500; ++round) {
    Launch L;
    for (int w = 0; w < kAll; ++w) {
      L.late[w] = rng() % 4 ? 0 : (int)(rng() % 300);
      L.patience[w] = round % 3 == 0 ? 1 << 30 : (int)(rng() % (round % 3 == 1 ? 40 : 2000));
    }
    std::vector<int> patience(L.patience, L.patience + kAll);
    std::vector<std::thread> t;
    for (int w = 0; w < kAll; ++w)
      t.emplace_back([&L, w] {
        L.started.fetch_add(1);
        while (L.started < kAll) std::this_thread::yield();
        idle(L.late[w]);
        const int patience = L.patience[w];
        counted(L, w);
        L.patience[w] = patience;
        listed(L, w);
      });
    for (auto& x : t) x.join();
    int went = 0, on = 0, n = 0;
    bool seen[kAll] = {};
    for (int w = 0; w < kAll; ++w) {
      went += L.went[w];
      if (L.id[w] < 0) continue;
      ++on;
      CHECK(L.id[w] < kAll && !seen[L.id[w]]);
      seen[L.id[w]] = true;
      CHECK(n == 0 || n == L.n[w]);
      n = L.n[w];
    }
    CHECK(went == 0 || went == kAll);             // all of them or none
    CHECK(went == 0 || L.ended == 0);
    CHECK(on >= 1 && on == n && (int)L.list == n);  // everybody on the list knows its length
    for (int i = 0; i < n; ++i) CHECK(seen[i]);
    if (round % 3 == 0) CHECK(went == kAll && n == kAll);
    ++(went ? ran : given_up);
    ++(n == kAll ? whole : shorter);
  }
  CHECK(ran > 500 && given_up > 20 && whole > 500 && shorter > 20);
  std::printf("ok\n");
  return 0;
}
