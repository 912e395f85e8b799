// Stub items in the cache of decode-step graphs: each knows whether work on it is queued, and a table counts what becomes of
// it.  Compiled and run by test_lease_cache.py; exits non-zero at the first claim that does not hold.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <random>
#include <thread>
#include <vector>

#include "lease_cache.h"

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); std::exit(1); } } while (0)

struct State { std::atomic<int> destroyed{0}, queued{0}, held{0}, waits{0}; };
struct Item {
  State* s;
  explicit Item(State* st) : s(st) {}
  Item(Item&& o) noexcept : s(o.s) { o.s = nullptr; }
  ~Item() {
    if (!s) return;
    CHECK(s->queued == 0 && s->held == 0 && s->destroyed == 0);  // never while in use, never twice
    s->destroyed = 1;
  }
  bool idle() { return s->queued == 0; }
  void wait() { ++s->waits; s->queued = 0; }
};
using Cache = mtmc::LeaseCache<int, Item>;

static void order_of_replacement() {
  std::vector<State> st(8);
  Cache c(3);
  for (int k = 0; k < 3; ++k) c.release(c.insert(k, Item(&st[k])));
  c.release(c.acquire(0));                       // 1 is now the one used longest ago
  c.release(c.insert(3, Item(&st[3])));
  CHECK(st[1].destroyed && !st[0].destroyed && !st[2].destroyed && c.live() == 3);
  CHECK(c.acquire(1) == nullptr);
  for (int k : {0, 2, 3}) {
    Cache::Entry* e = c.acquire(k);
    CHECK(e && e->key == k && e->item.s == &st[k]);
    c.release(e);
  }
}

static void held_or_queued_entries_outlive_their_place() {
  std::vector<State> st(12);
  Cache c(2);
  Cache::Entry* a = c.insert(0, Item(&st[0]));
  st[0].held = 1;
  for (int k = 1; k < 4; ++k) c.release(c.insert(k, Item(&st[k])));  // 0 and 1 have lost their places
  CHECK(!st[0].destroyed && st[1].destroyed && c.retired() == 1);
  CHECK(a->item.s == &st[0]);                    // the holder's entry stays where it was
  st[0].queued = 1;                              // it launches, and lets go
  st[0].held = 0;
  c.release(a);
  c.release(c.insert(4, Item(&st[4])));
  CHECK(!st[0].destroyed && st[0].waits == 0);   // its work is still queued: nobody waits for it
  st[0].queued = 0;
  c.release(c.insert(5, Item(&st[5])));
  CHECK(st[0].destroyed);
}

static void the_number_of_replaced_entries_is_bounded() {
  std::vector<State> st(40);
  Cache c(2);
  for (int k = 0; k < 40; ++k) {
    Cache::Entry* e = c.insert(k, Item(&st[k]));
    st[k].queued = 1;                            // work that never ends by itself
    c.release(e);
    CHECK(c.live() <= 2 && c.retired() <= 2);
  }
  int waits = 0;
  for (int k = 0; k < 40; ++k) waits += st[k].waits;
  CHECK(waits == 36);                            // the oldest one each time, nothing else
  for (int k = 0; k < 36; ++k) CHECK(st[k].destroyed && st[k].waits == 1);
}

static void the_end_waits_for_queued_work() {
  State st[3];
  {
    Cache c(1);
    for (int k = 0; k < 3; ++k) {
      Cache::Entry* e = c.insert(k, Item(&st[k]));
      st[k].queued = 1;
      c.release(e);
    }
  }
  for (State& s : st) CHECK(s.destroyed && s.waits == 1);
}

static void threads() {
  constexpr int kKeys = 10, kThreads = 4, kRounds = 4000;
  std::mutex mu;
  std::vector<State> st((size_t)kThreads * kRounds);
  std::atomic<int> used{0};
  {
    Cache c(3);
    auto work = [&](int seed) {
      std::mt19937 rng(seed);
      for (int i = 0; i < kRounds; ++i) {
        const int key = rng() % kKeys;
        Cache::Entry* e;
        {
          std::lock_guard<std::mutex> lock(mu);
          e = c.acquire(key);
          if (!e) e = c.insert(key, Item(&st[used++]));
          ++e->item.s->held;
        }
        State* s = e->item.s;
        for (int n = rng() % 4; n > 0; --n) {    // launches, outside the lock
          CHECK(e->key == key && !s->destroyed);
          if (rng() % 8 == 0) std::this_thread::yield();
        }
        std::lock_guard<std::mutex> lock(mu);
        --s->held;
        c.release(e);
      }
    };
    std::vector<std::thread> t;
    for (int i = 0; i < kThreads; ++i) t.emplace_back(work, i + 1);
    for (auto& x : t) x.join();
    CHECK(c.live() == 3);
  }
  for (int i = 0; i < used; ++i) CHECK(st[i].destroyed == 1);
}

int main() {
  order_of_replacement();
  held_or_queued_entries_outlive_their_place();
  the_number_of_replaced_entries_is_bounded();
  the_end_waits_for_queued_work();
  threads();
  std::puts("ok");
}
