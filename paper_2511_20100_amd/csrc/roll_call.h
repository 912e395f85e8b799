// Whether the workgroups of a launch that wait for each other are all there.  A workgroup takes a place on the device when one
// is free, and what holds it (another stream's kernel, another process) may itself wait; so no launch may count on all of
// them.  Two forms, both decided once, for all workgroups alike, by memory that only atomics touch; zero before the launch.
//
//   counted groups  the launch needs all of them: each counts itself into its group of `full`, and what is behind the first
//                   wait runs once every group is full.  Whoever has waited too long closes a group that is not: it never fills, so nobody gets
//                   past that wait, then or later.
//   roster          the launch runs with those that are there: each takes a number, and the list is closed when it is complete
//                   or somebody has waited too long.  Whoever comes later is not on it and leaves.
//
// Word: memory operations on one word (load, store, add, either, swap), of the device (device_scope::Word) or, in a check, of the host.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mtmc {
namespace roll_call {

constexpr uint32_t kClosed = 0x80000000u;

// Counts one in; true: the group is full for the `times`-th time.
template <class Word>
__host__ __device__ inline bool count_in(Word group, uint32_t full, uint32_t times) {
  return group.add(1) + 1 == times * full;  // a closed group never is
}
// Closes the first of the groups that is not full; false: all of them are (and stay open).
template <class Groups>
__host__ __device__ inline bool close(Groups group_of, int n_groups, uint32_t full) {
#pragma unroll 1
  for (int g = 0; g < n_groups; ++g) {
    auto group = group_of(g);
    uint32_t n = group.load();
    while (!(n & kClosed) && n < full)
      if (group.swap(n, n | kClosed)) return true;  // else n is what it holds now
    if (n & kClosed) return true;
  }
  return false;
}

struct Roster {
  int id, n;  // this one's number (-1: not on the list), and how many there are
};
// seats: the numbers given out; list: the length of the closed list.  expired(): whether this one has waited too long.
template <class Word, class Expired>
__host__ __device__ inline Roster join(Word seats, Word list, uint32_t all, Expired expired) {
  const uint32_t id = seats.add(1);
  if (id & kClosed) return Roster{-1, 0};
  for (bool complete = id + 1 == all;; complete = false) {
    if (const uint32_t n = list.load()) return Roster{(int)id, (int)n};
    if (complete || expired()) {
      const uint32_t n = seats.either(kClosed);
      if (!(n & kClosed)) list.store(n);
    }
  }
}

}  // namespace roll_call
}  // namespace mtmc
