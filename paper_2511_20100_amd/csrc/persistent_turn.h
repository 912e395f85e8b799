// Who may have a persistent launch (decode_persistent.hip) under way on a device.  Host code.
//
// Such a launch needs all of its workgroups resident at once; two of them under way together could each hold half of the CUs
// and wait for the other half for good.  So there is one turn per device: a call takes it without waiting for other threads
// or streams, and a call that does not get it runs the same step as separate launches, which give the same bits.
//   - threads: a mutex that is only ever tried;
//   - streams: an event behind the last launch of the turn before.  While that is still at work, only the stream it went to
//     may take the next turn (and waits for it on the device); where the runtime does not say, nobody;
//   - processes: the first that asks for a device keeps it until it ends, and then the next (an abstract socket name, given back
//     by the kernel whatever ends the process and what it has forked).  Processes of different network namespaces, as in two
//     containers, do not see each other's: each takes its own turns, and launches of both that are in each other's way are given up at
//     their roll call (roll_call.h).
#pragma once

#include <hip/hip_runtime.h>

#include <mutex>

namespace mtmc {

class PersistentTurn {
 public:
  static constexpr int kWorkgroups = 256;  // of a persistent launch, one per CU
  PersistentTurn() = default;
  PersistentTurn(const PersistentTurn&) = delete;
  PersistentTurn& operator=(const PersistentTurn&) = delete;
  ~PersistentTurn() { release(); }
  // Whether work enqueued on st from now on, until release(), may hold persistent launches.  Takes the turn if it is not held.
  bool take(int device, hipStream_t st);
  void release();

 private:
  void* held_ = nullptr;
  hipStream_t st_ = nullptr;
};

// Whether the calls on a weights handle try persistent launches at all.  A launch that was given up says that other work shares the
// device; its call took longer than with separate launches and so would the next ones.  These run separate launches then: 16
// calls, twice as many after each further time (1024 at most), half as many after each call that was allowed and went well.
class PersistentBackoff {
 public:
  // gave_up: the pinned word that a launch sets when it is given up; taken back here.
  bool allows(int* gave_up);
  void forget(int* gave_up);

 private:
  static constexpr int kFewest = 16, kMost = 1024;
  std::mutex mu_;
  int left_ = 0, next_ = kFewest;
};

}  // namespace mtmc
