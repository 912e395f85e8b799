// Who may have a persistent launch (decode_persistent.hip) under way on a device.  Host code.
//
// Such a launch needs all of its workgroups resident at once; two of them under way together could each hold half of the CUs
// and wait for the other half for good.  So there is one turn per device: a call takes it without waiting for other threads
// or streams, and a call that does not get it runs the same step as separate launches, which give the same bits.
//   - threads: a mutex that is only ever tried;
//   - streams: an event behind the last launch of the turn before.  While that is still at work, only the stream it went to
//     may take the next turn (and waits for it on the device); where the runtime does not say, nobody;
//   - processes: the first that asks for a device keeps it until it ends (an abstract socket name of the host's network
//     namespace, given back by the kernel whatever ends the process).
#pragma once

#include <hip/hip_runtime.h>

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

}  // namespace mtmc
