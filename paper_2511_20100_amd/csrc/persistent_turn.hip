// The turn of the persistent launches on a device: see persistent_turn.h.
#include "persistent_turn.h"

#include <stddef.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/socket.h>
#include <sys/un.h>
#include <unistd.h>

#include <algorithm>

#include "outside_captures.h"

namespace mtmc {
namespace {

struct DeviceTurn {
  std::mutex mu;
  bool asked = false, able = false, leased = false;
  hipEvent_t last = nullptr;  // behind the launches of the latest turn
  hipStream_t stream = nullptr;
  bool recorded = false;
};
constexpr int kMaxDevices = 64;
DeviceTurn g_turns[kMaxDevices];  // events stay until the process ends

// The name is held by a socket that is never closed: the lease ends with the process.
bool lease_device(int device) {
  char bus[32];
  if (hipDeviceGetPCIBusId(bus, sizeof bus, device) != hipSuccess) return false;
  const int fd = socket(AF_UNIX, SOCK_DGRAM | SOCK_CLOEXEC, 0);
  if (fd < 0) return false;
  sockaddr_un addr;
  memset(&addr, 0, sizeof addr);
  addr.sun_family = AF_UNIX;
  const int n = snprintf(addr.sun_path + 1, sizeof addr.sun_path - 1, "mtmc-persistent-%s", bus);
  if (bind(fd, (const sockaddr*)&addr, (socklen_t)(offsetof(sockaddr_un, sun_path) + 1 + n)) != 0) {
    close(fd);
    return false;
  }
  return true;
}

// Every CU has to be open to the stream.
bool whole_device(hipStream_t st) {
  if (getenv("HSA_CU_MASK") || getenv("ROC_GLOBAL_CU_MASK")) return false;
  if (st == nullptr || st == hipStreamPerThread || st == hipStreamLegacy) return true;  // these have no mask of their own
  uint32_t mask[16] = {};
  if (hipExtStreamGetCUMask(st, 16, mask) != hipSuccess) return false;
  int open = 0;
  for (uint32_t m : mask) open += __builtin_popcount(m);
  return open >= PersistentTurn::kWorkgroups;
}

bool usable(DeviceTurn& t, int device) {
  if (!t.asked) {
    t.asked = true;
    int cus = 0;
    t.able = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess &&
             cus >= PersistentTurn::kWorkgroups &&
             hipEventCreateWithFlags(&t.last, hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess;
  }
  if (t.able && !t.leased) t.leased = lease_device(device);  // at every turn: whoever has the device may end
  return t.able && t.leased;
}

// Whether the launches of the latest turn have ended, or st (theirs) waits for them.  Any other answer than "ended" or "not yet"
// says nothing about them: they may be under way.
bool clear_for(DeviceTurn& t, hipStream_t st) {
  if (!t.recorded) return true;
  const hipError_t e = hipEventQuery(t.last);
  if (e == hipSuccess) return true;
  (void)hipGetLastError();
  if (e != hipErrorNotReady || t.stream != st) return false;
  if (hipStreamWaitEvent(st, t.last, 0) == hipSuccess) return true;
  (void)hipGetLastError();
  return false;
}

}  // namespace

bool PersistentTurn::take(int device, hipStream_t st) {
  if (held_) return true;
  if (device < 0 || device >= kMaxDevices) return false;
  OutsideCaptures outside;
  if (!whole_device(st)) return false;
  DeviceTurn& t = g_turns[device];
  if (!t.mu.try_lock()) return false;
  if (!usable(t, device) || !clear_for(t, st)) {
    t.mu.unlock();
    return false;
  }
  held_ = &t;
  st_ = st;
  return true;
}

void PersistentTurn::release() {
  if (!held_) return;
  OutsideCaptures outside;
  DeviceTurn& t = *(DeviceTurn*)held_;
  t.recorded = hipEventRecord(t.last, st_) == hipSuccess;
  // no event to wait for: wait here, or nobody takes a turn any more
  if (!t.recorded && hipStreamSynchronize(st_) != hipSuccess) t.able = false;
  t.stream = st_;
  t.mu.unlock();
  held_ = nullptr;
}

bool PersistentBackoff::allows(int* gave_up) {
  std::lock_guard<std::mutex> lock(mu_);
  if (__atomic_exchange_n(gave_up, 0, __ATOMIC_RELAXED)) {
    left_ = next_;
    next_ = std::min(2 * next_, kMost);
  } else if (left_ == 0) {
    next_ = std::max(next_ / 2, kFewest);
  }
  if (left_ == 0) return true;
  --left_;
  return false;
}

void PersistentBackoff::forget(int* gave_up) {
  std::lock_guard<std::mutex> lock(mu_);
  __atomic_store_n(gave_up, 0, __ATOMIC_RELAXED);
  left_ = 0;
  next_ = kFewest;
}

}  // namespace mtmc
