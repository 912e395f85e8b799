// Who gets the turn of the persistent launches, with a runtime whose answers are set here.  Compiled (with persistent_turn.hip)
// and run by test_persistent_turn.py; exits non-zero at the first claim that does not hold.
#include <sys/wait.h>
#include <unistd.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "persistent_turn.h"

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); std::exit(1); } } while (0)

// ---- the runtime
static hipError_t g_query = hipSuccess, g_wait = hipSuccess, g_record = hipSuccess, g_sync = hipSuccess;
static int g_waits = 0, g_cus = 256, g_open_words = 8;
static hipStreamCaptureMode g_mode = hipStreamCaptureModeGlobal;
static const char* g_bus = nullptr;
extern "C" {
hipError_t hipDeviceGetPCIBusId(char* bus, int n, int device) {
  if (g_bus) std::snprintf(bus, n, "%s", g_bus);
  else std::snprintf(bus, n, "check-%d-%d", (int)getpid(), device);
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = g_cus; return hipSuccess; }
hipError_t hipExtStreamGetCUMask(hipStream_t, uint32_t n, uint32_t* mask) {
  for (uint32_t i = 0; i < n; ++i) mask[i] = (int)i < g_open_words ? ~0u : 0u;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)(uintptr_t)1; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return g_mode == hipStreamCaptureModeRelaxed ? g_query : hipErrorStreamCaptureUnsupported; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return g_record; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { ++g_waits; return g_wait; }
hipError_t hipStreamSynchronize(hipStream_t) { return g_sync; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) { std::swap(*m, g_mode); return hipSuccess; }
}

static const hipStream_t kA = (hipStream_t)(uintptr_t)64, kB = (hipStream_t)(uintptr_t)128;

static bool takes(int device, hipStream_t st) {
  mtmc::PersistentTurn turn;
  const bool got = turn.take(device, st);
  CHECK(g_mode == hipStreamCaptureModeGlobal);  // the thread's own mode is back
  return got;
}

// The launches of the last turn: ended, under way, or the runtime does not say.
static void what_the_last_turn_left() {
  const int dev = 1;
  CHECK(takes(dev, kA));
  g_query = hipSuccess;
  CHECK(takes(dev, kB));  // ended; now kB's are the last
  g_query = hipErrorNotReady;
  g_waits = 0;
  CHECK(!takes(dev, kA) && g_waits == 0);
  CHECK(takes(dev, kB) && g_waits == 1);
  g_wait = hipErrorInvalidValue;
  CHECK(!takes(dev, kB));
  g_wait = hipSuccess;
  for (hipError_t e : {hipErrorStreamCaptureUnsupported, hipErrorStreamCaptureInvalidated, hipErrorCapturedEvent, hipErrorLaunchFailure,
                       hipErrorUnknown, hipErrorInvalidHandle}) {
    g_query = e;
    CHECK(!takes(dev, kA) && !takes(dev, kB));
  }
  g_query = hipSuccess;
  CHECK(takes(dev, kA));
}

static void one_at_a_time() {
  mtmc::PersistentTurn a, b;
  CHECK(a.take(2, kA) && a.take(2, kA) && !b.take(2, kA) && !b.take(2, kB) && b.take(3, kB));
  a.release();
  CHECK(!a.take(3, kA) && a.take(2, kB));
}

static void without_an_event() {
  g_record = hipErrorUnknown;
  CHECK(takes(4, kA));
  g_query = hipErrorNotReady;
  CHECK(takes(4, kB));  // waited for on the host
  g_sync = hipErrorUnknown;
  CHECK(takes(4, kB));
  g_record = g_sync = g_query = hipSuccess;
  CHECK(!takes(4, kB) && !takes(4, kA));  // what it launched may be under way for good
}

static void not_the_whole_device() {
  CHECK(!takes(-1, kA) && !takes(64, kA));
  g_open_words = 7;
  CHECK(!takes(5, kA) && takes(5, nullptr));
  g_open_words = 8;
  g_cus = 255;
  CHECK(!takes(6, kA));
  g_cus = 256;
}

// A launch that was given up: 16 calls without, then 32, ... 1024; fewer again when it goes well.
static void after_a_launch_that_was_given_up() {
  mtmc::PersistentBackoff b;
  int word = 0;
  auto without = [&] {  // calls until one is allowed
    int n = 0;
    while (!b.allows(&word)) ++n;
    return n;
  };
  CHECK(without() == 0 && without() == 0);
  for (int want : {16, 32, 64, 128, 256, 512, 1024, 1024}) {
    word = 1;
    CHECK(!b.allows(&word) && word == 0);
    // the call that is allowed again has the next strike at once, which the pause is doubled by
    int n = 1;
    for (; n < want; ++n) CHECK(!b.allows(&word));
  }
  CHECK(b.allows(&word) && b.allows(&word));
  word = 1;
  CHECK(without() == 256);
  word = 1;
  CHECK(!b.allows(&word));
  word = 1;
  b.forget(&word);
  CHECK(word == 0 && b.allows(&word));
  word = 1;
  CHECK(without() == 16);
}

// Two processes on one device: whoever asked first, and the other one when that has ended.
static void one_process_at_a_time() {
  static char name[64];
  std::snprintf(name, sizeof name, "check-shared-%d", (int)getpid());
  g_bus = name;
  int has[2], end[2];
  CHECK(pipe(has) == 0 && pipe(end) == 0);
  const pid_t pid = fork();
  char c = 0;
  if (pid == 0) {
    const bool got = takes(7, kA) && takes(7, kB);
    CHECK(write(has[1], got ? "y" : "n", 1) == 1 && read(end[0], &c, 1) == 1);
    _exit(0);
  }
  CHECK(pid > 0 && read(has[0], &c, 1) == 1 && c == 'y');
  CHECK(!takes(7, kA) && !takes(7, kB));
  CHECK(write(end[1], "e", 1) == 1 && waitpid(pid, nullptr, 0) == pid);
  CHECK(takes(7, kA) && takes(7, kB));
  g_bus = nullptr;
}

int main() {
  one_process_at_a_time();
  what_the_last_turn_left();
  one_at_a_time();
  without_an_event();
  not_the_whole_device();
  after_a_launch_that_was_given_up();
  std::printf("ok\n");
  return 0;
}
