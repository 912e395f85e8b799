// Host code that asks the runtime about its own work, whatever other threads capture.
#pragma once

#include <hip/hip_runtime.h>

namespace mtmc {

// Another thread may be capturing a stream in global mode, which refuses other threads' queries of an event and ends with them.
// What is asked while one of these lives is no part of such a capture.
class OutsideCaptures {
 public:
  OutsideCaptures() { swap(); }
  OutsideCaptures(const OutsideCaptures&) = delete;
  OutsideCaptures& operator=(const OutsideCaptures&) = delete;
  ~OutsideCaptures() { swap(); }

 private:
  void swap() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
  hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
};

}  // namespace mtmc
