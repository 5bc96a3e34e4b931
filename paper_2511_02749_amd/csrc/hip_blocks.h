// The HIP runtime as block_cache.h takes it.
#pragma once
#include <hip/hip_runtime.h>

#include "block_cache.h"

namespace spanq {

// Makes `device` the current one (none for a host-only pool's -1) until it goes out of scope.
class DeviceScope {
 public:
  explicit DeviceScope(int device) {
    if (device < 0 || hipGetDevice(&before_) != hipSuccess || before_ == device) return;
    changed_ = hipSetDevice(device) == hipSuccess;
  }
  ~DeviceScope() {
    if (changed_) (void)hipSetDevice(before_);
  }
  DeviceScope(const DeviceScope&) = delete;
  DeviceScope& operator=(const DeviceScope&) = delete;

 private:
  int before_ = -1;
  bool changed_ = false;
};

struct HipBlocks {
  using Stream = hipStream_t;
  using Event = hipEvent_t;
  using Error = hipError_t;
  using Device = DeviceScope;
  static bool capturing(Stream s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError();  // (the null stream while another one is captured)
    return true;
  }
  static Error alloc(void** p, size_t bytes, Stream s) {
    const hipError_t r = hipMallocAsync(p, bytes, s);
    if (r != hipSuccess) (void)hipGetLastError();  // returned, and perhaps mended by a second try
    return r;
  }
  static void free(void* p, Stream s) { (void)hipFreeAsync(p, s); }
  static Event make_event() {
    hipEvent_t e = nullptr;
    return hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess ? e : nullptr;
  }
  static void destroy(Event e) { (void)hipEventDestroy(e); }
  static Error record(Event e, Stream s) {
    const hipError_t r = hipEventRecord(e, s);
    if (r != hipSuccess) (void)hipGetLastError();  // handled by the caller: not for the next launch's check to find
    return r;
  }
  static bool done(Event e) {
    // relaxed: the thread may be capturing some other stream, which a query must not disturb
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool swapped = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    const hipError_t r = hipEventQuery(e);
    if (swapped) (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (r != hipSuccess) (void)hipGetLastError();  // (hipErrorNotReady)
    return r == hipSuccess;
  }
  static Error wait(Stream s, Event e) { return hipStreamWaitEvent(s, e, 0); }
};

}  // namespace spanq
