// The HIP runtime as block_cache.h takes it.
#pragma once
#include <hip/hip_runtime.h>

#include "block_cache.h"

namespace spanq {

struct HipBlocks {
  using Stream = hipStream_t;
  using Event = hipEvent_t;
  using Error = hipError_t;
  static bool capturing(Stream s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError();  // (the null stream while another one is captured)
    return true;
  }
  static Error alloc(void** p, size_t bytes, Stream s) { return hipMallocAsync(p, bytes, s); }
  static void free(void* p, Stream s) { (void)hipFreeAsync(p, s); }
  static Event make_event() {
    hipEvent_t e = nullptr;
    return hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess ? e : nullptr;
  }
  static void destroy(Event e) { (void)hipEventDestroy(e); }
  static Error record(Event e, Stream s) { return hipEventRecord(e, s); }
  static Error wait(Stream s, Event e) { return hipStreamWaitEvent(s, e, 0); }
};

}  // namespace spanq
