// A stand-in for the HIP runtime with which host checks drive csrc/workspace.hpp without a GPU: memory
// is a counter per device, streams are numbers, work on a stream stays pending until the check ends it,
// and each refusal that the code has to handle can be switched on.
#pragma once

#include <cstddef>
#include <cstdint>
#include <map>
#include <set>

enum hipError_t {
  hipSuccess = 0,
  hipErrorOutOfMemory = 2,
  hipErrorInvalidHandle = 400,
  hipErrorNotReady = 600,
  hipErrorStreamCaptureUnsupported = 900,
  hipErrorStreamCaptureIsolation = 905
};
struct ihipStream {
  int device = 0;
  bool capturing = false;
  uint64_t issued = 0, ended = 0;  // work enqueued, work finished
};
using hipStream_t = ihipStream *;
struct ihipEvent {
  int device;
  hipStream_t stream = nullptr;
  uint64_t mark = 0;
};
using hipEvent_t = ihipEvent *;
using hipMemPool_t = int;
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeThreadLocal, hipStreamCaptureModeRelaxed };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
enum { hipEventDisableTiming = 2, hipMemPoolAttrReleaseThreshold = 4 };

struct FakeHip {
  int device = 0;
  size_t total = (size_t)64 << 30, free = (size_t)64 << 30;  // of device 0
  bool sync_refused = false;                                 // hipDeviceSynchronize
  hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
  std::map<void *, size_t> live;        // by hipMalloc
  std::map<void *, size_t> pool_live;   // by hipMallocAsync
  size_t pool_free = 0;                 // freed into the pool, not yet given back
  std::set<hipStream_t> streams{nullptr};
  ihipStream null_stream;
  int waits = 0, syncs = 0, mallocs = 0, frees = 0, trims = 0;
  uintptr_t next = 4096;
};
inline FakeHip &fake() {
  static FakeHip f;
  return f;
}
inline hipStream_t fake_stream(hipStream_t s) { return s ? s : &fake().null_stream; }

inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int *d) { return *d = fake().device, hipSuccess; }
inline hipError_t hipSetDevice(int d) { return fake().device = d, hipSuccess; }
inline hipError_t hipDeviceTotalMem(size_t *n, int) { return *n = fake().total, hipSuccess; }
inline hipError_t hipMalloc(void **p, size_t n) {
  ++fake().mallocs;
  if (n > fake().free) return hipErrorOutOfMemory;
  fake().free -= n;
  *p = (void *)fake().next;
  fake().next += n;
  fake().live[*p] = n;
  return hipSuccess;
}
template <class T>
hipError_t hipMalloc(T **p, size_t n) {
  return hipMalloc((void **)p, n);
}
inline hipError_t hipFree(void *p) {
  ++fake().frees;
  if (!fake().live.count(p)) return hipErrorInvalidHandle;
  fake().free += fake().live[p];
  fake().live.erase(p);
  return hipSuccess;
}
inline hipError_t hipMallocAsync(void **p, size_t n, hipStream_t) {
  ++fake().mallocs;
  if (n > fake().free) return hipErrorOutOfMemory;
  fake().free -= n;
  *p = (void *)fake().next;
  fake().next += n;
  fake().pool_live[*p] = n;
  return hipSuccess;
}
inline hipError_t hipFreeAsync(void *p, hipStream_t) {
  fake().pool_free += fake().pool_live[p];
  fake().pool_live.erase(p);
  return hipSuccess;
}
inline hipError_t hipDeviceGetDefaultMemPool(hipMemPool_t *p, int dev) { return *p = dev, hipSuccess; }
inline hipError_t hipMemPoolSetAttribute(hipMemPool_t, int, void *) { return hipSuccess; }
inline hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) {
  ++fake().trims;
  fake().free += fake().pool_free;
  fake().pool_free = 0;
  return hipSuccess;
}
inline hipError_t hipDeviceSynchronize() {
  ++fake().syncs;
  if (fake().sync_refused) return hipErrorStreamCaptureUnsupported;
  for (hipStream_t s : fake().streams)
    if (fake_stream(s)->device == fake().device) fake_stream(s)->ended = fake_stream(s)->issued;
  return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  return *e = new ihipEvent{fake().device}, hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) { return delete e, hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (s && s->device != e->device) return hipErrorInvalidHandle;
  e->stream = s;
  e->mark = fake_stream(s)->issued;
  return hipSuccess;
}
inline hipError_t hipEventQuery(hipEvent_t e) {
  return fake_stream(e->stream)->ended >= e->mark ? hipSuccess : hipErrorNotReady;
}
inline hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned) {
  ++fake().waits;
  return fake_stream(s)->capturing ? hipErrorStreamCaptureIsolation : hipSuccess;
}
inline hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c) {
  *c = fake_stream(s)->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
inline hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m) {
  const hipStreamCaptureMode old = fake().mode;
  fake().mode = *m;
  *m = old;
  return hipSuccess;
}
