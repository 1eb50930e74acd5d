// A stand-in for the few runtime calls that scratch.hpp makes, so that its
// bookkeeping can be tested without a GPU: allocations and events are counted,
// any call can be made to fail once, and like the runtime's a failing call
// leaves its error for hipGetLastError.
#pragma once
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <map>
#include <set>
#include <string>

enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorUnknown = 999,
                  hipErrorNotReady = 600 };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeRelaxed };
constexpr unsigned hipEventDisableTiming = 2;

struct StubStream { bool capturing = false; bool pending = false; };
struct StubEvent { StubStream* on = nullptr; };
typedef StubStream* hipStream_t;
typedef StubEvent* hipEvent_t;
typedef void* hipMemPool_t;

namespace stub {
inline std::set<std::string> fail;             // calls that fail the next time
inline hipError_t last = hipSuccess;
inline std::map<void*, size_t> live;           // allocations
inline std::map<std::string, int> calls;
inline size_t limit = SIZE_MAX;                // bytes that can be had
inline size_t total() {
  size_t t = 0;
  for (auto& a : live) t += a.second;
  return t;
}
inline hipError_t ret(const char* name, hipError_t e = hipSuccess) {
  ++calls[name];
  if (fail.erase(name)) e = hipErrorUnknown;
  if (e != hipSuccess) last = e;
  return e;
}
}  // namespace stub

inline hipError_t hipGetLastError() {
  const hipError_t e = stub::last;
  stub::last = hipSuccess;
  return e;
}
inline hipError_t hipMallocFromPoolAsync(void** p, size_t n, hipMemPool_t, hipStream_t) {
  if (stub::total() + n > stub::limit) return stub::ret("malloc", hipErrorOutOfMemory);
  const hipError_t e = stub::ret("malloc");
  if (e == hipSuccess) stub::live[*p = std::malloc(1)] = n;
  return e;
}
inline hipError_t hipFreeAsync(void* p, hipStream_t) {
  if (!stub::live.erase(p)) std::abort();      // not an allocation, or freed twice
  std::free(p);
  return stub::ret("free");
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  const hipError_t r = stub::ret("event");
  if (r == hipSuccess) *e = new StubEvent;
  return r;
}
inline hipError_t hipEventDestroy(hipEvent_t e) {
  delete e;
  return stub::ret("event_destroy");
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  e->on = s;
  return stub::ret("record");
}
inline hipError_t hipEventQuery(hipEvent_t e) {
  return stub::ret("query", e->on && e->on->pending ? hipErrorNotReady : hipSuccess);
}
inline hipError_t hipEventSynchronize(hipEvent_t) { return stub::ret("event_sync"); }
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) {
  return stub::ret("wait");
}
inline hipError_t hipStreamSynchronize(hipStream_t) { return stub::ret("sync"); }
inline hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c) {
  *c = s && s->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return stub::ret("capturing");
}
inline hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) {
  return stub::ret("mode");
}
