// A stand-in for the HIP runtime's host API, for checks of libnetsim's host
// code on the CPU (tests/native/host_failures.cpp): device memory is host
// memory, a stream only counts the work queued on it, and any one call can be
// made to fail.
#pragma once

#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <set>

struct int2 { int x, y; };
struct uint4 { unsigned x, y, z, w; };

enum hipError_t { hipSuccess = 0, hipErrorInvalidConfiguration = 9, hipErrorUnknown = 999 };
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2, hipMemcpyDeviceToDevice = 3 };
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount, hipDeviceAttributeWallClockRate };
enum hipStreamCaptureMode { hipStreamCaptureModeThreadLocal };
constexpr unsigned hipStreamNonBlocking = 1, hipEventDisableTiming = 2, hipHostMallocDefault = 0;

struct ihipStream {
  int queued = 0;                  // pieces of work not waited for
  std::set<ihipStream*> after;     // streams whose work this one waits for
};
struct ihipEvent { ihipStream* on = nullptr; };
typedef ihipStream* hipStream_t;
typedef ihipEvent* hipEvent_t;
typedef struct ihipGraph* hipGraph_t;
typedef struct ihipGraphExec* hipGraphExec_t;
struct hipDeviceProp_t { int multiProcessorCount; };

struct FakeHip {
  long calls = 0, fail_at = 0;     // the call that fails (0: none)
  ihipStream null_stream;
  std::set<ihipStream*> streams;
  std::set<ihipEvent*> events;
  std::set<void*> device, pinned;
  hipError_t next() { return ++calls == fail_at ? hipErrorUnknown : hipSuccess; }
  ihipStream* of(hipStream_t s) {
    if (!s) return &null_stream;
    if (!streams.count(s)) bug("a stream that does not exist is used");
    return s;
  }
  [[noreturn]] static void bug(const char* what) {
    printf("BUG: %s\n", what);
    exit(1);
  }
  hipError_t work(hipStream_t s) {
    if (const hipError_t e = next()) return e;
    of(s)->queued += 1;
    return hipSuccess;
  }
  void wait(ihipStream* s) {
    s->queued = 0;
    const std::set<ihipStream*> a = s->after;
    s->after.clear();
    for (ihipStream* x : a) wait(x);
  }
  long queued() const {
    long n = null_stream.queued;
    for (ihipStream* s : streams) n += s->queued;
    return n;
  }
};
extern FakeHip fake;

inline const char* hipGetErrorString(hipError_t) { return "made to fail"; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipSetDevice(int) { return fake.next(); }
inline hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 100000;
  return fake.next();
}
inline hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
  p->multiProcessorCount = 256;
  return fake.next();
}
template <class T>
hipError_t hipMalloc(T** p, size_t n) {
  if (const hipError_t e = fake.next()) return e;
  *p = (T*)calloc(1, n ? n : 1);
  fake.device.insert((void*)*p);
  return hipSuccess;
}
inline hipError_t hipFree(void* p) {  // waits for the device
  fake.wait(&fake.null_stream);
  for (ihipStream* s : fake.streams) fake.wait(s);
  if (p && !fake.device.erase(p)) FakeHip::bug("device memory given back twice");
  free(p);
  return hipSuccess;
}
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (const hipError_t e = fake.next()) return e;
  *p = calloc(1, n);
  fake.pinned.insert(*p);
  return hipSuccess;
}
inline hipError_t hipHostFree(void* p) {
  if (p && !fake.pinned.erase(p)) FakeHip::bug("pinned memory given back twice");
  free(p);
  return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t s) {
  if (const hipError_t e = fake.next()) return e;
  fake.wait(fake.of(s));
  return hipSuccess;
}
inline hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  if (const hipError_t e = fake.next()) return e;
  fake.wait(&fake.null_stream);
  memmove(d, s, n);
  return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  if (const hipError_t e = fake.work(st)) return e;
  memmove(d, s, n);
  return hipSuccess;
}
inline hipError_t hipMemset(void* d, int v, size_t n) {
  memset(d, v, n);
  return fake.next();
}
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  if (const hipError_t e = fake.next()) return e;
  fake.streams.insert(*s = new ihipStream);
  return hipSuccess;
}
inline hipError_t hipStreamDestroy(hipStream_t s) {
  if (!fake.streams.erase(s)) FakeHip::bug("a stream given back twice");
  delete s;
  return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  if (const hipError_t r = fake.next()) return r;
  fake.events.insert(*e = new ihipEvent);
  return hipSuccess;
}
inline hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
inline ihipEvent* fake_event(hipEvent_t e) {
  if (!fake.events.count(e)) FakeHip::bug("an event that does not exist is used");
  return e;
}
inline hipError_t hipEventDestroy(hipEvent_t e) {
  fake.events.erase(fake_event(e));
  delete e;
  return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  fake_event(e)->on = fake.of(s);
  return fake.next();
}
inline hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  if (const hipError_t r = fake.next()) return r;
  if (fake_event(e)->on && e->on != fake.of(s)) fake.of(s)->after.insert(e->on);
  return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t e) {
  if (const hipError_t r = fake.next()) return r;
  if (fake_event(e)->on) fake.wait(e->on);
  return hipSuccess;
}
inline hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  fake_event(a);
  fake_event(b);
  *ms = 1.0f;
  return fake.next();
}
inline hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorUnknown; }
inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorUnknown; }
inline hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, void*, char*, size_t) { return hipErrorUnknown; }
inline hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
inline hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorUnknown; }
inline hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
