// The few runtime calls that host_io.hpp makes, on the CPU: two devices,
// pinned memory and events that belong to the device they were made on, and
// streams whose copies run as late as the waits allow.  A copy that nothing
// waits for has not happened, and one that runs after its slot was used again
// moves the wrong values: a missing wait shows as a wrong result.
#pragma once
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>

enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorInvalidDevice = 101, hipErrorInvalidHandle = 400 };
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2 };
enum { hipHostMallocDefault = 0, hipEventDisableTiming = 2 };

struct MockStream {
  int device = 0;
  long done = 0;                           // copies that have run
  std::deque<std::function<void()>> todo;  // the ones after them
  void run_to(long k) {
    for (; done < k && !todo.empty(); ++done) {
      todo.front()();
      todo.pop_front();
    }
  }
};
struct MockEvent {
  int device = 0;
  MockStream* s = nullptr;
  long at = 0;  // copies of s before it
};
typedef MockStream* hipStream_t;
typedef MockEvent* hipEvent_t;

struct Mock {
  int device = 0;            // the current one (the checks make runtime calls from one thread)
  long pins = 0, freed = 0;  // pinned allocations made and given back
  long copies = 0;
  const void* host = nullptr;  // host side of the last copy
  long fail_record = -1;       // the record that fails, counted from 0
  long records = 0;
};
inline Mock& mock() {
  static Mock m;
  return m;
}

inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) {
  *d = mock().device;
  return hipSuccess;
}
inline hipError_t hipSetDevice(int d) {
  if (d < 0 || d > 1) return hipErrorInvalidDevice;
  mock().device = d;
  return hipSuccess;
}
inline hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
  *p = std::malloc(bytes);
  ++mock().pins;
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
inline hipError_t hipHostFree(void* p) {
  std::free(p);
  ++mock().freed;
  return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = new MockEvent{mock().device};
  return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) {
  delete e;
  return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind kind, hipStream_t s) {
  ++mock().copies;
  mock().host = kind == hipMemcpyHostToDevice ? src : dst;
  s->todo.push_back([=] { std::memcpy(dst, src, bytes); });
  return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (mock().records++ == mock().fail_record || e->device != s->device) return hipErrorInvalidHandle;
  e->s = s;
  e->at = s->done + long(s->todo.size());
  return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t e) {
  if (e->s) e->s->run_to(e->at);
  return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t s) {
  s->run_to(s->done + long(s->todo.size()));
  return hipSuccess;
}
