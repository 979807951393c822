// The part of the HIP runtime that the hand-off table uses, on the host: streams are queues of operations that run when
// what they come after has run, memory is host memory registered as a device's, kernels are loops over their threads.
// Tests build csrc/handoff.hip against it and see what its calls queue, on as many devices as they like, without a GPU.
//
// What is modelled: an event is the end of its last recording; the null stream and the blocking streams of a device come
// after one another as they were queued; a query answers for the operations of that stream alone; an event belongs
// to the device it was created on and only that device's streams take its recording; asking a stream under capture or an
// event recorded in it, or anything while a capture in global mode is on and the thread has not said relaxed, ends the capture.
// Workgroups run in descending order: a launch promises none.
#pragma once
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <memory>
#include <tuple>
#include <vector>

enum hipError_t {
  hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorInvalidDevice = 101, hipErrorInvalidHandle = 400, hipErrorNotReady = 600,
  hipErrorStreamCaptureUnsupported = 900
};
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone = 0, hipStreamCaptureStatusActive = 1, hipStreamCaptureStatusInvalidated = 2 };
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal = 0, hipStreamCaptureModeThreadLocal = 1, hipStreamCaptureModeRelaxed = 2 };
enum hipMemoryType { hipMemoryTypeHost = 1, hipMemoryTypeDevice = 2 };
enum hipMemcpyKind { hipMemcpyDeviceToDevice = 3 };
enum { hipStreamDefault = 0, hipStreamNonBlocking = 1, hipEventDisableTiming = 2 };
typedef int hipDevice_t;
typedef void* hipDeviceptr_t;
struct hipPointerAttribute_t { hipMemoryType type; int device; };
struct dim3 { unsigned x = 1, y = 1, z = 1; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };

#define __global__
#define __launch_bounds__(...)

namespace host_hip {
typedef std::shared_ptr<bool> Done;
struct Op { std::function<void()> fn; std::vector<Done> after; Done done; };
struct Stream {
  int device = 0;
  bool blocking = true;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
  std::deque<Op> ops;
  int recorded = 0;  // operations that went into a capture
};
struct Event { int device = 0; Done done; Stream* captured = nullptr; };
struct Block { size_t bytes; int device; };

constexpr int kDevices = 2;
inline Stream null_stream[kDevices];
inline std::vector<std::unique_ptr<Stream>> streams;
inline std::map<uintptr_t, Block> memory;
inline std::vector<Done> gates;
inline int device = 0, launches = 0, copies = 0, waits = 0, live_events = 0;
inline hipStreamCaptureMode thread_mode = hipStreamCaptureModeGlobal;
inline thread_local dim3 block_index, thread_index;

inline Stream* resolve(void* s) { return s ? (Stream*)s : &null_stream[device]; }
inline std::vector<Stream*> all() {
  std::vector<Stream*> v;
  for (auto& s : null_stream) v.push_back(&s);
  for (auto& s : streams) v.push_back(s.get());
  return v;
}
inline bool is_null(const Stream* s) { return s >= null_stream && s < null_stream + kDevices; }

// The streams whose earlier operations an operation on `s` comes after.
inline void enqueue(Stream* s, std::function<void()> fn, std::vector<Done> after = {}, Done done = std::make_shared<bool>(false)) {
  if (s->capture != hipStreamCaptureStatusNone) { s->recorded += 1; return; }
  for (Stream* o : all())
    if (o != s && o->device == s->device && !o->ops.empty() && ((is_null(s) && o->blocking) || (is_null(o) && s->blocking)))
      after.push_back(o->ops.back().done);
  s->ops.push_back({std::move(fn), std::move(after), done});
}

inline void pump() {
  for (bool moved = true; moved;) {
    moved = false;
    for (Stream* s : all())
      while (!s->ops.empty()) {
        Op& op = s->ops.front();
        bool go = true;
        for (auto& d : op.after) go = go && *d;
        if (!go) break;
        if (op.fn) op.fn();
        *op.done = true;
        s->ops.pop_front();
        moved = true;
      }
  }
}

// A question that a capture does not survive.
inline bool breaks_capture(Stream* asked) {
  bool broke = false;
  for (Stream* s : all())
    if (s->capture == hipStreamCaptureStatusActive &&
        (s == asked || (s->mode == hipStreamCaptureModeGlobal && thread_mode != hipStreamCaptureModeRelaxed))) {
      s->capture = hipStreamCaptureStatusInvalidated;
      broke = true;
    }
  return broke;
}

template <class... P, class... A>
void launch(void (*kernel)(P...), dim3 grid, dim3 block, Stream* s, A... args) {
  launches += 1;
  std::tuple<P...> copy(args...);
  enqueue(s, [=]() {
    for (unsigned b = grid.x; b-- > 0;)
      for (unsigned t = 0; t < block.x; ++t) {
        block_index = dim3(b, 0, 0);
        thread_index = dim3(t, 0, 0);
        std::apply(kernel, copy);
      }
  });
}
}  // namespace host_hip

typedef host_hip::Stream* hipStream_t;
typedef host_hip::Event* hipEvent_t;
#define hipStreamPerThread ((hipStream_t)2)
#define hipStreamLegacy ((hipStream_t)1)
#define blockIdx host_hip::block_index
#define threadIdx host_hip::thread_index
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) host_hip::launch(kernel, grid, block, host_hip::resolve(stream), __VA_ARGS__)

inline const char* hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : e == hipErrorInvalidHandle ? "invalid resource handle" : "error"; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipSetDevice(int d) {
  if (d < 0 || d >= host_hip::kDevices) return hipErrorInvalidDevice;
  host_hip::device = d;
  return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = new host_hip::Event{host_hip::device};
  host_hip::live_events += 1;
  return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) {
  delete e;
  host_hip::live_events -= 1;
  return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t stream) {
  host_hip::Stream* s = host_hip::resolve(stream);
  if (s->device != e->device) return hipErrorInvalidHandle;
  auto done = std::make_shared<bool>(false);
  host_hip::enqueue(s, nullptr, {}, done);
  e->captured = s->capture == hipStreamCaptureStatusNone ? nullptr : s;
  e->done = e->captured ? nullptr : done;
  return hipSuccess;
}
inline hipError_t hipEventQuery(hipEvent_t e) {
  if (host_hip::breaks_capture(e->captured)) return hipErrorStreamCaptureUnsupported;
  host_hip::pump();
  return !e->done || *e->done ? hipSuccess : hipErrorNotReady;
}
inline hipError_t hipStreamWaitEvent(hipStream_t stream, hipEvent_t e, unsigned) {
  host_hip::waits += 1;
  if (e->done) host_hip::enqueue(host_hip::resolve(stream), nullptr, {e->done});
  return hipSuccess;
}
inline hipError_t hipStreamQuery(hipStream_t stream) {
  host_hip::Stream* s = host_hip::resolve(stream);
  if (host_hip::breaks_capture(s)) return hipErrorStreamCaptureUnsupported;
  host_hip::pump();
  return s->ops.empty() ? hipSuccess : hipErrorNotReady;
}
inline hipError_t hipStreamIsCapturing(hipStream_t stream, hipStreamCaptureStatus* st) {
  *st = host_hip::resolve(stream)->capture;
  return hipSuccess;
}
inline hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
  std::swap(*m, host_hip::thread_mode);
  return hipSuccess;
}
inline hipError_t hipStreamGetDevice(hipStream_t stream, hipDevice_t* d) {
  *d = host_hip::resolve(stream)->device;
  return hipSuccess;
}
inline hipError_t hipStreamGetFlags(hipStream_t stream, unsigned* f) {
  if (!stream) return hipErrorInvalidValue;
  *f = stream->blocking ? hipStreamDefault : hipStreamNonBlocking;
  return hipSuccess;
}
inline hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* n, hipDeviceptr_t p) {
  auto it = host_hip::memory.upper_bound((uintptr_t)p);
  if (it == host_hip::memory.begin()) return hipErrorInvalidValue;
  --it;
  if ((uintptr_t)p - it->first >= it->second.bytes) return hipErrorInvalidValue;
  *base = (void*)it->first;
  *n = it->second.bytes;
  return hipSuccess;
}
inline hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  void* base;
  size_t n;
  if (hipMemGetAddressRange(&base, &n, (void*)p) != hipSuccess) return hipErrorInvalidValue;
  *a = {hipMemoryTypeDevice, host_hip::memory[(uintptr_t)base].device};
  return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t stream) {
  host_hip::copies += 1;
  host_hip::enqueue(host_hip::resolve(stream), [=]() { memmove(to, from, n); });
  return hipSuccess;
}
