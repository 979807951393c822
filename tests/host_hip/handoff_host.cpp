// csrc/handoff.hip on the host runtime beside this file, and what a test needs to set a scene: memory and streams of a
// device, work that lasts until the test ends it, captures, and counts of what was queued.
#include "../../paper_2502_00937_amd/csrc/handoff.hip"

#include <cstdarg>
#include <cstdio>
#include <cstdlib>

static char g_err[512];
namespace vitenc {
vit_status_t set_error(vit_status_t st, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return st;
}
}  // namespace vitenc

extern "C" {
const char* host_error() { return g_err; }
void* host_alloc(int device, size_t bytes) {
  void* p = aligned_alloc(4096, (bytes + 4095) / 4096 * 4096);
  memset(p, 0, bytes);
  host_hip::memory[(uintptr_t)p] = {bytes, device};
  return p;
}
void* host_stream(int device, int blocking) {
  host_hip::streams.emplace_back(new host_hip::Stream);
  host_hip::streams.back()->device = device;
  host_hip::streams.back()->blocking = blocking != 0;
  return host_hip::streams.back().get();
}
// queues work on `stream` that ends when the test says so, then writes `value` over p[0, bytes)
int host_work(void* stream, void* p, int value, size_t bytes) {
  auto gate = std::make_shared<bool>(false);
  host_hip::gates.push_back(gate);
  host_hip::enqueue(host_hip::resolve(stream), [=]() { memset(p, value, bytes); }, {gate});
  return (int)host_hip::gates.size() - 1;
}
void host_end_work(int gate) {
  *host_hip::gates[(size_t)gate] = true;
  host_hip::pump();
}
void host_pump() { host_hip::pump(); }
void host_capture(void* stream, int mode) {
  ((host_hip::Stream*)stream)->capture = mode < 0 ? hipStreamCaptureStatusNone : hipStreamCaptureStatusActive;
  if (mode >= 0) ((host_hip::Stream*)stream)->mode = (hipStreamCaptureMode)mode;
}
int host_captured(void* stream, int* recorded) {
  *recorded = ((host_hip::Stream*)stream)->recorded;
  return ((host_hip::Stream*)stream)->capture;
}
void host_counts(int* out) {
  out[0] = host_hip::launches; out[1] = host_hip::copies; out[2] = host_hip::waits; out[3] = host_hip::live_events;
  host_hip::launches = host_hip::copies = host_hip::waits = 0;
}
}
