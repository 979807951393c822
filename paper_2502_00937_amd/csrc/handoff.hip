// Pull-style hand-off of finished image tokens (paper Sec. 4.3, "Image Token Transfer").
//
// A producer (an encoder launch) publishes where the tokens of one image of a request lie in device
// memory and, unless it would be behind nothing, records an event on its stream; nothing is copied then.
// When every image of the request has been published the consumer, which by now knows where the request
// will run, pulls: the images are moved on the consumer's stream behind the producers' events
// (many-to-one aggregation, transfer deferred until the request is complete).  Images that lie on the
// table's GPU are gathered by one kernel, or a few if some are not finished yet; anything else (another
// GPU's memory, pinned host memory, pieces that do not meet 16-byte alignment, a destination that overlaps
// the sources) is a copy of its own.
// No arithmetic of the encoder happens here.
#include "../../include/vitenc.h"

#include <hip/hip_runtime.h>

#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

namespace vitenc {
vit_status_t set_error(vit_status_t st, const char* fmt, ...);  // vitenc_api.hip: message for vit_last_error()
}
using vitenc::set_error;

namespace {
struct Piece {
  const void* ptr = nullptr;
  size_t bytes = 0;
  hipEvent_t ready = nullptr;
  bool published = false;
  bool late = false;  // of the pull at hand: the event had not come when the pull was queued
};
struct Request {
  std::vector<Piece> pieces;
  int published = 0;
  size_t total = 0;
  bool busy = false;  // a producer was found at work when it published: the later images get their events unasked
  bool captured = false;  // an image was published on a stream under capture: its event must not be asked
};
}  // namespace

struct vit_handoff {
  int device = 0;
  std::mutex mu;
  std::unordered_map<int64_t, Request> requests;
};

namespace {
void drop(Request& r) {
  for (auto& p : r.pieces)
    if (p.ready) (void)hipEventDestroy(p.ready);
}

// Whether `s` is a stream of `device`, on which that device's events can be recorded and its kernels launched.
bool stream_of(hipStream_t s, int device) {
  if (!s || s == hipStreamPerThread || s == hipStreamLegacy) return true;  // of whichever device is current
  hipDevice_t d = -1;
  const bool ok = hipStreamGetDevice(s, &d) == hipSuccess && (int)d == device;
  if (!ok) (void)hipGetLastError();
  return ok;
}

// Keeps what is asked meanwhile out of captures that other streams are in.
struct RelaxedCapture {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  bool ok;
  RelaxedCapture() : ok(hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess) {
    if (!ok) (void)hipGetLastError();
  }
  ~RelaxedCapture() {
    if (ok) (void)hipThreadExchangeStreamCaptureMode(&mode);
  }
};

// A stream that is being captured must not be asked how far it is, nor an event recorded in it: neither has any progress to
// report, and the question would end the capture.
bool capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

// Whether an event recorded on `s` now would be behind nothing.
// A stream of another device never counts as finished, so that it is refused where its event is recorded, at work or not.
// What a blocking stream is given comes after the null stream's earlier work, of which a query of it says nothing.
bool finished(hipStream_t s, int device) {
  if (!stream_of(s, device)) return false;
  RelaxedCapture relaxed;
  auto idle = [](hipStream_t q) { return !capturing(q) && hipStreamQuery(q) == hipSuccess; };
  unsigned flags = hipStreamDefault;
  bool done = relaxed.ok && idle(s);
  if (done && s) done = hipStreamGetFlags(s, &flags) == hipSuccess && ((flags & hipStreamNonBlocking) || idle(nullptr));
  if (!done) (void)hipGetLastError();  // "not ready" is an answer
  return done;
}

// ---- one launch for the images of a request ------------------------------------------------------
// Bound by HBM: every byte is read and written once.  A copy of its own per image costs the stream 6 us between the
// copies on top of 3.9 us for an image of 4.7 MB, and one such copy is too short to reach the memory's rate.
// The images are moved in no order, so none may lie where another one is to go (meets_destination).
// Measured with 32 images of 577 x 4096 bf16 tokens that were finished (302 MB moved), handed off again and again: 50 us,
// of which the kernel 49 (6.1 TB/s; a large copy reaches 4.9, but of these 302 MB part stays in the 256 MB memory-side
// cache).  With a copy and an event per image 270 to 287; the gather brought 245 with an event per image, the
// events' absence 79 and the non-temporal hints 61 on the machine of that day.
// A workgroup moves one 32 KiB chunk, eight 16-byte loads in flight per lane; the table of images travels as the
// kernel's argument (no staging buffer), so that a launch holds at most kGatherPieces of them.
typedef uint32_t chunk_t __attribute__((ext_vector_type(4)));
constexpr int kGatherPieces = 128;
constexpr int kGatherLoads = 8, kGatherChunk = 256 * 16 * kGatherLoads;
constexpr size_t kGroupBytes = (size_t)16 << 20;
struct GatherArgs {
  const unsigned char* src[kGatherPieces];
  unsigned char* dst[kGatherPieces];
  size_t bytes[kGatherPieces];
  int32_t first_chunk[kGatherPieces + 1];
  int32_t n;
};
static_assert(sizeof(GatherArgs) <= 4096, "kernel arguments");

__global__ __launch_bounds__(256) void gather_kernel(const GatherArgs a) {
  const int chunk = (int)blockIdx.x;
  int lo = 0, hi = a.n;  // the image whose chunks hold this one: first_chunk[lo] <= chunk < first_chunk[lo + 1]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (a.first_chunk[mid] <= chunk) lo = mid; else hi = mid;
  }
  const size_t off = (size_t)(chunk - a.first_chunk[lo]) * kGatherChunk;
  const unsigned char* s = a.src[lo] + off;
  unsigned char* d = a.dst[lo] + off;
  const size_t left = a.bytes[lo] - off;
  const int tid = (int)threadIdx.x;
  if (left >= (size_t)kGatherChunk) {
    chunk_t v[kGatherLoads];
#pragma unroll
    for (int i = 0; i < kGatherLoads; ++i) v[i] = __builtin_nontemporal_load((const chunk_t*)s + i * 256 + tid);
#pragma unroll
    for (int i = 0; i < kGatherLoads; ++i) __builtin_nontemporal_store(v[i], (chunk_t*)d + i * 256 + tid);
  } else {
    const int n16 = (int)(left / 16), tail = (int)(left % 16);
    for (int i = tid; i < n16; i += 256) ((chunk_t*)d)[i] = ((const chunk_t*)s)[i];
    if (tid < tail) d[n16 * 16 + tid] = s[n16 * 16 + tid];
  }
}

// Whether [p, p + bytes) lies inside one allocation on `device`.  [base, base + size) is the last range that passed, of
// this pull alone: the images of a launch usually share an allocation.
bool on_device(const void* p, size_t bytes, int device, uintptr_t& base, size_t& size) {
  const uintptr_t u = (uintptr_t)p;
  auto inside = [&]() { return u >= base && u - base <= size && bytes <= size - (u - base); };
  if (size && inside()) return true;
  hipPointerAttribute_t at;
  hipDeviceptr_t b = nullptr;
  size_t n = 0;
  if (hipPointerGetAttributes(&at, p) != hipSuccess || hipMemGetAddressRange(&b, &n, (hipDeviceptr_t)p) != hipSuccess) {
    (void)hipGetLastError();  // not memory that HIP knows: the copy call will say so
    return false;
  }
  if (at.type != hipMemoryTypeDevice || at.device != device) return false;
  base = (uintptr_t)b;
  size = n;
  return inside();
}

// Whether an image lies where another one is to go: the copies then have to be made one after the other, in image order.
bool meets_destination(const Request& r, const void* dst) {
  uintptr_t to = (uintptr_t)dst;
  const uintptr_t first = to, end = to + r.total;
  for (const Piece& p : r.pieces) {
    const uintptr_t from = (uintptr_t)p.ptr;
    if (from != to && from < end && from + p.bytes > first) return true;
    to += p.bytes;
  }
  return false;
}
}  // namespace

extern "C" {

vit_status_t vit_handoff_create(int device, vit_handoff_t** out) {
  if (!out || device < 0) return set_error(VIT_EINVAL, "vit_handoff_create: bad argument");
  vit_handoff_t* h = new (std::nothrow) vit_handoff_t;
  if (!h) return set_error(VIT_ENOMEM, "vit_handoff_create: out of host memory");
  h->device = device;
  *out = h;
  return VIT_OK;
}

void vit_handoff_destroy(vit_handoff_t* h) {
  if (!h) return;
  for (auto& kv : h->requests) drop(kv.second);
  delete h;
}

vit_status_t vit_handoff_expect(vit_handoff_t* h, int64_t request_id, int32_t n_images) {
  if (!h || n_images <= 0 || n_images > 65536)
    return set_error(VIT_EINVAL, "vit_handoff_expect: need a handle and 1 <= n_images <= 65536");
  std::lock_guard<std::mutex> lock(h->mu);
  if (h->requests.count(request_id)) return set_error(VIT_EINVAL, "vit_handoff_expect: request %lld is already known", (long long)request_id);
  try {
    h->requests[request_id].pieces.resize((size_t)n_images);
  } catch (...) {  // out of host memory: nothing of the request stays behind
    h->requests.erase(request_id);
    return set_error(VIT_ENOMEM, "vit_handoff_expect: out of host memory for %d images", n_images);
  }
  return VIT_OK;
}

vit_status_t vit_handoff_publish(vit_handoff_t* h, int64_t request_id, int32_t image_index, const void* tokens,
                                 size_t bytes, void* stream) {
  if (!h || !tokens || bytes == 0) return set_error(VIT_EINVAL, "vit_handoff_publish: bad argument");
  std::lock_guard<std::mutex> lock(h->mu);
  auto it = h->requests.find(request_id);
  if (it == h->requests.end()) return set_error(VIT_EINVAL, "vit_handoff_publish: unknown request %lld", (long long)request_id);
  Request& r = it->second;
  if (image_index < 0 || (size_t)image_index >= r.pieces.size())
    return set_error(VIT_EINVAL, "vit_handoff_publish: image %d outside the %zu images expected", image_index, r.pieces.size());
  Piece& p = r.pieces[(size_t)image_index];
  if (p.published) return set_error(VIT_EINVAL, "vit_handoff_publish: image %d was already published", image_index);
  hipError_t e = hipSetDevice(h->device);
  // An event costs its stream 4 us on the GPU, in which neither the stream nor a consumer that waits for it gets on:
  // 130 us for the 32 images of a request.  Tokens that are there already need none.
  const bool busy = r.busy || (e == hipSuccess && !finished((hipStream_t)stream, h->device));
  if (e == hipSuccess && busy) {
    e = hipEventCreateWithFlags(&p.ready, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventRecord(p.ready, (hipStream_t)stream);
  }
  if (e != hipSuccess) {
    if (p.ready) (void)hipEventDestroy(p.ready);
    p.ready = nullptr;
    return set_error(VIT_EDEVICE, "vit_handoff_publish: %s", hipGetErrorString(e));
  }
  r.busy = busy;
  r.captured = r.captured || (busy && capturing((hipStream_t)stream));
  p.ptr = tokens;
  p.bytes = bytes;
  p.published = true;
  r.published += 1;
  r.total += bytes;
  return VIT_OK;
}

int32_t vit_handoff_complete(vit_handoff_t* h, int64_t request_id, size_t* total_bytes) {
  if (!h) return 0;
  std::lock_guard<std::mutex> lock(h->mu);
  auto it = h->requests.find(request_id);
  if (it == h->requests.end()) return 0;
  if (total_bytes) *total_bytes = it->second.total;
  return it->second.published == (int)it->second.pieces.size() ? 1 : 0;
}

vit_status_t vit_handoff_pull(vit_handoff_t* h, int64_t request_id, void* dst, size_t capacity, void* stream,
                              size_t* bytes) {
  if (!h || !dst) return set_error(VIT_EINVAL, "vit_handoff_pull: bad argument");
  std::lock_guard<std::mutex> lock(h->mu);
  auto it = h->requests.find(request_id);
  if (it == h->requests.end()) return set_error(VIT_EINVAL, "vit_handoff_pull: unknown request %lld", (long long)request_id);
  Request& r = it->second;
  if (r.published != (int)r.pieces.size())
    return set_error(VIT_ENOTREADY, "vit_handoff_pull: %d of %zu images published", r.published, r.pieces.size());
  if (r.total > capacity) return set_error(VIT_ECAPACITY, "vit_handoff_pull: %zu bytes needed, %zu given", r.total, capacity);
  hipStream_t s = (hipStream_t)stream;
  hipError_t e = hipSetDevice(h->device);
  auto wait = [&](const Piece& p) {
    if (e == hipSuccess && p.ready) e = hipStreamWaitEvent(s, p.ready, 0);
  };
  auto copy = [&](const Piece& p, unsigned char* to) {
    if (e == hipSuccess) e = hipMemcpyAsync(to, p.ptr, p.bytes, hipMemcpyDeviceToDevice, s);
  };
  uintptr_t base = 0;
  size_t size = 0;
  if (e == hipSuccess && stream_of(s, h->device) && on_device(dst, r.total, h->device, base, size) && !meets_destination(r, dst)) {
    // Images whose producer has finished are gathered at once; the others behind their own events, in groups of half of
    // what is left but at least kGroupBytes, so that what comes out of an earlier launch is moved before the last
    // launch ends.  32 images of 4.7 MB are there, after the event that the last one waits for: 21 us if the others come
    // from an earlier launch and 17 if they are finished (64 behind all events at once, 19 with a copy and an event per
    // image), 220 if all come from one launch (221 and 266: their events take 4 us each).  Groups of 16 MB throughout
    // cost that last case 20 us, of at least 8 MB 8 us.
    // In captures nothing is asked and everything waits.
    bool ask = !r.captured && !capturing(s);
    size_t left = 0;  // bytes of late images that no group holds yet
    {
      RelaxedCapture relaxed;
      ask = ask && relaxed.ok;
      for (Piece& p : r.pieces) {
        p.late = ask && p.ready && hipEventQuery(p.ready) != hipSuccess;
        if (p.late) (void)hipGetLastError();  // "not ready" is an answer
        if (p.late) left += p.bytes;
      }
    }
    if (!ask)
      for (const Piece& p : r.pieces) wait(p);
    GatherArgs g;
    g.n = 0;
    g.first_chunk[0] = 0;
    size_t group = 0;
    auto flush = [&]() {
      if (e == hipSuccess && g.n > 0) {
        hipLaunchKernelGGL(gather_kernel, dim3((unsigned)g.first_chunk[g.n]), dim3(256), 0, s, g);
        e = hipGetLastError();
      }
      g.n = 0;
      group = 0;
    };
    base = size = 0;
    for (const bool late : {false, true}) {
      unsigned char* to = (unsigned char*)dst;
      for (const Piece& p : r.pieces) {
        if (p.late == late && e == hipSuccess) {
          if (late) {
            wait(p);
            left -= p.bytes;
          }
          if ((((uintptr_t)p.ptr | (uintptr_t)to) & 15) == 0 && on_device(p.ptr, p.bytes, h->device, base, size)) {
            g.src[g.n] = (const unsigned char*)p.ptr;
            g.dst[g.n] = to;
            g.bytes[g.n] = p.bytes;
            g.first_chunk[g.n + 1] = g.first_chunk[g.n] + (int32_t)((p.bytes + kGatherChunk - 1) / kGatherChunk);
            group += p.bytes;
            if (++g.n == kGatherPieces || (late && group >= kGroupBytes && group >= left)) flush();
          } else {
            copy(p, to);
          }
        }
        to += p.bytes;
      }
      flush();
    }
  } else {
    unsigned char* to = (unsigned char*)dst;
    for (const Piece& p : r.pieces) {
      wait(p);
      copy(p, to);
      to += p.bytes;
    }
  }
  if (e != hipSuccess) return set_error(VIT_EDEVICE, "vit_handoff_pull: %s", hipGetErrorString(e));
  if (bytes) *bytes = r.total;
  return VIT_OK;
}

vit_status_t vit_handoff_release(vit_handoff_t* h, int64_t request_id) {
  if (!h) return set_error(VIT_EINVAL, "vit_handoff_release: NULL handle");
  std::lock_guard<std::mutex> lock(h->mu);
  auto it = h->requests.find(request_id);
  if (it == h->requests.end()) return set_error(VIT_EINVAL, "vit_handoff_release: unknown request %lld", (long long)request_id);
  drop(it->second);
  h->requests.erase(it);
  return VIT_OK;
}

}  // extern "C"
