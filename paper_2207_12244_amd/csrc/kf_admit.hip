// The admission of solver launches (kf_admit.h) over HIP streams and events.
#include "kf_admit.h"

#include "kf_internal.h"

namespace kf {

namespace {

// Calls on other streams than a captured one are legal, but a capture in global
// mode of some other thread objects to an event query unless this one is relaxed.
struct Relaxed {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  bool on;
  Relaxed() : on(hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess) {}
  ~Relaxed() {
    if (on) (void)hipThreadExchangeStreamCaptureMode(&mode);
  }
};

bool good(hipError_t e) {
  if (e == hipSuccess) return true;
  (void)hipGetLastError();
  return false;
}

struct HipOps {
  using Stream = hipStream_t;
  using Event = hipEvent_t;
  int device;
  Stream own = nullptr;   // takes over events of streams that may go (detach)

  template <typename F>
  bool on_device(F&& f) const {
    int cur = -1;
    if (!good(hipGetDevice(&cur)) || (cur != device && !good(hipSetDevice(device)))) return false;
    const bool ok = f();
    if (cur != device) (void)good(hipSetDevice(cur));
    return ok;
  }
  // orders work of this device only, so without the system-scope fence
  bool create(Event& e) const {
    return on_device([&] { return good(hipEventCreateWithFlags(&e, hipEventDisableTiming | hipEventDisableSystemFence)); });
  }
  void destroy(Event& e) const { (void)good(hipEventDestroy(e)); }
  bool record(Event& e, Stream s) const { return !capturing(s) && good(hipEventRecord(e, s)); }
  bool done(Event& e) const {
    Relaxed relaxed;
    const hipError_t r = hipEventQuery(e);
    if (r != hipSuccess) (void)hipGetLastError();
    return r != hipErrorNotReady;
  }
  // An event keeps referring to the stream that it was last recorded on: asked for
  // after that stream is destroyed, the runtime answers at random (seen: that it was
  // recorded in a capture). So a stream of the library's waits for it and records
  // one of its own.
  bool detach(Event& e) {
    Relaxed relaxed;
    if (!own && !on_device([&] { return good(hipStreamCreateWithFlags(&own, hipStreamNonBlocking)); })) own = nullptr;
    Event mine = nullptr;
    if (own && create(mine) && wait(own, e) && good(hipEventRecord(mine, own))) {
      destroy(e);
      e = mine;
      return true;
    }
    if (mine) destroy(mine);
    (void)good(hipEventSynchronize(e));
    return false;
  }
  bool wait(Stream s, Event& e) const { return good(hipStreamWaitEvent(s, e, 0)); }
  // (a per-thread default stream is another one in every thread)
  bool same(Stream a, Stream b) const { return a == b && a != hipStreamPerThread; }
  bool idle(Stream s) const {
    Relaxed relaxed;
    return !capturing(s) && good(hipStreamQuery(s));
  }
  bool capturing(Stream s) const {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    return !good(hipStreamIsCapturing(s, &st)) || st != hipStreamCaptureStatusNone;
  }
};

using Device = Admission<HipOps>;

// One per device for the life of the process (contexts may outlive static objects).
Device* admission_of(int device) {
  constexpr int MAX_DEVICES = 64;
  static std::mutex mu;
  static Device* all[MAX_DEVICES] = {};
  if (device < 0 || device >= MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lock(mu);
  if (!all[device]) all[device] = new (std::nothrow) Device(device_cus(device), HipOps{device, nullptr});
  return all[device];
}

}  // namespace

bool admit_join(kf_ctx* c) {
  if (c->lane) return true;
  Device* d = admission_of(c->device);
  c->lane = d ? d->join(c->solve_stream ? c->solve_stream : c->stream) : nullptr;
  return c->lane != nullptr;
}

hipError_t admit_launch(kf_ctx* c, int blocks, int coresident, hipError_t (*go)(void*), void* arg) {
  return admission_of(c->device)
      ->launch(static_cast<Device::Lane*>(c->lane), blocks, coresident / c->cus, hipSuccess, hipErrorInvalidHandle,
               [&] { return go(arg); });
}

void admit_leave(kf_ctx* c) {
  // (a solve stream of the context's own has been waited for)
  if (c->lane) admission_of(c->device)->leave(static_cast<Device::Lane*>(c->lane), c->solve_stream != nullptr);
  c->lane = nullptr;
}

}  // namespace kf
