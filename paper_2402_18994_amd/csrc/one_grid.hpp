// Order between launches whose workgroups wait for each other.
//
// Two such grids must not share the compute units half and half: each would hold what the other's missing
// workgroups need.  They are therefore ordered one behind the other on a device, whatever streams of this
// process they are on, by an event per device.  A stream that is being captured cannot be ordered (its launches
// run whenever the graph is replayed, beside whatever else runs then), and a call that fails orders nothing.
// `ordered()` says whether a launch may
// wait for its own workgroups; if not, it must be one that waits for nothing.
#pragma once
#include <hip/hip_runtime_api.h>

#include <mutex>

namespace snn {

class OneGridAtATime {
 public:
  // `wanted`: false leaves the streams alone (ordered() is false then).
  OneGridAtATime(hipStream_t st, bool wanted) : st_(st) {
    if (!wanted) return;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    int dev = 0;
    bool ok = hipStreamIsCapturing(st, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone && hipGetDevice(&dev) == hipSuccess &&
              dev >= 0 && dev < MAX_DEVICES;
    if (ok) {
      lock_ = std::unique_lock<std::mutex>(mutex());
      hipEvent_t &ev = events()[dev];
      if (ev) ok = hipStreamWaitEvent(st, ev, 0) == hipSuccess;
      else if (!(ok = hipEventCreateWithFlags(&ev, hipEventDisableTiming) == hipSuccess)) ev = nullptr;
      if (ok) ev_ = ev;
      else lock_.unlock();
    }
    if (!ok) (void)hipGetLastError();                     // (the launch that follows checks for its own errors)
  }
  // The next grid waits for what the stream holds now; without the record, the host does so here.
  ~OneGridAtATime() {
    if (!ev_ || hipEventRecord(ev_, st_) == hipSuccess) return;
    (void)hipGetLastError();
    (void)hipStreamSynchronize(st_);
  }
  OneGridAtATime(const OneGridAtATime &) = delete;
  OneGridAtATime &operator=(const OneGridAtATime &) = delete;
  bool ordered() const { return ev_ != nullptr; }

 private:
  static constexpr int MAX_DEVICES = 64;
  static std::mutex &mutex() { static std::mutex m; return m; }
  static hipEvent_t *events() { static hipEvent_t e[MAX_DEVICES] = {}; return e; }
  hipStream_t st_;
  std::unique_lock<std::mutex> lock_;                     // (held until after the record)
  hipEvent_t ev_ = nullptr;
};

}  // namespace snn
