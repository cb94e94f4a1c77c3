// The one-shot timing request behind aura_time_next_fusion: a pair of events that the next launch of a
// fusion kernel (made by the same host thread) records on its stream right before and right after itself.
#pragma once

#include <hip/hip_runtime.h>

namespace aura {

struct TimingRequest {
  hipEvent_t start = nullptr, stop = nullptr;
};

// Returns this thread's pending request and clears it (both events null when there is none).
TimingRequest take_timing_request();

// Records this thread's pending request around its own lifetime: the second event on every way out, also where a launch in between
// fails (a caller may wait for it).
class TimedLaunch {
 public:
  explicit TimedLaunch(hipStream_t stream) : request_(take_timing_request()), stream_(stream) {
    if (request_.start) (void)hipEventRecord(request_.start, stream_);
  }
  ~TimedLaunch() {
    if (request_.stop) (void)hipEventRecord(request_.stop, stream_);
  }
  TimedLaunch(const TimedLaunch&) = delete;
  TimedLaunch& operator=(const TimedLaunch&) = delete;

 private:
  const TimingRequest request_;
  const hipStream_t stream_;
};

}  // namespace aura
