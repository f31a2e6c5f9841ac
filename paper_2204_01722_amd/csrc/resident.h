// Admission of launches whose workgroups wait for each other.
#pragma once

#include <chrono>
#include <condition_variable>
#include <mutex>

namespace hpmg {

// All workgroups of such a launch have to be resident together, so at most `limit` of them
// (one per compute unit) are let in at a time on a device.  A launch that would exceed that
// waits for earlier ones to leave, other threads' that are read back before they do; what
// those have ahead of them on their streams is not known here, so the wait is bounded and
// the caller takes the form without such waits when admitted() is false.
class ResidentGroups {
 public:
  ResidentGroups(int device, int groups, int limit, double seconds) : device_(device), groups_(groups) {
    if (device < 0 || device >= DEVICES) return;
    State &s = state();
    std::unique_lock<std::mutex> lock(s.mutex);
    admitted_ = s.freed.wait_for(lock, std::chrono::duration<double>(seconds),
                                 [&] { return s.in_use[device_] + groups_ <= limit; });
    if (admitted_) s.in_use[device_] += groups_;
  }
  ~ResidentGroups() {
    if (!admitted_) return;
    State &s = state();
    {
      std::lock_guard<std::mutex> lock(s.mutex);
      s.in_use[device_] -= groups_;
    }
    s.freed.notify_all();
  }
  ResidentGroups(const ResidentGroups &) = delete;
  ResidentGroups &operator=(const ResidentGroups &) = delete;
  bool admitted() const { return admitted_; }

 private:
  static constexpr int DEVICES = 64;
  struct State {
    std::mutex mutex;
    std::condition_variable freed;
    int in_use[DEVICES] = {};
  };
  static State &state() {
    static State s;
    return s;
  }
  int device_, groups_;
  bool admitted_ = false;
};

}  // namespace hpmg
