// A setting that is made once on each device of the process, such as a
// kernel's LDS limit: the first call on a device makes it, every call on that
// device returns what that gave (a failure too).  Safe with several threads.
#pragma once
#include <mutex>

namespace lat {

template <typename R>
class PerDevice {
 public:
  static constexpr int MAX = 64;
  template <typename F>
  R get(int device, F make) {
    if (device < 0 || device >= MAX) return make();
    std::call_once(once_[device], [&] { result_[device] = make(); });
    return result_[device];
  }

 private:
  std::once_flag once_[MAX];
  R result_[MAX] = {};
};

}  // namespace lat
