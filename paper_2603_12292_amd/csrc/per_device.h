// A value found once for each device of the process.
#pragma once

#include <map>
#include <mutex>

namespace bgl {

// get(dev, make): the value of make() from the first call with `dev`, for which
// the others wait.  (Attributes of a kernel and its occupancy belong to the
// device that is current when they are set or asked for.)
template <class T>
class PerDevice {
  std::mutex mu;
  std::map<int, T> values;

 public:
  template <class F>
  T get(int dev, F make) {
    std::lock_guard<std::mutex> lock(mu);
    const auto it = values.find(dev);
    if (it != values.end()) return it->second;
    return values.emplace(dev, make()).first->second;
  }
};

}  // namespace bgl
