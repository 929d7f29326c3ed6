// Limits and attributes of a kernel belong to a device; a process may use several.
#pragma once

#include <hip/hip_runtime_api.h>

#include <map>
#include <mutex>

namespace amg355 {

// find(device) for the current device, found out once for each (any thread); a
// value-initialized result if there is none
template <class F>
auto per_device(F&& find) -> decltype(find(0)) {
    static std::mutex lock;
    static std::map<int, decltype(find(0))> known;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return {};
    const std::lock_guard<std::mutex> guard(lock);
    auto it = known.find(dev);
    if (it == known.end()) it = known.emplace(dev, find(dev)).first;
    return it->second;
}

}  // namespace amg355
