// What the mocked kernel launches leave for the tests (see mock_launch.cpp).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <functional>
#include <map>
#include <string>
#include <vector>

namespace mock {
struct Launch {
  std::string name;  // mangled
  dim3 grid, block;
};
std::vector<Launch>& launches();
// Called with the arguments of every launch whose mangled name holds the key.
std::map<std::string, std::function<void(void**)>>& hooks();
// Fills what a copy to the host brings (zeros before).
std::function<void(void*, size_t)>& readback();
template <class T>
T arg(void** args, int k) {
  return *static_cast<T*>(args[k]);
}
}  // namespace mock
