// Host-only stand-in for kernel launches and copies (with mock_hip.cpp): the
// kernels do not run; every launch is kept with its kernel's name, grid and
// arguments, and what a copy to the host brings is set by the test.
#include <hip/hip_runtime.h>

#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "mock_launch.h"

namespace mock {
std::vector<Launch>& launches() {
  static std::vector<Launch> v;
  return v;
}
std::function<void(void*, size_t)>& readback() {
  static std::function<void(void*, size_t)> f;
  return f;
}
}  // namespace mock

namespace {
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t st;
};
thread_local Config g_config;
void* g_handle = nullptr;
}  // namespace

extern "C" {
char mock_fatbin[16];
void** __hipRegisterFatBinary(const void*) { return &g_handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*,
                           int*) {
  names()[host] = device;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st) {
  g_config = {grid, block, lds, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st) {
  *grid = g_config.grid;
  *block = g_config.block;
  *lds = g_config.lds;
  *st = g_config.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
  mock::launches().push_back({names()[f], grid, block});
  for (auto& hook : mock::hooks())
    if (mock::launches().back().name.find(hook.first) != std::string::npos) hook.second(args);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void*, size_t n, hipMemcpyKind kind, hipStream_t) {
  if (kind == hipMemcpyDeviceToHost) {
    std::memset(dst, 0, n);
    if (mock::readback()) mock::readback()(dst, n);
  }
  return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
}  // extern "C"

namespace mock {
std::map<std::string, std::function<void(void**)>>& hooks() {
  static std::map<std::string, std::function<void(void**)>> m;
  return m;
}
}  // namespace mock
