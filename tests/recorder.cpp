// Stand-in for the HIP runtime calls that the library makes, for tests of its
// host code without a GPU: kernel launches are written down instead of made.
// Linked into a host-only build of the library (tests/recorder.py).
#include <hip/hip_runtime_api.h>

#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Launch {
  std::string kernel;
  dim3 grid, block;
  size_t lds;
};
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
};
std::map<const void*, std::string>& kernels() {
  static std::map<const void*, std::string> m;
  return m;
}
std::vector<Launch> launches;
std::vector<Config> configs;
long fail_at = -1;
hipError_t last = hipSuccess;
void* module = nullptr;
}  // namespace

extern "C" {
char __hip_fatbin = 0;
void** __hipRegisterFatBinary(const void*) { return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  kernels()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  configs.push_back({grid, block, lds, stream});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  const Config c = configs.back();
  configs.pop_back();
  *grid = c.grid, *block = c.block, *lds = c.lds, *stream = c.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t lds, hipStream_t) {
  if ((long)launches.size() == fail_at) return last = hipErrorLaunchFailure;
  launches.push_back({kernels()[f], grid, block, lds});
  return hipSuccess;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) { return *d = 0, hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { return *p = const_cast<void*>(s), hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }

// Forget the launches; launch number `fail` (counted from 0; -1: none) will be refused.
void rec_reset(long fail) {
  launches.clear();
  fail_at = fail;
}
long rec_count(void) { return (long)launches.size(); }
// Launch i: its kernel's (mangled) name, and {grid.x, grid.y, block.x, LDS bytes}.
const char* rec_launch(long i, unsigned* out) {
  const Launch& l = launches[(size_t)i];
  out[0] = l.grid.x, out[1] = l.grid.y, out[2] = l.block.x, out[3] = (unsigned)l.lds;
  return l.kernel.c_str();
}
}
