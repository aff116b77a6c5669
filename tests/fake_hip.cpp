// Stand-ins for the HIP runtime calls of plan creation and kernel launches, so
// that the host side of libcgconv.so runs without a GPU: device memory is host
// memory, launches and function attributes are recorded and nothing runs.
// Loaded with global visibility before libcgconv.so (tests/host_runtime.py).
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>

namespace {
struct Launch {
  int64_t grid[3], block[3], lds, allowed;  // allowed: the kernel's dynamic LDS limit at the launch
};
std::vector<Launch> g_launches;
std::map<const void*, int64_t> g_allowed;
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
} g_config;
constexpr int64_t kDefaultLds = 64 * 1024;
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = aligned_alloc(256, (n + 255) / 256 * 256); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute a, int v) {
  if (a == hipFuncAttributeMaxDynamicSharedMemorySize) g_allowed[f] = v;
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  g_config = {grid, block, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = g_config.grid;
  *block = g_config.block;
  *lds = g_config.lds;
  *s = g_config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t lds, hipStream_t) {
  const auto it = g_allowed.find(f);
  g_launches.push_back({{g.x, g.y, g.z}, {b.x, b.y, b.z}, (int64_t)lds, it == g_allowed.end() ? kDefaultLds : it->second});
  return hipSuccess;
}
// the launches since the last call, eight values each; returns their number
int64_t fake_hip_launches(int64_t* out, int64_t cap) {
  const int64_t n = (int64_t)g_launches.size();
  for (int64_t i = 0; i < n && i < cap; ++i) memcpy(out + 8 * i, &g_launches[i], sizeof(Launch));
  g_launches.clear();
  return n;
}
}
