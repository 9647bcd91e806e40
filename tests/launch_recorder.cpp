// Stands in for the HIP calls that libdpia.so makes to launch a kernel: every
// launch is kept (kernel, grid, work-group, LDS) and nothing is run, so that
// which launch a call leads to can be looked at without a GPU.
#include <dlfcn.h>

#include <cstddef>
#include <cstdint>
#include <vector>

namespace {
struct Dim {
  uint32_t x, y, z;
};
struct Launch {
  const void* kernel;
  uint64_t grid, block, lds;
};
std::vector<Launch> launches;
}  // namespace

extern "C" {
int hipLaunchKernel(const void* f, Dim grid, Dim block, void**, size_t lds, void*) {
  launches.push_back({f, grid.x, block.x, lds});
  return 0;
}
int hipGetDevice(int* dev) { return *dev = 0; }
int hipDeviceGetAttribute(int* value, int, int) {   // (compute units are all that is asked for)
  *value = 256;
  return 0;
}
int launches_made() { return static_cast<int>(launches.size()); }
void launches_clear() { launches.clear(); }
uint64_t launch_grid(int i) { return launches[i].grid; }
uint64_t launch_block(int i) { return launches[i].block; }
uint64_t launch_lds(int i) { return launches[i].lds; }
const char* launch_kernel(int i) {
  Dl_info info;
  return dladdr(launches[i].kernel, &info) && info.dli_sname ? info.dli_sname : "";
}
}
