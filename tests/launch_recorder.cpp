// Stands in for the HIP runtime's launch calls, so that a process without a GPU sees which kernels an entry point would launch: loaded
// with RTLD_GLOBAL before the library, its hipLaunchKernel is the one that the library finds. Nothing is executed.
#include <cxxabi.h>
#include <dlfcn.h>

#include <cstdint>
#include <cstdlib>
#include <string>

namespace {
struct Dim3 {
  uint32_t x, y, z;
};
std::string launches;  // "kernel|workgroups x|workgroups y|threads\n", one line per launch since the last call of recorded()
thread_local struct {
  Dim3 grid, block;
  size_t shared;
  void* stream;
} pushed;
}  // namespace

extern "C" {
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t, void*) {
  Dl_info info;
  const char* name = dladdr(f, &info) && info.dli_saddr == f ? info.dli_sname : "?";
  int status = 0;
  char* plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  launches += std::string(plain ? plain : name) + "|" + std::to_string(grid.x) + "|" + std::to_string(grid.y) + "|" +
              std::to_string(block.x) + "\n";
  free(plain);
  return 0;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void* stream) {
  pushed = {grid, block, shared, stream};
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream) {
  *grid = pushed.grid, *block = pushed.block, *shared = pushed.shared, *stream = pushed.stream;
  return 0;
}
int hipGetLastError() { return 0; }

const char* recorded() {
  static std::string last;
  last.swap(launches);
  launches.clear();
  return last.c_str();
}
}
