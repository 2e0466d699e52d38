// hip_shim.cpp -- stands in for the HIP runtime in a process without a GPU: kernel launches are counted, one of them can be
// made to fail, and nothing is run (tests/test_launch_errors.py).
#include <cstddef>
#include <cstdint>

struct dim3 { uint32_t x, y, z; };
namespace {
int launches = 0, fail_at = 0, last_error = 0;
char symbol[1 << 20] __attribute__((aligned(256)));
}  // namespace

extern "C" {
void shim_arm(int nth) { launches = 0; fail_at = nth; last_error = 0; }   // the nth launch from here fails (0: none)
int shim_launches() { return launches; }

int hipGetDevice(int* dev) { *dev = 0; return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = symbol; return 0; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
int __hipPushCallConfiguration(dim3, dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, void** stream) {
  *grid = *block = dim3{1, 1, 1};
  *shmem = 0;
  *stream = nullptr;
  return 0;
}
int hipLaunchKernel(const void*, dim3, dim3, void**, size_t, void*) {
  ++launches;
  return last_error = launches == fail_at ? 719 /* hipErrorLaunchFailure */ : 0;
}
}
