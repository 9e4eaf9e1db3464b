// Stands in for the HIP runtime where there is no GPU: loaded ahead of libfastkv_select.so it takes the library's runtime calls,
// writes down each kernel launch and runs none.  Device memory is host memory that nothing reads.
#include <cxxabi.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

#include "fkv_internal.h"

namespace {
struct Launch {
  std::string kernel;
  unsigned grid[3], block;
  unsigned long long wait_ticks;  // of kernels that wait for other blocks
};
std::map<const void *, std::string> &kernels() {
  static std::map<const void *, std::string> m;
  return m;
}
std::vector<Launch> launches;
int fail_at = -1;  // launch that is refused, counted from the last reset
dim3 next_grid, next_block;
size_t next_shared;
hipStream_t next_stream;
}  // namespace

extern "C" {

void recorder_reset(int refuse) {
  launches.clear();
  fail_at = refuse;
}
int recorder_launches(void) { return (int)launches.size(); }
const char *recorder_kernel(int i) { return launches[i].kernel.c_str(); }
unsigned recorder_blocks(int i) { return launches[i].grid[0] * launches[i].grid[1] * launches[i].grid[2]; }
unsigned recorder_threads(int i) { return launches[i].block; }
unsigned long long recorder_wait_ticks(int i) { return launches[i].wait_ticks; }

void **__hipRegisterFatBinary(const void *) {
  static void *handle;
  return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *, int *) {
  int status = 0;
  char *plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  std::string s = status == 0 && plain ? plain : name;
  free(plain);
  kernels()[host] = s.substr(0, s.find('('));
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
  next_grid = grid;
  next_block = block;
  next_shared = shared;
  next_stream = stream;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *stream) {
  *grid = next_grid;
  *block = next_block;
  *shared = next_shared;
  *stream = next_stream;
  return hipSuccess;
}

static hipError_t last_error = hipSuccess;
hipError_t hipGetLastError(void) {
  const hipError_t e = last_error;
  last_error = hipSuccess;
  return e;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t, hipStream_t) {
  if ((int)launches.size() == fail_at) {
    fail_at = -1;
    return last_error = hipErrorLaunchFailure;
  }
  Launch l{kernels()[f], {grid.x, grid.y, grid.z}, block.x * block.y * block.z, 0};
  auto has = [&](const char *name) { return l.kernel.find(name) != std::string::npos; };
  if (has("k_wout_partial")) l.wait_ticks = static_cast<const fkv::WoutArgs *>(args[0])->timeout_ticks;
  if (has("k_score_fused") || has("k_score_keep")) l.wait_ticks = static_cast<const fkv::FusedArgs *>(args[1])->timeout_ticks;
  launches.push_back(l);
  return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n) {
  *p = aligned_alloc(256, (n + 255) / 256 * 256);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) {
  free(p);
  return hipSuccess;
}
hipError_t hipMemset(void *p, int v, size_t n) {
  memset(p, v, n);
  return hipSuccess;
}
hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind) {
  memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int *dev) {
  *dev = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  memset(p, 0, sizeof *p);
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) {
  static void *scratch = aligned_alloc(256, 8 << 20);
  *p = scratch;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) {
  *e = reinterpret_cast<hipEvent_t>(malloc(1));
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
  free(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = 0.001f;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }

}  // extern "C"
