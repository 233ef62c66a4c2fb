/* The HIP entry points that libecrpic calls, on host memory and without a
 * device: copies are memcpy, launches do nothing.  Loaded ahead of the
 * library, it shows what the library's host code does when a launch is
 * refused, and which calls it makes.  Any device pointer is host memory. */
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

namespace {
int launches, refuse_at = -1, syncs, host_allocs, host_frees, mode_changes;
hipError_t last = hipSuccess;
dim3 cfg_grid, cfg_block;
}  // namespace

extern "C" {

/* the launch after n more ones is refused (-1: none) */
void stub_refuse(int n) {
  refuse_at = n < 0 ? -1 : launches + n;
  last = hipSuccess;
}
int stub_launches() { return launches; }
int stub_syncs() { return syncs; }
int stub_host_allocs() { return host_allocs; }
int stub_host_frees() { return host_frees; }

hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) {
  if (launches++ != refuse_at) return hipSuccess;
  return last = hipErrorLaunchFailure;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t) {
  cfg_grid = g;
  cfg_block = b;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shared, hipStream_t *st) {
  *g = cfg_grid;
  *b = cfg_block;
  *shared = 0;
  *st = nullptr;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char *hipGetErrorString(hipError_t) { return "refused by the stub"; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  ++syncs;
  return hipSuccess;
}
/* fresh pinned memory holds anything */
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  ++host_allocs;
  *p = malloc(n);
  memset(*p, 0x5a, n);
  return hipSuccess;
}
hipError_t hipHostFree(void *p) {
  ++host_frees;
  free(p);
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
}
