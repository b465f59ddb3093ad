// Functions in the place of the HIP runtime's for programs that drive the library
// without a GPU (a program's definitions come before the library's): kernels are
// not run, device memory is host memory.  `note` and `launched` are the program's.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>

hipError_t note(const char* what);
hipError_t launched(dim3 grid, dim3 block, bool cooperative);

static int current = 0;               // device
static bool capturing = false;

template <typename T>
static hipError_t give(T** p, size_t bytes, const char* what) {
  *p = static_cast<T*>(std::calloc(1, bytes ? bytes : 1));
  return note(what);
}

extern "C" {
hipError_t hipGetDeviceCount(int* n) { *n = 2; return hipSuccess; }
hipError_t hipSetDevice(int d) { current = d; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) { static char word[256]; *p = word; return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return give(p, n, "hipHostMalloc"); }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { return give(p, n, "hipMalloc"); }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* to, const void* from, size_t n, hipMemcpyKind) { std::memcpy(to, from, n); return note("hipMemcpy"); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(&current); return note("event"); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return note("hipEventRecord"); }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return note("hipStreamSynchronize"); }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
static dim3 pushed_grid, pushed_block;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
  pushed_grid = grid;
  pushed_block = block;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = pushed_grid;
  *block = pushed_block;
  *lds = 0;
  *stream = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
  return launched(grid, block, false);
}
hipError_t hipLaunchCooperativeKernel(const void*, dim3 grid, dim3 block, void**, unsigned, hipStream_t) {
  return launched(grid, block, true);
}
}
