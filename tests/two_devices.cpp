// Two contexts on two devices, the other one current: what the library
// allocates, creates and launches for a context has to be on its device.  The
// program stands in for the HIP runtime (its definitions come before the
// library's), so it runs without a GPU: kernels are not run, and device memory
// is host memory.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "pdd.h"

namespace {
int current = 0, wanted = 0, made = 0, wrong = 0;

hipError_t note(const char* what) {
  ++made;
  if (current != wanted) {
    ++wrong;
    std::printf("%s on device %d instead of %d\n", what, current, wanted);
  }
  return hipSuccess;
}
template <typename T>
hipError_t give(T** p, size_t bytes, const char* what) {
  *p = static_cast<T*>(std::calloc(1, bytes ? bytes : 1));
  return note(what);
}
}  // namespace

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
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return note("hipFuncSetAttribute"); }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return note("launch"); }
hipError_t hipLaunchCooperativeKernel(const void*, dim3, dim3, void**, unsigned, hipStream_t) { return note("cooperative launch"); }
}

int main() {
  pdd_ctx* ctx[2];
  for (int d = 0; d < 2; ++d) {
    wanted = d;
    if (pdd_create(&ctx[d], d, nullptr) != PDD_OK) return 2;
  }
  std::vector<float> f(4 * PDD_MLP_PARAMS), xy(2 * 70000), t(70000);
  std::vector<int32_t> order(70000);
  float* p = f.data();
  bool ok = true;
  for (int d = 0; d < 2; ++d) {
    for (int batch : {32, 256, 1300, 66000}) {
      wanted = d;
      current = 1 - d;
      ok &= pdd_mlp_train(ctx[d], p, p + PDD_MLP_PARAMS, p + 2 * PDD_MLP_PARAMS, 70000, xy.data(), t.data(), order.data(),
                          70000, batch, 3, 0, 1e-3f, nullptr) == PDD_OK;
      current = 1 - d;
      ok &= pdd_mlp_grad(ctx[d], p, batch, xy.data(), t.data(), p + 3 * PDD_MLP_PARAMS, nullptr) == PDD_OK;
    }
  }
  for (int d = 0; d < 2; ++d) pdd_destroy(ctx[d]);
  std::printf("%d made, %d on the wrong device\n", made, wrong);
  return !ok ? 3 : wrong || made < 50 ? 1 : 0;
}
