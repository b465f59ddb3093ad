// Two contexts on two devices, the other one current: what the library
// allocates, creates and launches for a context has to be on its device.
#include "host_runtime.h"

#include <cstdio>
#include <vector>

#include "pdd.h"

static int wanted = 0, made = 0, wrong = 0;

hipError_t note(const char* what) {
  ++made;
  if (current != wanted) {
    ++wrong;
    std::printf("%s on device %d instead of %d\n", what, current, wanted);
  }
  return hipSuccess;
}
hipError_t launched(dim3, dim3, bool) { return note("launch"); }

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
  for (int d = 0; d < 2; ++d) {
    wanted = d;
    pdd_destroy(ctx[d]);
  }
  std::printf("%d made, %d on the wrong device\n", made, wrong);
  return !ok ? 3 : wrong || made < 50 ? 1 : 0;
}
