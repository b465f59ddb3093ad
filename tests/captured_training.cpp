// Launches of the trainer's calls, printed as "batch steps eager|captured: grid x
// block (c: cooperative) ...".  Captured calls allocate and wait for nothing.
#include "host_runtime.h"

#include <cstdio>
#include <vector>

#include "pdd.h"

static int refused = 0;

hipError_t note(const char* what) {
  if (capturing && what[0] == 'h' && what[3] != 'E') {
    ++refused;
    std::printf(" %s!", what);
  }
  return hipSuccess;
}
hipError_t launched(dim3 grid, dim3 block, bool cooperative) {
  std::printf(" %ux%u%s", grid.x, block.x, cooperative ? "c" : "");
  return hipSuccess;
}

int main() {
  std::vector<float> f(3 * PDD_MLP_PARAMS), xy(2 * 20000), t(20000);
  std::vector<int32_t> order(20000);
  float* p = f.data();
  for (int batch : {32, 96, 128, 256, 1024, 4096, 20000}) {
    pdd_ctx* ctx;
    if (pdd_create(&ctx, 0, nullptr) != PDD_OK) return 2;
    for (int call = 0; call < 4; ++call) {          // captured on a fresh context, eager, captured, one eager step
      const int steps = call == 3 ? 1 : 2;
      capturing = call == 0 || call == 2;
      std::printf("%d %d %s:", batch, steps, call == 0 ? "fresh" : capturing ? "captured" : "eager");
      if (pdd_mlp_train(ctx, p, p + PDD_MLP_PARAMS, p + 2 * PDD_MLP_PARAMS, 20000, xy.data(), t.data(), order.data(), 20000,
                        batch, steps, 0, 1e-3f, nullptr) != PDD_OK)
        return 3;
      std::printf("\n");
    }
    capturing = false;
    pdd_destroy(ctx);
  }
  return refused ? 1 : 0;
}
