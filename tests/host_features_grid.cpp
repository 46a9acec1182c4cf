// Host replay of eodabe_features: prints the grid of its launch for the sizes
// given as arguments (pixels, rank pairs).  No device is touched.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>

static dim3 launched;
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kern, grid, ...) (launched = (grid))
#define hipGetLastError() hipSuccess
#include "eodabe.hip"

int main() {
  eodabe_ctx ctx{};
  eodabe_default_opts(&ctx.o);
  for (int64_t m : {1, 63, 64, 65, 300, 1024, 4096, 5001, 16384, 65536, 262144, 1000003})
    for (int64_t r : {1, 15, 16, 17, 33, 64, 100, 200, 500, 1000, 4000}) {
      if (r > m) continue;
      if (eodabe_features(&ctx, (const float*)4096, (const float*)4096, m, r, r, (float*)4096, r) != 0) return 1;
      printf("%ld %ld %u %u %u\n", (long)m, (long)r, launched.x, launched.y, launched.z);
    }
  return 0;
}
