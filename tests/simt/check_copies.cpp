// A copy to LDS seen too early and in time: only the wait brings the data.
#include <hip/hip_runtime.h>
#include "gear_internal.h"
static uint32_t source[4 * 64], early[64], late[64];
static void kernel() {
  __shared__ uint4 tile[64];
  const GEAR_BUF_T b = GEAR_BUF_MAKE(source, sizeof source);
  const int lane = simt::lane();
  GEAR_DMA16(b, lane * 16, tile);
  early[lane] = tile[lane].x;
  GEAR_DMA_WAIT();
  late[lane] = tile[63 - lane].x;
}
int main() {
  for (int i = 0; i < 4 * 64; ++i) source[i] = 1000 + i;
  hipLaunchKernelGGL(kernel, dim3(1), dim3(64), 0, nullptr);
  for (int l = 0; l < 64; ++l) {
    if (late[l] != source[4 * (63 - l)]) { fprintf(stderr, "lane %d: %u after the wait\n", l, late[l]); return 1; }
    if (early[l] == source[4 * l]) { fprintf(stderr, "lane %d has the data before the wait\n", l); return 1; }
  }
  return 0;
}
