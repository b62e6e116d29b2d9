// How reads are launched: for each line "bits group B H_kv H_q n rank n_buf n_buf_cap chunks" of standard input, a line with the
// kernel, the blocks that share a slab's query columns and the dynamic LDS.  Nothing runs (the pointers are not memory).
#include <stdio.h>
#include <string.h>
#include <hip/hip_runtime.h>
#include "gear.h"
static int slabs;
int main() {
  simt::dry = true;
  void* const p = reinterpret_cast<void*>(uintptr_t(1) << 40);
  gear_config c;
  memset(&c, 0, sizeof c);
  c.d_h = 128;
  c.outlier_ppm = 20000;
  int n, rank, n_buf, chunks;
  while (scanf("%d %d %d %d %d %d %d %d %d %d", &c.bits, &c.group, &c.B, &c.H_kv, &c.H_q, &n, &rank, &n_buf, &c.n_buf_cap, &chunks) == 10) {
    c.n_prefill_max = n;
    c.n_chunks_max = chunks;
    c.rank_max = rank;
    gear_cache cache;
    size_t arena = 0, work = 0;
    if (gear_cache_bytes(&c, &arena, &work) != GEAR_OK || gear_cache_init(&c, p, arena, &cache) != GEAR_OK) return 2;
    simt::observer = nullptr;
    if (gear_compress(&cache, p, p, n, rank, 1, nullptr, 1, p, work, nullptr) != GEAR_OK) return 3;
    for (int j = 0; j < chunks; ++j)
      if (gear_compress(&cache, p, p, c.n_buf_cap, rank, 1, nullptr, 1, p, work, nullptr) != GEAR_OK) return 4;
    slabs = c.B * c.H_kv;
    simt::observer = [](const char* kernel, dim3 grid, dim3, size_t lds) {
      if (strstr(kernel, "single")) printf("single %u %zu\n", grid.x / slabs, lds);
      else if (strstr(kernel, "split")) printf("split %u %zu\n", grid.y / slabs, lds);
    };
    if (gear_decode_attn(&cache, p, p, p, n_buf, p, p, work, nullptr) != GEAR_OK) return 5;
  }
  return 0;
}
