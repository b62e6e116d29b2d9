// Calls whose kernels ask for more than 64 KB of dynamic LDS, on one device after another of a process: each is accepted on every
// device.  Launches end at the stand-in (the pointers are not memory).
#include <stdio.h>
#include <string.h>
#include <hip/hip_runtime.h>
#include "gear.h"
static size_t most;
int main() {
  simt::dry = true;
  simt::observer = [](const char*, dim3, dim3, size_t lds) { most = lds > most ? lds : most; };
  void* const p = reinterpret_cast<void*>(uintptr_t(1) << 40);
  struct { const char* what; gear_config cfg; int n, rank; bool read; } cases[] = {
      {"Key selection by lists", {1, 32, 32, 128, 2, 128, 10000, 64, 32768, 1, 0, 0}, 32768, 0, false},
      {"low-rank solver", {1, 4, 4, 128, 2, 64, 0, 64, 1000, 1, 8, 0}, 1000, 8, false},
      {"read in one launch", {64, 8, 32, 128, 4, 64, 20000, 20, 1400, 1, 4, 0}, 1400, 0, true},
  };
  int bad = 0;
  for (auto& c : cases)
    for (int dev = 0; dev < 3; ++dev) {
      hipSetDevice(dev);
      gear_cache cache;
      size_t arena = 0, work = 0;
      if (gear_cache_bytes(&c.cfg, &arena, &work) != GEAR_OK || gear_cache_init(&c.cfg, p, arena, &cache) != GEAR_OK) return 2;
      most = 0;
      int s = gear_compress(&cache, p, p, c.n, c.rank, 3, nullptr, 1, p, work, nullptr);
      if (c.read) {
        most = 0;
        if (s == GEAR_OK) s = gear_decode_attn(&cache, p, p, p, 9, p, p, work, nullptr);
      }
      if (s != GEAR_OK || most <= 64 * 1024) {
        fprintf(stderr, "%s, device %d: %s, %zu bytes of LDS\n", c.what, dev, gear_strerror(s), most);
        bad = 1;
      }
    }
  return bad;
}
