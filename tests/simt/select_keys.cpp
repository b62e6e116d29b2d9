// The Key selection alone: for each line "file slabs n ppm per_vector" of standard input, the keys of `file` (fp16 [slabs][n][128]) through
// launch_k_select, the mask (16 bytes per row) to file.mask and, with per-vector groups, the channels' (scale, zero) to file.sz.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <vector>
#include "gear_launch.h"
int main() {
  using namespace gear;
  char file[400];
  int slabs, n, ppm, kcvt;
  while (scanf("%399s %d %d %d %d", file, &slabs, &n, &ppm, &kcvt) == 5) {
    uint16_t* K = static_cast<uint16_t*>(aligned_alloc(16, (size_t)slabs * n * D * 2));   // exact sizes: the sanitizer sees a step beyond
    FILE* f = fopen(file, "rb");
    if (!f || fread(K, 1, (size_t)slabs * n * D * 2, f) != (size_t)slabs * n * D * 2) return 2;
    fclose(f);
    uint4* mask = static_cast<uint4*>(aligned_alloc(16, (size_t)slabs * n * 16));
    memset(mask, 0xEE, (size_t)slabs * n * 16);
    std::vector<uint32_t> sz((size_t)slabs * D), zero(1000, 7u);
    std::vector<uint16_t> kt((size_t)slabs * D * ((n + 7) & ~7));
    Dims dm;
    memset(&dm, 0, sizeof dm);
    dm.B = 1;
    dm.H = dm.Hq = slabs;
    dm.bits = 2;
    dm.g = D;
    dm.kcvt = kcvt;
    dm.ppm = ppm;
    dm.qmax = 3.0f;
    SegView sv;
    memset(&sv, 0, sizeof sv);
    sv.sz = sz.data();
    sv.n = sv.n_cap = n;
    sv.ng_cap = 1;
    const int k = (int)(((long long)ppm * n + 999999) / 1000000);
    simt::observer = [](const char* kernel, dim3, dim3, size_t) { printf("launch %s\n", kernel + (kernel[0] == '(')); };
    if (launch_k_select(K, dm, n, (k + 1) / 2, k / 2, mask, zero.data(), (int)zero.size(), sv, kt.data(), nullptr) != hipSuccess) return 3;
    for (uint32_t z : zero)
      if (z != 0u) return 4;
    char out[420];
    snprintf(out, sizeof out, "%s.mask", file);
    f = fopen(out, "wb");
    fwrite(mask, 16, (size_t)slabs * n, f);
    fclose(f);
    snprintf(out, sizeof out, "%s.sz", file);
    f = fopen(out, "wb");
    fwrite(sz.data(), 4, sz.size(), f);
    fclose(f);
    free(K);
    free(mask);
  }
  return 0;
}
