// pi_gram_strips_max, by which the workspace is sized, against pi_gram_strip over every length and many slab counts.
#include "gear_launch.h"
int main() {
  using namespace gear;
  for (int slabs = 1; slabs <= 1200; slabs += slabs < 40 ? 1 : slabs < 300 ? 7 : 61) {
    int most = 0, last = 0;
    for (int n = 1; n <= 32768; ++n) {
      const int strip = pi_gram_strip(n, slabs), count = (n + strip - 1) / strip;
      if (strip < last || strip % 128 || strip > 2048) return fprintf(stderr, "strip %d of n %d, %d slabs\n", strip, n, slabs), 1;
      last = strip;
      if (count > most) most = count;
      if (pi_gram_strips_max(n, slabs) != most)
        return fprintf(stderr, "n_max %d, %d slabs: bound %d, strips %d\n", n, slabs, pi_gram_strips_max(n, slabs), most), 1;
    }
  }
  return 0;
}
