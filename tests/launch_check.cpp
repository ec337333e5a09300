// Launch geometry for sizes that no test could hold in memory: grids stay under 2^32 work items per
// dimension and 65535 blocks in y, strided blocks cover the work, and the batches of the sliced
// Wasserstein distance fit their kernels' grids.  Built and run by tests/test_launch_cpu.py.
#include <cstdio>
#include <initializer_list>

#include "../paper_2606_04895_amd/csrc/launch.hpp"

using namespace best;

int main() {
  long n = 0;
  for (int sh = 0; sh <= 42; ++sh)
    for (int64_t w : {((int64_t)1 << sh) - 1, (int64_t)1 << sh, ((int64_t)1 << sh) + 1})
      for (int thr : {64, 256, 512, 1024}) {
        const int64_t g = capped_blocks(w, thr);
        if (g < 1 || (w >= 1 && g > w) || g * thr >= (int64_t)1 << 32 || g > 0x7fffffff) {
          std::printf("blocks %ld threads %d -> %ld\n", (long)w, thr, (long)g);
          return 1;
        }
        // block b takes work b, b + g, ...: nothing left out, nothing twice
        if (w >= 1 && g < w && g * thr + thr < (int64_t)1 << 32) {
          std::printf("capped below the limit: %ld of %ld\n", (long)g, (long)w);
          return 1;
        }
        ++n;
      }
  for (int sh = 1; sh <= 31; ++sh)
    for (int64_t draws : {((int64_t)1 << sh) - 1, (int64_t)1 << sh, ((int64_t)1 << sh) + 1})
      for (int64_t proj : {(int64_t)1, (int64_t)500, (int64_t)300000, ((int64_t)1 << 31) - 1}) {
        if (draws < 2) continue;
        const int64_t p = sliced_batch(draws, proj), tiles = (draws + 4095) / 4096 + 1;
        if (p < 1 || p > proj || (p > 1 && p * draws > (int64_t)1 << 23) || (p + 3) / 4 > kMaxGridYZ ||
            p * tiles * 256 >= (int64_t)1 << 32) {
          std::printf("draws %ld projections %ld -> %ld\n", (long)draws, (long)proj, (long)p);
          return 1;
        }
        ++n;
      }
  std::printf("ok %ld checks\n", n);
  return 0;
}
