// Host-side checks of the counted build's choice and tiling (no GPU, no HIP):
// compiled with g++ by tests/test_host_count.py.
#include <stdio.h>

#include "build_plan.hpp"

using namespace compass;

static int fails = 0;
#define CHECK(c)                                                   \
  do {                                                             \
    if (!(c)) {                                                    \
      printf("FAIL %s:%d %s\n", __FILE__, __LINE__, #c);           \
      ++fails;                                                     \
    }                                                              \
  } while (0)

int main() {
  const int64_t top = (int64_t)1 << 31;
  for (int64_t n : {(int64_t)1, (int64_t)16383, (int64_t)16385, (int64_t)1000003,
                    (int64_t)4500000, (int64_t)36000000, (int64_t)1000000000,
                    top - kCntTile - 1, top - kCntTile, top, ((int64_t)1 << 46)}) {
    for (int slices : {1, 3, 4, 5, 7, 11, 14, 32, 512}) {
      const int bins = counted_bins(n, slices);
      CHECK(bins >= 0 && bins <= kCntMaxBins);
      // int32 multiplicities, and small tables and few sketch rows never
      if (n >= top - kCntTile || (double)n * slices < kCntMinUpdates || slices < 4)
        CHECK(bins == 0);
      // at most one distinct key per value of the range: the hashing saved
      // covers the counting
      if (bins > 0)
        CHECK((double)bins * kCntBinKeys * slices + kCntRowCost * n < 0.95 * n * slices);
    }
    if (n > top) continue;
    for (int cols : {1, 2, 16})
      for (int slots : {2, 512}) {
        const CountTiles t = count_tiles(n, cols, slots);
        CHECK((int64_t)t.n_tiles * kCntTile >= n);
        CHECK((int64_t)(t.n_tiles - 1) * kCntTile < n);
        CHECK((int64_t)t.n_wg * t.tiles_per_wg >= t.n_tiles);
        CHECK((t.n_wg - 1) * t.tiles_per_wg < t.n_tiles);   // no empty one
        CHECK(t.n_sg >= 1 && t.n_sg <= kCntMaxSg);
        CHECK(t.n_sg * t.wg_per_sg >= t.n_wg);
        CHECK((t.n_sg - 1) * t.wg_per_sg < t.n_wg);
      }
  }
  if (!fails) printf("ok\n");
  return fails != 0;
}
