// Host-side check of how a fused scan's workgroups are shared out to the slice
// groups that are left to it (no GPU, no HIP): compiled with g++ by
// tests/test_host_split.py.
#include <stdio.h>

#include <random>
#include <vector>

#include "build_plan.hpp"

using namespace compass;

int main() {
  std::mt19937 rng(1);
  auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  const int64_t tile = 8192;
  long fails = 0;
  for (int rep = 0; rep < 4000; ++rep) {
    const int ng = pick(1, 16), size = pick(1, 3);
    int32_t begin[17] = {0};
    for (int g = 0; g < ng; ++g)
      begin[g + 1] = begin[g] + (rep % 2 ? size : pick(1, 3));
    const uint32_t live = rep % 3 ? rng() & ((1u << ng) - 1) : (1u << ng) - 1;
    const int64_t cus = pick(48, 400), max_chunks = pick(1, 600), blocks = 2 * cus;
    const int64_t n_rows = rep % 5 ? pick(1, 30000000) : pick(1, 3 * 8192);
    std::vector<std::vector<int>> seen(ng);
    std::vector<int64_t> per(ng, 0);
    long idle = 0;
    const int64_t grid = (blocks + 7) / 8 * 8;
    int per_die[8] = {0};
    for (int64_t block = 0; block < grid; ++block) {
      const LiveSplit s = live_split(begin, ng, live, (uint32_t)block, 8, (uint32_t)cus,
                                     (uint32_t)((n_rows + tile - 1) / tile), max_chunks);
      if (s.group < 0) {
        ++idle;
        continue;
      }
      if (!((live >> s.group) & 1u) || s.chunk < 0 || s.chunk >= s.chunks ||
          s.chunks > max_chunks || s.chunk * s.chunk_tiles * tile >= n_rows ||
          s.chunks * s.chunk_tiles * tile < n_rows ||
          (per[s.group] && per[s.group] != s.chunk_tiles)) {
        ++fails;
        break;
      }
      ++per_die[block % 8];
      per[s.group] = s.chunk_tiles;
      seen[s.group].resize(s.chunks, 0);
      ++seen[s.group][s.chunk];
    }
    // every chunk of every live group by exactly one workgroup
    for (int g = 0; g < ng; ++g) {
      if (((live >> g) & 1u) != !seen[g].empty()) ++fails;
      for (int c : seen[g]) fails += c != 1;
    }
    // the dies have equal shares, the last ones less
    for (int k = 0; k < 8; ++k) fails += per_die[k] > per_die[0];
    if (per_die[0] > 8) fails += per_die[6] < per_die[0] - 8;
    // one live group of a large table has a workgroup on most units
    if (__builtin_popcount(live) == 1 && n_rows > 4 * cus * tile &&
        grid - idle < std::min(cus, max_chunks) * 3 / 4)
      ++fails;
  }
  for (int run = 1; run <= 512; ++run)
    for (int per_max : {1, 4, 48})
      for (int64_t t : {1, 30, 122, 256, 5000}) {
        const int g = live_groups(run, per_max, t, 256);
        fails += g < 1 || g > run || (run + g - 1) / g > per_max;
        // a workgroup per unit, as far as there are tiles and slices
        fails += g * t < std::min<int64_t>(256, run * t);
      }
  printf(fails ? "%ld failures\n" : "ok\n", fails);
  return fails != 0;
}
