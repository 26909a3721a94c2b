// build_plan.hpp -- host-side work decomposition of the sketch builds.
//
// Plain integer arithmetic with no HIP dependency, so the host tests can
// compile and check it on a machine without a GPU.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace compass {

// Rows of one chunk of the fused scan.  A workgroup adds at most one +-1
// per row of its chunk to an int32 LDS partial and writes that partial to
// an int32 slab, so a chunk never exceeds INT32_MAX rows (rounded down to
// whole tiles); the chunk count grows instead.  Returns rows per chunk
// (a multiple of `tile`, >= tile) for the wanted number of chunks.
inline int64_t fused_rows_per_chunk(int64_t n_rows, int64_t chunks, int64_t tile) {
  if (chunks < 1) chunks = 1;
  int64_t r = (n_rows + chunks - 1) / chunks;
  r = (r + tile - 1) / tile * tile;
  const int64_t most = (int64_t)INT32_MAX / tile * tile;
  if (r > most) r = most;
  if (r < tile) r = tile;
  return r;
}

// Whether a kernel's LDS (static + dynamic) fits what one workgroup may
// allocate on the device.
inline bool lds_fits(size_t dynamic_bytes, size_t static_bytes, size_t limit) {
  return dynamic_bytes + static_bytes <= limit;
}

// Plan of the two-phase build (survivor compaction, then hashing of the
// buffered survivors into LDS counters, then a slab reduction).
//
// Rows are compacted in batches of `batch` rows; the buffer holds `cap`
// survivors per sketch.  After a batch the buffer is flushed (hashed and
// reduced into the counters, then emptied) only if the next batch might not
// fit, so selective scans hash once per build.  cap >= 2 * batch unless one
// batch covers the whole table.
struct TwoPhasePlan {
  int64_t cap = 0;        // survivors per sketch the buffer holds
  int64_t batch = 0;      // rows per compaction launch
  int32_t chunks = 1;     // survivor chunks per slice in one flush
  int32_t ranges = 1;     // bucket ranges of at most 65536 per slice
  size_t seeds_bytes = 0, ctl_bytes = 0, surv_bytes = 0, slab_bytes = 0;
  size_t total_bytes = 0; // seeds | count, ticket | survivors | slab
  bool ok = false;
};

inline size_t plan_align(size_t x) { return (x + 255) & ~(size_t)255; }

// n_cu: compute units (one hashing workgroup per CU: 128 KiB of LDS);
// budget: bytes of scratch the plan may use; cap_rows_max: an upper bound
// on the buffer's survivors (0 = none).  The survivor chunk count is picked
// so that the workgroups of a flush fill whole waves of the CUs as far as
// the slab (chunks x slices x w int32) stays within a quarter of the budget.
inline TwoPhasePlan plan_two_phase(int64_t n_rows, int n_sketches, int d,
                                   int w, int n_cu, size_t budget,
                                   int64_t cap_rows_max, int64_t tile,
                                   int seed_bytes_per_slice) {
  TwoPhasePlan p;
  const int S = n_sketches * d;
  p.ranges = (w + 65535) / 65536;
  const size_t slab_row = (size_t)S * w * 4;
  p.seeds_bytes = plan_align((size_t)S * seed_bytes_per_slice);
  p.ctl_bytes = 256;
  const int items1 = S * p.ranges;
  int best_c = 1;
  double best_eff = 0.0;
  const int c_max = std::max(1, 4 * n_cu / std::max(1, items1));
  for (int c = 1; c <= c_max; ++c) {
    if ((size_t)c * slab_row > budget / 4 && c > 1) break;
    const int64_t items = (int64_t)items1 * c;
    const int64_t waves = (items + n_cu - 1) / n_cu;
    const double eff = (double)items / (double)(waves * n_cu);
    // more chunks only for a clearly better fill (each costs a slab row)
    if (eff > best_eff + 0.02) {
      best_eff = eff;
      best_c = c;
    }
  }
  p.chunks = best_c;
  p.slab_bytes = plan_align((size_t)p.chunks * slab_row);
  const size_t fixed = p.seeds_bytes + p.ctl_bytes + p.slab_bytes;
  if (fixed >= budget) return p;
  const int64_t worst = (n_rows + tile - 1) / tile * tile;
  int64_t cap = (int64_t)((budget - fixed) / (8 * (size_t)n_sketches)) / tile * tile;
  if (cap_rows_max > 0) cap = std::min(cap, std::max(tile, cap_rows_max / tile * tile));
  if (cap >= worst) {
    p.cap = std::max<int64_t>(worst, tile);
    p.batch = p.cap;
  } else {
    p.cap = cap;
    p.batch = cap / 2 / tile * tile;
    if (p.batch < tile) return p;  // too small for one tile per batch
  }
  p.surv_bytes = plan_align((size_t)p.cap * 8 * n_sketches);
  p.total_bytes = fixed + p.surv_bytes;
  p.ok = p.total_bytes <= budget;
  return p;
}

// Chunks the n survivors of a flush are hashed in: at least kWideMinChunk
// survivors each (a chunk's fixed cost is clearing, folding and writing w
// counters), at most `chunks`.  Where that is more than one round of the CUs,
// of the counts that fill one to four rounds the one with the least time --
// rounds of items (0.31 ns per survivor, 0.2 ns per counter, 2 us), then the
// reduction (0.4 ns per KB of slab).  1.5M survivors of 66 slices of 65,536
// counters: the 15 chunks of the best fill took 180 us and 101 to reduce, the
// fewer picked here take 143 and 67.
// Every workgroup of the hashing evaluates this and all have to agree, so the
// times are whole picoseconds (floating point may be contracted differently
// from one compilation to the next); the reduction reads what the hashing
// stored.
constexpr int64_t kWideMinChunk = 16384;
constexpr int kWideRange = 65536;   // counters of one hashing item at most
constexpr int hash_chunks(int64_t n, int64_t chunks, int n_slices, int w, int n_cu) {
  const int64_t need = (n + kWideMinChunk - 1) / kWideMinChunk;
  const int most = (int)(need < 1 ? 1 : (need < chunks ? need : chunks));
  const int items = n_slices * ((w + kWideRange - 1) / kWideRange);
  if (most * items <= n_cu) return most;
  const uint32_t n32 = n < 0xFFFFFFFFll ? (uint32_t)n : 0xFFFFFFFFu;
  const int64_t fixed = 200ll * (w < kWideRange ? w : kWideRange) + 2000000;
  int best = 1;
  int64_t least = INT64_MAX;
  for (int k = 1; k <= 4; ++k) {
    const int fill = k * n_cu / items;
    const int c = fill < 1 ? 1 : (fill < most ? fill : most);
    const int rounds = (c * items + n_cu - 1) / n_cu;
    const int64_t cost = rounds * (310ll * (n32 / (uint32_t)c) + fixed) +
                         (int64_t)c * n_slices * w * 3 / 2;
    if (cost < least) {
      least = cost;
      best = c;
    }
  }
  return best;
}

// Counted build (tables without predicates): a key column's rows are
// partitioned by key range, its distinct keys counted, and only those
// hashed, each with its multiplicity as the weight.
constexpr int kCntBinBits = 14;                     // keys per bin: 64 KiB of int32
constexpr int kCntBinKeys = 1 << kCntBinBits;
constexpr int kCntMaxBins = 1024;
constexpr int kCntTile = 16384;                     // rows per partition tile
constexpr int kCntMaxSg = 64;

// The key range [0, range) within which a column of n_rows keys hashed into
// `slices` sketch rows is counted, in bins of kCntBinKeys; 0 bins: not at
// all.  The range bounds the distinct keys (at most one per value), so it
// is what the choice guarantees: hashing every row costs n_rows * slices
// updates, the counted build at most range * slices of them plus the
// partition and counting passes, which cost about as much as kCntRowCost
// updates per row: 3.3 ns per 1000 rows of a column against 1.6 ns per 1000
// updates is 2.1, taken with a margin for clustered keys and narrow tables.
// Below kCntMinUpdates the seven launches eat the gain: 63M updates of 4.5M
// rows take 108 us counted and 146 us hashed row by row.  Where another
// column of the table pays for them, kCntAlsoUpdates is enough
// (7 sketch rows of 4.5M keys beside 14 of another column: 145 us hashed row
// by row, 35 counted).
constexpr double kCntRowCost = 3.5;
constexpr double kCntMinUpdates = 5.0e7;   // below: launches would not pay
constexpr double kCntAlsoUpdates = 1.5e7;
inline int counted_bins(int64_t n_rows, int slices, bool also = false) {
  if (n_rows >= ((int64_t)1 << 31) - kCntTile) return 0;  // int32 weights
  if ((double)n_rows * slices < (also ? kCntAlsoUpdates : kCntMinUpdates)) return 0;
  const double share = 0.9 - kCntRowCost / slices;
  if (share <= 0) return 0;
  const double bins = (double)n_rows * share / kCntBinKeys;
  return (int)std::min<double>(bins, kCntMaxBins);
}

// A workgroup's decision on a word that other workgroups of the same launch
// may be writing: one lane reads it and every lane acts on what that lane
// saw.  Waves that read for themselves may see different values, and one that
// leaves no longer takes part in the barriers of those that stay.  (constexpr:
// callable on the host and on the device.)
template <class Load, class Barrier>
constexpr bool block_reads(uint32_t *shared, bool reader, Load load, Barrier barrier) {
  if (reader) *shared = load();
  barrier();
  return *shared != 0;
}

// Tiles of a partitioned column: workgroups of tiles_per_wg tiles each,
// wg_per_sg workgroups per super-group, at most kCntMaxSg super-groups.
struct CountTiles {
  int32_t n_tiles, tiles_per_wg, n_wg, wg_per_sg, n_sg;
};
inline CountTiles count_tiles(int64_t n_rows, int n_cols, int slots) {
  CountTiles t;
  t.n_tiles = (int32_t)((n_rows + kCntTile - 1) / kCntTile);
  const int want = std::max(1, slots / std::max(1, n_cols));
  t.tiles_per_wg = std::max(1, (t.n_tiles + want - 1) / want);
  t.n_wg = (t.n_tiles + t.tiles_per_wg - 1) / t.tiles_per_wg;
  t.wg_per_sg = (t.n_wg + kCntMaxSg - 1) / kCntMaxSg;
  t.n_sg = (t.n_wg + t.wg_per_sg - 1) / t.wg_per_sg;
  return t;
}

}  // namespace compass
