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
// all.  The range bounds the distinct keys of a column that fits it (at most
// one per value): hashing every row costs n_rows * slices updates, the
// counted build at most range * slices of them plus the partition and
// counting passes, which cost about as much as kCntRowCost updates per row:
// 3.3 ns per 1000 rows of a column against 1.6 ns per 1000 updates is 2.1,
// taken with a margin for clustered keys and narrow tables.
// The host does not know which columns fit.  One that does not (a primary
// key, keys that hardly repeat) is found out by a sample on the device and
// hashed row by row, but pays for five launches without work, some 17 us:
// 3 % at 5e8 updates, 6 to 12 at 2e8, up to 22 at 8e7 (140 -> 170 us); one
// that the sample lets pass and that overflows the list of outside keys pays
// the partition as well (4.3M rows, 190 -> 290 us).  Columns that fit gain
// from about 5e7 updates on (7 sketch rows, keys repeated 20 times: 113 ->
// 85 us at 5e7, 320 -> 158 at 2e8; 4 times: 113 -> 105 and 318 -> 229), with
// few sketch rows later (5 rows, 20 times: 104 -> 101 us at 5e7, 152 -> 107
// at 8e7): the updates saved have to pay too.  Where another column of the
// table pays for the launches, kCntAlsoUpdates is enough (2e7 beside the
// first column's 3 sketches: 133 -> 101 us repeated 10 times, 133 -> 130 if it
// does not fit; the least gain is at 1.5e7, 133 -> 98 and 133 -> 136).
constexpr double kCntRowCost = 3.5;
constexpr double kCntMinUpdates = 5.0e7;   // below: launches would not pay
constexpr double kCntMinSaved = 2.0e7;     // updates beyond the rows' own cost
constexpr double kCntAlsoUpdates = 1.5e7;
inline int counted_bins(int64_t n_rows, int slices, bool also = false) {
  if (n_rows >= ((int64_t)1 << 31) - kCntTile) return 0;  // int32 weights
  if ((double)n_rows * slices < (also ? kCntAlsoUpdates : kCntMinUpdates)) return 0;
  if (!also && (double)n_rows * (slices - kCntRowCost) < kCntMinSaved) return 0;
  const double share = 0.9 - kCntRowCost / slices;
  if (share <= 0) return 0;
  const double bins = (double)n_rows * share / kCntBinKeys;
  return (int)std::min<double>(bins, kCntMaxBins);
}

// Slice groups of a run of one column's slices in a counted build's scan: as
// few as the LDS allows (per_max slices each), but enough of them for a
// workgroup per compute unit where the column alone is left to the scan.
constexpr int live_groups(int run, int per_max, int64_t tiles, int cus) {
  const int64_t fill = (cus + tiles - 1) / tiles;
  const int least = (run + per_max - 1) / per_max;
  return least > fill ? least : (int)(fill < run ? fill : run);
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

// Workgroups are dealt to the dies round-robin; pieces of work are numbered die
// by die, so that neighbours run on one die and share its L2.  The piece of
// workgroup `block`, -1: none (the last die's share is not full).
constexpr int32_t piece_by_die(uint32_t block, uint32_t pieces, uint32_t dies) {
  const uint32_t per_die = (pieces + dies - 1) / dies, at = block / dies;
  const uint32_t piece = block % dies * per_die + at;
  return at < per_die && piece < pieces ? (int32_t)piece : -1;
}

// The workgroups of a counted build's scan, which takes the slice groups whose
// columns are not counted ("live", known on the device only): one per compute
// unit, or two where that leaves each eight tiles, shared out to the live
// groups in proportion to their slices, each group's rows cut into that many
// chunks of whole tiles, at most max_chunks.  Groups of one size keep the
// plain scan's numbering (the groups of a chunk in a row, to read its keys
// through one L2).  (constexpr: callable on the host and on the device.)
struct LiveSplit {
  int32_t group, chunk, chunks;   // group -1: the workgroup has no work
  uint32_t chunk_tiles;
};
struct LiveChunks {
  uint32_t chunks, tiles;   // chunks of a group, tiles of a chunk
};
constexpr LiveChunks live_chunks(uint32_t blocks, uint32_t share, uint32_t of, uint32_t tiles,
                                 uint32_t max_chunks) {
  uint32_t c = blocks * share / of;
  c = c < max_chunks ? c : max_chunks;
  c = c < tiles ? c : tiles;
  c = c > 1 ? c : 1;
  const uint32_t per = (tiles + c - 1) / c;
  return LiveChunks{(tiles + per - 1) / per, per};
}
constexpr LiveSplit live_split(const int32_t *group_begin, int n_groups, uint32_t live,
                               uint32_t block, uint32_t dies, uint32_t cus, uint32_t tiles,
                               uint32_t max_chunks) {
  const LiveSplit none{-1, 0, 0, 0};
  uint32_t slices = 0, size = 0, n_live = 0;
  bool equal = true;
  for (int g = 0; g < n_groups; ++g) {
    if (!((live >> g) & 1u)) continue;
    const uint32_t ns = (uint32_t)(group_begin[g + 1] - group_begin[g]);
    equal = equal && (n_live == 0 || ns == size);
    size = ns;
    slices += ns;
    ++n_live;
  }
  if (n_live == 0) return none;
  const uint32_t blocks = tiles * n_live >= 16 * cus ? 2 * cus : cus;
  LiveChunks c = live_chunks(blocks, size, slices, tiles, max_chunks);
  uint32_t used = n_live * c.chunks;
  if (!equal) {
    used = 0;
    for (int g = 0; g < n_groups; ++g)
      if ((live >> g) & 1u)
        used += live_chunks(blocks, (uint32_t)(group_begin[g + 1] - group_begin[g]), slices,
                            tiles, max_chunks).chunks;
  }
  const int32_t piece = piece_by_die(block, used, dies);
  if (piece < 0) return none;
  uint32_t at = equal ? (uint32_t)piece % n_live : (uint32_t)piece;
  for (int g = 0; g < n_groups; ++g) {
    if (!((live >> g) & 1u)) continue;
    if (equal) {
      if (at-- == 0)
        return LiveSplit{g, (int32_t)((uint32_t)piece / n_live), (int32_t)c.chunks, c.tiles};
      continue;
    }
    c = live_chunks(blocks, (uint32_t)(group_begin[g + 1] - group_begin[g]), slices, tiles,
                    max_chunks);
    if (at < c.chunks) return LiveSplit{g, (int32_t)at, (int32_t)c.chunks, c.tiles};
    at -= c.chunks;
  }
  return none;
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
