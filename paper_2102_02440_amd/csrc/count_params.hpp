// count_params.hpp -- kernel arguments of the counted build: the fused scan
// of a table without predicates whose key columns hold few distinct keys.
#pragma once
#include <stdint.h>

#include "build_params.hpp"
#include "build_plan.hpp"
#include "device_math.hpp"

namespace compass {

constexpr int kCntThreads = 1024;
constexpr int kCntKeys = kCntTile / kCntThreads;  // keys per lane and tile
static_assert(kCntKeys * kCntThreads == kCntTile, "whole keys per lane");
static_assert(kCntMaxBins == kCntThreads, "one lane per bin");

// One counting item: the records of `bin` in super-groups [g0, g1).
struct CountItem {
  int32_t bin, g0, g1;
  uint32_t records;
};

struct CountCol {
  const void *col;
  int32_t dtype;
  uint32_t range;       // keys counted are below it (nbins << kCntBinBits)
  int32_t nbins;
  int32_t rec_stride;   // records per tile, padding included
  uint16_t *recs;       // [tile][rec_stride] offsets in the bin, by bin
  uint16_t *tab;        // [tile][nbins + 1] first record of a bin / 4
  uint32_t *sgtot;      // [super-group][nbins] records
  CountItem *items;
  uint2 *bin_item;      // [nbins] first item of a bin, its items
  int32_t *part;        // [item][kCntBinKeys] counts
  uint32_t *keys;       // distinct keys, in no particular order
  int32_t *wts;         // and their multiplicities
  uint64_t *exc;        // field elements of the keys outside the range
};

struct CountArgs {
  int64_t n_rows;
  int64_t *n_selected;
  CountState *st;       // per counted column
  int32_t n_cols;
  int32_t n_tiles;
  int32_t n_sg;         // super-groups of wg_per_sg x tiles_per_wg tiles
  int32_t wg_per_sg;
  int32_t tiles_per_wg;
  int32_t item_records; // records an item takes before the next one starts
  uint32_t max_exc;     // entries of each column's `exc`
  uint32_t pad;
  CountCol c[kMaxSketches];
};
static_assert(sizeof(CountArgs) <= 4096, "kernel arguments must stay small");

// Weighted scan: launch-local slice groups, each of one column's slices.
struct WeightedArgs {
  const CountState *st;
  int32_t *slice_chunks;   // [slice] slab rows written
  int32_t *slab;
  int32_t n_groups;
  int32_t n_slices_total;
  int32_t slots;           // resident workgroups
  int32_t max_chunks;      // slab rows there are
  BucketMod bm;
  const uint32_t *keys[kMaxSketches];
  const int32_t *wts[kMaxSketches];
  const uint64_t *exc[kMaxSketches];
  int16_t group_begin[kMaxLaunchGroups + 1];
  int16_t gs[kMaxLaunchSlices];   // the call's slice (sketch * d + row)
  int8_t group_col[kMaxLaunchGroups];
  RowSeeds seeds[kMaxLaunchSlices];
};
static_assert(sizeof(WeightedArgs) <= 4096, "kernel arguments must stay small");

}  // namespace compass
