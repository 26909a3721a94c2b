// agms_params.hpp -- kernel arguments of the AGMS baseline (Section 4.1).
#pragma once
#include <stdint.h>

#include "build_params.hpp"

namespace compass {

constexpr int kAgmsMaxJoins = 4;
constexpr int kAgmsMaxCounters = 1024;  // r * b: at most one lane each

// Sign tables (large tables without predicates, agms_signs_kernel): for every
// distinct key column the K signs of each key of [0, range), 128 basic
// sketches to a 16-byte word group.
constexpr int kAgmsGroup = 128;                       // sketches per uint4
constexpr uint32_t kAgmsMaxRange = 1u << 24;
struct AgmsState {
  uint32_t bad;                  // hash every row instead
  uint32_t range[kAgmsMaxJoins]; // per column: keys below it have signs
  uint32_t pad[3];
};

struct AgmsTables {
  AgmsState *st;               // nullptr: no sign tables
  int32_t n_cols, n_groups;    // distinct columns; ceil(K / kAgmsGroup)
  KeyDev col[kAgmsMaxJoins];
  uint32_t cap[kAgmsMaxJoins];       // keys a column's table can hold
  uint4 *signs[kAgmsMaxJoins];       // [group][cap]
  int32_t col_joins[kAgmsMaxJoins];  // joins on the column ...
  int32_t join[kAgmsMaxJoins][kAgmsMaxJoins];  // ... and which
  int64_t most_lanes;          // keys x joins x lanes the signs may cost
};

struct AgmsParams {
  int64_t n_rows;
  int32_t tile;                // rows per tile, at most kBuildTile
  int64_t rows_per_chunk;
  int32_t n_preds;
  int32_t n_joins;
  int32_t K;                   // r * b basic sketches
  int32_t count_selected;
  int64_t *n_selected;
  int64_t *counters;           // K int64
  const RowSeeds *seeds;       // device, n_joins x K (b0, b1 unused)
  PredDev preds[kMaxPreds];
  KeyDev keys[kAgmsMaxJoins];
  AgmsTables tab;
};

struct AgmsEstArgs {
  const int64_t *sk[16];       // per table: r x b counters
  const int64_t *n_sel[16];    // per table: selected rows (device)
  int32_t n_tables, r, b, pad;
};

}  // namespace compass
