// count_kernels.hip -- the counted build of a table without predicates.
//
// A sketch row adds xi(key) to counter h(key) once per row of the table, so
// a key that occurs c times adds c * xi(key): hashing each distinct key
// once, with its multiplicity as the weight, gives the same integers
// (Section 4.2 counter definition; integer addition).  Foreign keys repeat
// (a fact table of 36M rows references 2.5M movies), and the fused scan is
// bound by the hash (41 VALU instructions per row and sketch row), so
// counting first removes most of the work:
//   1. count_partition_kernel: tiles of 16384 keys are sorted by bin (16384
//      consecutive keys) in LDS and written back as 16-bit offsets, with a
//      table of each bin's first record;
//   2. count_plan_kernel: (bin, run of tiles) items of about equal records;
//   3. count_items_kernel: an item's records counted in LDS (64 KiB);
//   4. count_emit_kernel: a bin's items summed, its non-zero counts appended
//      to the column's list of (key, multiplicity);
//   5. weighted_scan_kernel: the list hashed into LDS partials and written
//      to the slab of the fused scan, which slab_reduce_kernel sums.
// Keys outside the range the host chose are listed one by one and hashed
// with weight 1.  A column with too many of them (a sample says so before
// anything else, or the list overflows) is marked `bad`: every kernel here
// then leaves it and scan_sketch_kernel hashes its rows, as it does for
// tables this path is not chosen for.
//
// Measured, 36M rows, two 32-bit columns (2.5M and 4.2M Zipf keys), 21 sketch
// rows of 8192 buckets: every row hashed 1205 us; counted 336 us = partition
// 112 + plan 9 + items 91 + emit 29 + weighted scan 76 (6.0M distinct keys)
// + the empty scan 5 + reduction 8.  Uniform keys (4 per value, 14 sketch
// rows) 887 -> 477 us.  A table whose columns turn out bad pays the five
// empty launches, 17 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "count_params.hpp"

namespace compass {

__device__ __forceinline__ uint32_t column_bad(const CountState *st) {
  return __hip_atomic_load(&st->bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Exclusive sums of v over the block's 1024 lanes; *total = the block's sum.
// `s_wave` holds 16 words; one barrier before it is read.
__device__ __forceinline__ uint32_t block_exclusive_sum(uint32_t v, uint32_t *s_wave,
                                                       uint32_t *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = __shfl_up(inc, o);
    if (lane >= o) inc += u;
  }
  if (lane == 63) s_wave[wave] = inc;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll 4
  for (int k = 0; k < kCntThreads / 64; ++k) {
    const uint32_t u = s_wave[k];
    before += k < wave ? u : 0u;
    all += u;
  }
  *total = all;
  return before + inc - v;
}

constexpr uint32_t kNoKey = 0xFFFFFFFFu;   // a key of more than 32 bits
constexpr uint16_t kNoRec = kCntBinKeys;   // padding: counted past the bin

// The tile's raw keys of one lane (rows tid + k * 1024), streamed.  A whole
// tile by buffer loads: one lane offset for every row, the row step in the
// scalar offset.  The last tile's by plain loads at clamped rows: the range
// check of a buffer load compares with the buffer's size less the scalar
// offset, which a short buffer does not hold.
typedef int int2v __attribute__((ext_vector_type(2)));
template <class T>
struct RawKeys;
template <>
struct RawKeys<int32_t> {
  int v[kCntKeys];
  __device__ __forceinline__ void load(const CountCol &c, int64_t base, int nt) {
    const int32_t *col = reinterpret_cast<const int32_t *>(c.col) + base;
    if (nt == kCntTile) {
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(col), 0,
                                                          kCntTile * 4, 0x00027000);
#pragma unroll
      for (int k = 0; k < kCntKeys; ++k)
        v[k] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)threadIdx.x * 4,
                                                    k * kCntThreads * 4, 2);
    } else {
#pragma unroll
      for (int k = 0; k < kCntKeys; ++k) {
        v[k] = col[min((int)threadIdx.x + k * kCntThreads, nt - 1)];
        if (k % 4 == 3) __asm__ volatile("" ::: "memory");  // few addresses at once
      }
    }
  }
  __device__ __forceinline__ uint32_t key(int k) const { return (uint32_t)v[k]; }
};
template <>
struct RawKeys<int64_t> {
  int2v v[kCntKeys];
  __device__ __forceinline__ void load(const CountCol &c, int64_t base, int nt) {
    const int64_t *col = reinterpret_cast<const int64_t *>(c.col) + base;
    if (nt == kCntTile) {
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<int64_t *>(col), 0,
                                                          kCntTile * 8, 0x00027000);
#pragma unroll
      for (int k = 0; k < kCntKeys; ++k)
        v[k] = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)threadIdx.x * 8,
                                                    k * kCntThreads * 8, 2);
    } else {
#pragma unroll
      for (int k = 0; k < kCntKeys; ++k) {
        v[k] = *reinterpret_cast<const int2v *>(
            col + min((int)threadIdx.x + k * kCntThreads, nt - 1));
        if (k % 4 == 3) __asm__ volatile("" ::: "memory");
      }
    }
  }
  __device__ __forceinline__ uint32_t key(int k) const {
    return v[k].y ? kNoKey : (uint32_t)v[k].x;
  }
};

// Appends the tile's keys outside the range to the column's list (a rare
// path: the rows are read again, one by one); a full list marks the column
// bad.
template <class T>
__device__ __forceinline__ void list_exceptions(const CountCol &c, CountState *st,
                                                uint32_t max_exc, int64_t base, int nt) {
#pragma unroll 1
  for (int r = threadIdx.x; r < nt; r += kCntThreads) {
    const int64_t v = reinterpret_cast<const T *>(c.col)[base + r];
    if ((uint64_t)v < c.range) continue;
    const uint32_t at = atomicAdd(&st->n_exc, 1u);
    if (at < max_exc)
      c.exc[at] = key_field(v);
    else
      __hip_atomic_store(&st->bad, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Adds every key to its bin's count; rank[k] = the keys counted there before.
// One LDS word takes one add at a time, and in a clustered column the 64
// lanes meet in one bin: with kMatch the lanes of the first lane's bin add
// once between them.  All lanes active.
template <bool kMatch>
__device__ __forceinline__ void rank_keys(uint32_t *s_bin, const uint32_t (&key)[kCntKeys],
                                          uint32_t (&rank)[kCntKeys]) {
#pragma unroll
  for (int k = 0; k < kCntKeys; ++k) {
    const uint32_t b = key[k] >> kCntBinBits;
    if (!kMatch) {
      rank[k] = atomicAdd(&s_bin[b], 1u);
      continue;
    }
    const uint32_t first = __builtin_amdgcn_readfirstlane(b);
    const uint64_t same = __ballot(b == first);
    const uint32_t before = __builtin_amdgcn_mbcnt_hi(
        (uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
    const bool mine = b == first;
    uint32_t at = 0;
    if (!mine || before == 0)
      at = atomicAdd(&s_bin[b], mine ? (uint32_t)__popcll(same) : 1u);
    const uint32_t at0 = __builtin_amdgcn_readfirstlane(at);
    rank[k] = mine ? at0 + before : at;
  }
}

// What a counted build clears, and the first look at its columns: workgroup
// (0, c) of the last grid row reads 1024 keys spread over column c and marks
// it bad if more than 16 of them lie outside its range.
__global__ __launch_bounds__(256) void count_start_kernel(const ZeroSpans z,
                                                          const CountArgs A) {
  if ((int)blockIdx.y == z.n) {
    if ((int)blockIdx.x >= A.n_cols) return;
    __shared__ uint32_t s_out[4];
    const CountCol &c = A.c[blockIdx.x];
    uint32_t out = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t r = A.n_rows * (int64_t)(threadIdx.x + k * 256) / 1024;
      const uint64_t v = c.dtype == kDtI32
                             ? (uint64_t)reinterpret_cast<const uint32_t *>(c.col)[r]
                             : reinterpret_cast<const uint64_t *>(c.col)[r];
      out += (uint32_t)__popcll(__ballot(v >= c.range));
    }
    if ((threadIdx.x & 63) == 0) s_out[threadIdx.x >> 6] = out;
    __syncthreads();
    if (threadIdx.x == 0)
      A.st[blockIdx.x] = CountState{
          s_out[0] + s_out[1] + s_out[2] + s_out[3] > 16 ? 1u : 0u, 0u, 0u, 0u};
    return;
  }
  uint32_t *p = reinterpret_cast<uint32_t *>(z.p[blockIdx.y]);
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
       i < z.words[blockIdx.y]; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

// Lanes of a wave that share the first lane's bin (or record) from which on
// its adds are matched: sorted keys, matched never, take 237 us instead of
// 46 us (two columns of 10M).
constexpr int kMatchLanes = 10;

template <class T>
__device__ __forceinline__ void partition_tiles(const CountArgs &A, uint16_t *s_rec,
                                                uint32_t *s_bin, uint32_t *s_wave,
                                                uint32_t *s_stop) {
  const CountCol &c = A.c[blockIdx.y];
  CountState *st = A.st + blockIdx.y;
  const int tid = threadIdx.x;
  const int t0 = blockIdx.x * A.tiles_per_wg;
  const int t1 = min(A.n_tiles, t0 + A.tiles_per_wg);
  const uint32_t nb = (uint32_t)c.nbins, range = c.range;
  uint32_t mine = 0;   // records of bin `tid` over the workgroup's tiles
  auto rows = [&](int t) {
    return (int)min((int64_t)kCntTile, A.n_rows - (int64_t)t * kCntTile);
  };
  for (int t = t0; t < t1; ++t) {
    const int nt = rows(t);
    RawKeys<T> raw;
    raw.load(c, (int64_t)t * kCntTile, nt);
    s_bin[tid] = 0;
    if (tid == 0) {
      s_bin[nb] = 0;
      *s_stop = column_bad(st);
    }
    // rows past the end and keys outside the range: the bin past the last
    uint32_t key[kCntKeys], most = 0;
#pragma unroll
    for (int k = 0; k < kCntKeys; ++k) {
      key[k] = raw.key(k);
      most = max(most, key[k]);
      key[k] = min(key[k], range);
    }
    if (__any(most >= range))
      list_exceptions<T>(c, st, A.max_exc, (int64_t)t * kCntTile, nt);
    if (nt < kCntTile) {
#pragma unroll
      for (int k = 0; k < kCntKeys; ++k)
        if (tid + k * kCntThreads >= nt) key[k] = range;
    }
    __syncthreads();
    uint32_t rank[kCntKeys];
    const uint32_t b0 = key[0] >> kCntBinBits;
    if (__popcll(__ballot(b0 == (uint32_t)__builtin_amdgcn_readfirstlane(b0))) >= kMatchLanes)
      rank_keys<true>(s_bin, key, rank);
    else
      rank_keys<false>(s_bin, key, rank);
    // (opaque: the bins are formed again below, not kept meanwhile)
#pragma unroll
    for (int k = 0; k < kCntKeys; ++k) __asm__ volatile("" : "+v"(key[k]));
    __syncthreads();
    if (*s_stop) return;   // uniform
    const uint32_t n = (uint32_t)tid < nb ? s_bin[tid] : 0u;
    const uint32_t padded = (n + 3u) & ~3u;
    mine += n;
    uint32_t total;
    const uint32_t first = block_exclusive_sum(padded, s_wave, &total);
    if ((uint32_t)tid < nb) s_bin[tid] = first;
    if (tid == 0) s_bin[nb] = total;
    uint16_t *tab = c.tab + (int64_t)t * (c.nbins + 1);
    if ((uint32_t)tid < nb) tab[tid] = (uint16_t)(first >> 2);
    if (tid == 0) tab[nb] = (uint16_t)(total >> 2);
#pragma unroll
    for (uint32_t q = 1; q < 4; ++q)
      if (padded - n >= q) s_rec[first + padded - q] = kNoRec;
    __syncthreads();
    // keys of no bin land after `total`, inside the stride
#pragma unroll
    for (int k = 0; k < kCntKeys; ++k) rank[k] += s_bin[key[k] >> kCntBinBits];
#pragma unroll
    for (int k = 0; k < kCntKeys; ++k)
      s_rec[rank[k]] = (uint16_t)(key[k] & (kCntBinKeys - 1));
    __syncthreads();
    // 16-byte copies (the tile's stride is a multiple of 8 records; the
    // tail past `total` is never read)
    uint4 *dst = reinterpret_cast<uint4 *>(c.recs + (int64_t)t * c.rec_stride);
    const uint4 *src = reinterpret_cast<const uint4 *>(s_rec);
    for (int q = tid; q < (int)((total + 7) / 8); q += kCntThreads) dst[q] = src[q];
    // (s_rec is written again two barriers on; s_bin was read for the last
    // time before the barrier above)
  }
  if ((uint32_t)tid < nb && mine)
    atomicAdd(&c.sgtot[(int64_t)(blockIdx.x / A.wg_per_sg) * c.nbins + tid], mine);
}

// Two workgroups per CU (64 registers, 42 KiB of LDS): one loads while the
// other sorts.  Bound by its bytes and the LDS adds: two columns of 36M
// 32-bit keys (432 MB moved) in 112 us, 3.9 TB/s; one workgroup per CU of
// 32768-key tiles 128 us.
__global__ __launch_bounds__(kCntThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void count_partition_kernel(
    const CountArgs A) {
  extern __shared__ uint16_t s_rec[];        // rec_stride records
  __shared__ uint32_t s_bin[kCntMaxBins + 1];  // last used: keys of no bin
  __shared__ uint32_t s_wave[kCntThreads / 64];
  __shared__ uint32_t s_bad, s_stop;
  if ((int)blockIdx.x * A.tiles_per_wg >= A.n_tiles) return;   // uniform
  if (block_reads(&s_bad, threadIdx.x == 0,
                  [&] { return column_bad(A.st + blockIdx.y); },
                  [] { __syncthreads(); }))
    return;
  if (A.c[blockIdx.y].dtype == kDtI32)
    partition_tiles<int32_t>(A, s_rec, s_bin, s_wave, &s_stop);
  else
    partition_tiles<int64_t>(A, s_rec, s_bin, s_wave, &s_stop);
}

// One lane per bin: the bin's super-groups cut into items of equal shares,
// about item_records records each.
__global__ __launch_bounds__(64) void count_plan_kernel(const CountArgs A) {
  const CountCol &c = A.c[blockIdx.y];
  CountState *st = A.st + blockIdx.y;
  const int b = blockIdx.x * 64 + threadIdx.x;
  if (blockIdx.y == 0 && b == 0)   // every row of the table qualifies
    atomicAdd(reinterpret_cast<unsigned long long *>(A.n_selected),
              (unsigned long long)A.n_rows);
  if (blockIdx.x * 64 >= c.nbins || st->bad) return;
  uint32_t v[kCntMaxSg];
#pragma unroll
  for (int g = 0; g < kCntMaxSg; ++g)
    v[g] = b < c.nbins && g < A.n_sg ? c.sgtot[(int64_t)g * c.nbins + b] : 0u;
  uint32_t total = 0;
#pragma unroll
  for (int g = 0; g < kCntMaxSg; ++g) total += v[g];
  const uint32_t shares =
      max(1u, (total + (uint32_t)A.item_records / 2) / (uint32_t)A.item_records);
  const uint32_t want = (total + shares - 1) / shares;
  uint32_t acc = 0, n = 0;
#pragma unroll
  for (int g = 0; g < kCntMaxSg; ++g) {
    acc += v[g];
    if (total && acc >= want) {
      ++n;
      acc = 0;
    }
  }
  n += acc ? 1u : 0u;
  uint32_t inc = n;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = __shfl_up(inc, o);
    if ((int)threadIdx.x >= o) inc += u;
  }
  uint32_t at = 0;
  if (threadIdx.x == 63 && inc) at = atomicAdd(&st->n_items, inc);
  at = __shfl(at, 63) + inc - n;
  if (b < c.nbins) c.bin_item[b] = make_uint2(at, n);
  acc = 0;
  int g0 = 0;
#pragma unroll
  for (int g = 0; g < kCntMaxSg; ++g) {
    acc += v[g];
    if (total && acc >= want) {
      c.items[at++] = CountItem{b, g0, g + 1, acc};
      g0 = g + 1;
      acc = 0;
    }
  }
  if (acc) c.items[at] = CountItem{b, g0, A.n_sg, acc};
}

// One workgroup per item, two per CU (64 KiB of counters each).  A group of
// G lanes takes one tile's records of the bin (8 bytes = 4 records per lane),
// two sets of tiles in flight; G follows the item's records per tile, so that
// a spread bin (200 records a tile) keeps every lane busy and a clustered one
// (a whole tile) is read by the whole workgroup.
//
// An LDS word takes one add at a time, so equal records in a wave cost as
// much as that many adds.  A sample of the item's records picks how they are
// added: kSpread one by one; kHeavy counts the two most frequent records of
// the sample by ballots in a scalar register; kRuns (units of four equal
// records: a clustered column) adds once for the lanes that hold the first
// lane's record, and four records at a time where every lane holds four
// equal ones.
constexpr int kItemTiles = 4;
constexpr int kItemBatch = 2048;   // tiles whose segment bounds sit in LDS
enum { kSpread, kHeavy, kRuns };

struct ItemScan {
  const CountCol &c;
  int32_t *cnt;
  const uint32_t *seg;             // first and last unit of the k-th tile
  const uint16_t *at;              // that has any, and that tile - b0
  int G, groups, grp, lane;
  uint32_t hot0, hot1;             // kNoRec: none
  int n_hot0, n_hot1;

  __device__ __forceinline__ const uint2 *tile(int t) const {
    return reinterpret_cast<const uint2 *>(c.recs) + (int64_t)t * (c.rec_stride / 4);
  }

  // Counts the four records of the lanes with `in`; all lanes call it.
  template <int kMode>
  __device__ __forceinline__ void add4(bool in, const uint2 &q) {
    const uint32_t r[4] = {q.x & 0xFFFFu, q.x >> 16, q.y & 0xFFFFu, q.y >> 16};
    if (kMode == kSpread) {
      if (in) {
#pragma unroll
        for (int u = 0; u < 4; ++u) atomicAdd(&cnt[r[u]], 1);
      }
    } else if (kMode == kHeavy) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool h0 = in && r[u] == hot0, h1 = in && r[u] == hot1;
        n_hot0 += __popcll(__ballot(h0));
        n_hot1 += __popcll(__ballot(h1));
        if (in && !h0 && !h1) atomicAdd(&cnt[r[u]], 1);
      }
    } else if (in) {
      const uint32_t first = __builtin_amdgcn_readfirstlane(r[0]);
      const bool four = __all(!in || (q.x == q.y && r[0] == r[1]));
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t f = u ? __builtin_amdgcn_readfirstlane(r[u]) : first;
        const uint64_t same = __ballot(r[u] == f);
        const uint32_t before = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
        const int k = four ? 4 : 1;
        if (r[u] != f || before == 0)
          atomicAdd(&cnt[r[u]], r[u] == f ? k * __popcll(same) : k);
        if (four) break;   // uniform
      }
    }
  }

  // The n tiles of a batch from tile b0 on that hold records of the bin.
  template <int kMode>
  __device__ __forceinline__ void batch(int b0, int n) {
    const bool spare = grp >= groups;   // lanes left over by the division
    uint2 r[kItemTiles], nx[kItemTiles];
    bool in[kItemTiles], in_nx[kItemTiles];
    bool more = false, more_nx;
    auto load = [&](int kb, uint2 (&q)[kItemTiles], bool (&ok)[kItemTiles], bool &longer) {
      longer = false;
#pragma unroll
      for (int u = 0; u < kItemTiles; ++u) {
        const int k = kb + grp + u * groups;
        const uint32_t se = k < n && !spare ? seg[k] : 0u;
        const int j = (int)(se & 0xFFFFu) + lane, e = (int)(se >> 16);
        q[u] = make_uint2(0, 0);
        ok[u] = j < e;
        if (ok[u]) q[u] = tile(b0 + at[k])[j];
        longer = longer || j + G < e;
      }
    };
    load(0, r, in, more);
    for (int kb = 0; kb < n; kb += groups * kItemTiles) {
      load(kb + groups * kItemTiles, nx, in_nx, more_nx);
#pragma unroll
      for (int u = 0; u < kItemTiles; ++u) add4<kMode>(in[u], r[u]);
      if (__any(more)) {   // longer segments
#pragma unroll 1
        for (int u = 0; u < kItemTiles; ++u) {
          const int k = kb + grp + u * groups;
          const uint32_t se = k < n && !spare ? seg[k] : 0u;
          const int e = (int)(se >> 16);
          const uint2 *p = tile(b0 + at[min(k, n - 1)]);
          for (int j0 = (int)(se & 0xFFFFu) + G; __any(j0 < e); j0 += 4 * G) {
            uint2 q[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int j = j0 + G * v + lane;
              q[v] = make_uint2(0, 0);
              if (j < e) q[v] = p[j];
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) add4<kMode>(j0 + G * v + lane < e, q[v]);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kItemTiles; ++u) {
        r[u] = nx[u];
        in[u] = in_nx[u];
      }
      more = more_nx;
    }
  }

  // The adding mode from 64 units spread over the batch (the same in every
  // wave).  Heavy: of the first 16 lanes' first records the two
  // that occur most, if in four lanes or more.
  __device__ __forceinline__ int sample(int b0, int n) {
    const int l = threadIdx.x & 63;
    const uint32_t se = seg[n * l / 64];
    const int a = (int)(se & 0xFFFFu), e = (int)(se >> 16);
    const uint2 q = tile(b0 + at[n * l / 64])[a + (e - a) * (l & 7) / 8];
    const uint32_t r = q.x & 0xFFFFu;
    if (__popcll(__ballot(q.x == q.y && r == q.x >> 16)) >= 16) return kRuns;
    int c0 = 3, c1 = 3;
    for (int i = 0; i < 16; ++i) {
      const uint32_t v = __builtin_amdgcn_readlane(r, i);
      const int k = __popcll(__ballot(r == v));
      if (v == kNoRec || v == hot0 || v == hot1) continue;
      if (k > c0) {
        hot1 = hot0;
        c1 = c0;
        hot0 = v;
        c0 = k;
      } else if (k > c1) {
        hot1 = v;
        c1 = k;
      }
    }
    return c0 > 3 ? kHeavy : kSpread;
  }
};

__global__ __launch_bounds__(kCntThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void count_items_kernel(
    const CountArgs A) {
  __shared__ int32_t s_cnt[kCntBinKeys + 4];   // padding records count at the end
  __shared__ uint32_t s_seg[kItemBatch], s_n, s_units;
  __shared__ uint16_t s_at[kItemBatch];
  const CountCol &c = A.c[blockIdx.y];
  const CountState *st = A.st + blockIdx.y;
  if (st->bad) return;
  // items are handed out XCD by XCD (workgroup b runs on XCD b mod 8):
  // neighbouring bins, whose records and bounds share cache lines, meet in
  // one L2
  const uint32_t per = (st->n_items + kXcds - 1) / kXcds;
  const uint32_t item = (blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
  if (blockIdx.x / kXcds >= per || item >= st->n_items) return;
  const CountItem it = c.items[item];
  int4 *cnt4 = reinterpret_cast<int4 *>(s_cnt);
  for (int j = threadIdx.x; j < kCntBinKeys / 4; j += kCntThreads)
    cnt4[j] = make_int4(0, 0, 0, 0);
  const int per_sg = A.wg_per_sg * A.tiles_per_wg;
  const int t0 = it.g0 * per_sg, t1 = min(A.n_tiles, it.g1 * per_sg);
  ItemScan sc{c, s_cnt, s_seg, s_at, 0, 0, 0, 0, kNoRec, kNoRec, 0, 0};
  int mode = -1;
  for (int b0 = t0; b0 < t1; b0 += kItemBatch) {
    const int b1 = min(t1, b0 + kItemBatch);
    if (threadIdx.x == 0) s_n = s_units = 0;
    __syncthreads();   // counters cleared; the last batch's segments read
    // the batch's tiles that hold records of the bin, in any order
    for (int tw = b0; tw < b1; tw += kCntThreads) {
      const int t = tw + threadIdx.x;
      const uint16_t *tab = c.tab + (int64_t)min(t, b1 - 1) * (c.nbins + 1) + it.bin;
      const uint32_t a = tab[0], e = t < b1 ? tab[1] : 0u;
      const uint64_t some = __ballot(a < e);
      uint32_t units = a < e ? e - a : 0u;
#pragma unroll
      for (int o = 32; o; o >>= 1) units += __shfl_xor(units, o);
      uint32_t at = 0;
      if (__lane_id() == 0 && some) {
        at = atomicAdd(&s_n, (uint32_t)__popcll(some));
        atomicAdd(&s_units, units);
      }
      at = __builtin_amdgcn_readfirstlane(at) +
           __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u));
      if (a < e) {
        s_seg[at] = a | (e << 16);
        s_at[at] = (uint16_t)(t - b0);
      }
    }
    __syncthreads();
    const int n = (int)s_n;
    if (n == 0) continue;
    // lanes for the mean segment and three standard deviations of a spread
    // bin's (m units of 4 records: sqrt(4 m) / 4 each)
    const float m = (float)s_units / (float)n;
    sc.G = min(kCntThreads, (int)(m + 1.5f * sqrtf(m)) + 2);
    sc.groups = kCntThreads / sc.G;
    sc.grp = threadIdx.x / sc.G;
    sc.lane = threadIdx.x - sc.grp * sc.G;
    if (mode < 0) mode = sc.sample(b0, n);
    if (mode == kSpread)
      sc.batch<kSpread>(b0, n);
    else if (mode == kHeavy)
      sc.batch<kHeavy>(b0, n);
    else
      sc.batch<kRuns>(b0, n);
    __syncthreads();
  }
  if ((threadIdx.x & 63) == 0) {
    if (sc.n_hot0) atomicAdd(&s_cnt[sc.hot0], sc.n_hot0);
    if (sc.n_hot1) atomicAdd(&s_cnt[sc.hot1], sc.n_hot1);
  }
  __syncthreads();
  int4 *dst = reinterpret_cast<int4 *>(c.part + (int64_t)item * kCntBinKeys);
  for (int j = threadIdx.x; j < kCntBinKeys / 4; j += kCntThreads) dst[j] = cnt4[j];
}

// A quarter of a bin per workgroup of 256 lanes: the items' counts summed
// (16-byte loads, four items in flight), the non-zero ones gathered in LDS
// and appended to the column's list with coalesced stores.
constexpr int kEmitThreads = 256;
constexpr int kEmitKeys = 4096;

__global__ __launch_bounds__(kEmitThreads) void count_emit_kernel(const CountArgs A) {
  __shared__ uint32_t s_n, s_base;
  __shared__ uint16_t s_key[kEmitKeys];
  __shared__ int32_t s_wt[kEmitKeys];
  const CountCol &c = A.c[blockIdx.y];
  CountState *st = A.st + blockIdx.y;
  constexpr int kSub = kCntBinKeys / kEmitKeys;
  const int bin = blockIdx.x / kSub, sub = blockIdx.x % kSub;
  if (bin >= c.nbins || st->bad) return;
  const uint2 bi = c.bin_item[bin];
  if (bi.y == 0) return;
  constexpr int kQ = kEmitKeys / 4 / kEmitThreads;  // int4 per lane
  if (threadIdx.x == 0) s_n = 0;
  int4 a[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) a[q] = make_int4(0, 0, 0, 0);
  const int4 *p = reinterpret_cast<const int4 *>(c.part + (int64_t)bi.x * kCntBinKeys +
                                                 sub * kEmitKeys) + threadIdx.x;
  auto take = [&](int4 &t, const int4 &v) {
    t.x += v.x;
    t.y += v.y;
    t.z += v.z;
    t.w += v.w;
  };
  uint32_t i = 0;
  for (; i + 4 <= bi.y; i += 4, p += kCntBinKeys) {
    int4 v[4][kQ];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int q = 0; q < kQ; ++q) v[u][q] = p[u * (kCntBinKeys / 4) + q * kEmitThreads];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int q = 0; q < kQ; ++q) take(a[q], v[u][q]);
  }
  for (; i < bi.y; ++i, p += kCntBinKeys / 4)
#pragma unroll
    for (int q = 0; q < kQ; ++q) take(a[q], p[q * kEmitThreads]);
  __syncthreads();
  uint32_t n = 0;
#pragma unroll
  for (int q = 0; q < kQ; ++q)
    n += (a[q].x != 0) + (a[q].y != 0) + (a[q].z != 0) + (a[q].w != 0);
  uint32_t inc = n;
  const int lane = __lane_id();
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = __shfl_up(inc, o);
    if (lane >= o) inc += u;
  }
  uint32_t at = 0;
  if (lane == 63) at = atomicAdd(&s_n, inc);
  at = __shfl(at, 63) + inc - n;
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    const int32_t v[4] = {a[q].x, a[q].y, a[q].z, a[q].w};
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (v[u]) {
        s_key[at] = (uint16_t)(4 * (q * kEmitThreads + threadIdx.x) + u);
        s_wt[at] = v[u];
        ++at;
      }
  }
  __syncthreads();
  const uint32_t all = s_n;
  if (threadIdx.x == 0) s_base = atomicAdd(&st->n_keys, all);
  __syncthreads();
  const uint32_t base = s_base;
  const uint32_t key0 = ((uint32_t)bin << kCntBinBits) + sub * kEmitKeys;
  for (uint32_t k = threadIdx.x; k < all; k += kEmitThreads) {
    c.keys[base + k] = key0 + s_key[k];
    c.wts[base + k] = s_wt[k];
  }
}

// ---------------------------------------------------------------------
// weighted scan
// ---------------------------------------------------------------------
// R distinct keys per lane (below 2^31) into one slice's LDS counters.
template <int R>
__device__ __forceinline__ void weighted_adds(const uint32_t (&x)[R],
                                              const int32_t (&wt)[R],
                                              const RowSeeds &s, const BucketMod &bm,
                                              int32_t *cnt) {
  uint64_t v[R], g[R];
#pragma unroll
  for (int k = 0; k < R; ++k) v[k] = madd61_x31(s.a3, x[k], s.a2);
#pragma unroll
  for (int k = 0; k < R; ++k) g[k] = madd61_x31(s.b1, x[k], s.b0);
#pragma unroll
  for (int k = 0; k < R; ++k) v[k] = madd61_x31(v[k], x[k], s.a1);
#pragma unroll
  for (int k = 0; k < R; ++k) v[k] = madd61_x31(v[k], x[k], s.a0);
  uint32_t b[R];
  if (bm.pow2) {
#pragma unroll
    for (int k = 0; k < R; ++k) b[k] = low_of_residue(g[k]) & bm.mask;
  } else {
#pragma unroll
    for (int k = 0; k < R; ++k) b[k] = bucket_of(canon61(g[k]), bm);
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    uint32_t lr = low_of_residue(v[k]);
    __asm__("" : "+v"(lr));
    const int32_t par = __builtin_amdgcn_sbfe((int32_t)lr, 0, 1);  // 0 or -1
    atomicAdd(&cnt[b[k]], (wt[k] ^ par) - par);
  }
}

template <int R>
__device__ __forceinline__ void weighted_rows(const WeightedArgs &W, int col,
                                              uint32_t i0, uint32_t end, int sb,
                                              int ns, int32_t *cnt) {
  uint32_t x[R];
  int32_t wt[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const uint32_t i = i0 + threadIdx.x + k * kBuildThreads;
    const bool in = i < end;
    x[k] = in ? W.keys[col][i] : 0u;
    wt[k] = in ? W.wts[col][i] : 0;
  }
  for (int l0 = 0; l0 < ns; ++l0) {
    const int l = __builtin_amdgcn_readfirstlane(l0);
    const RowSeeds s = W.seeds[sb + l];
    weighted_adds<R>(x, wt, s, W.bm, cnt + (size_t)l * W.bm.w);
  }
}

// The lists' rows are cut into chunks of one size for every column, as many
// as the resident workgroups take in one wave (at least 4096 rows each:
// clearing and writing back a workgroup's partials costs about as much as
// hashing 2000); a workgroup finds its (slice group, chunk) from the lists'
// lengths.
__global__ __launch_bounds__(kBuildThreads) void weighted_scan_kernel(
    const WeightedArgs W) {
  extern __shared__ int32_t cnt[];
  const int ng = W.n_groups;
  uint64_t rows = 0;
  int live = 0;
  uint32_t longest = 0;
  for (int g = 0; g < ng; ++g) {
    const CountState &s = W.st[W.group_col[g]];
    const uint32_t n = s.bad ? 0u : s.n_keys;
    rows += n;
    live += n ? 1 : 0;
    longest = max(longest, n);
  }
  if (!live) return;
  const int slots = max(1, W.slots - live);
  uint32_t per = (uint32_t)((rows + slots - 1) / slots);
  per = max(per, 4096u);
  per = max(per, (longest + W.max_chunks - 1) / W.max_chunks);
  per = (per + 1023u) & ~1023u;
  uint32_t lin = blockIdx.x, chunk = 0, n = 0;
  int gi = -1;
  for (int g = 0; g < ng; ++g) {
    const CountState &s = W.st[W.group_col[g]];
    const uint32_t m = s.bad ? 0u : s.n_keys;
    const uint32_t chunks = (m + per - 1) / per;
    if (blockIdx.x == 0 && !s.bad && (int)threadIdx.x >= W.group_begin[g] &&
        (int)threadIdx.x < W.group_begin[g + 1])
      W.slice_chunks[W.gs[threadIdx.x]] = (int32_t)chunks;
    if (gi < 0) {
      if (lin < chunks) {
        gi = g;
        chunk = lin;
        n = m;
      } else {
        lin -= chunks;
      }
    }
  }
  gi = __builtin_amdgcn_readfirstlane(gi);
  if (gi < 0) return;
  const int sb = W.group_begin[gi], ns = W.group_begin[gi + 1] - sb;
  const int col = W.group_col[gi];
  const int w = (int)W.bm.w;
  for (int i = threadIdx.x; i < ns * w; i += kBuildThreads) cnt[i] = 0;
  __syncthreads();
  uint32_t a = chunk * per;
  const uint32_t b = min(n, a + per);
  for (; a + 8 * kBuildThreads <= b; a += 8 * kBuildThreads)
    weighted_rows<8>(W, col, a, b, sb, ns, cnt);
  for (; a < b; a += 2 * kBuildThreads)
    weighted_rows<2>(W, col, a, b, sb, ns, cnt);
  // the chunk's share of the keys outside the counted range
  const uint32_t ne = W.st[col].n_exc, nc = (n + per - 1) / per;
  const uint32_t e1 = (uint32_t)((uint64_t)ne * (chunk + 1) / nc);
  for (uint32_t e = (uint32_t)((uint64_t)ne * chunk / nc) + threadIdx.x; e < e1;
       e += kBuildThreads) {
    const uint64_t x = W.exc[col][e];
    for (int l = 0; l < ns; ++l) {
      int32_t sign;
      uint32_t bk;
      hash_xi_h<false>(x, W.seeds[sb + l], W.bm, sign, bk);
      atomicAdd(&cnt[(size_t)l * w + bk], sign);
    }
  }
  __syncthreads();
  for (int l = 0; l < ns; ++l) {
    const size_t gs = (size_t)W.gs[sb + l];
    int32_t *dst = W.slab + ((size_t)chunk * W.n_slices_total + gs) * w;
    const int32_t *src = cnt + (size_t)l * w;
    for (int j = threadIdx.x; j < w; j += kBuildThreads) dst[j] = src[j];
  }
}

hipError_t launch_count_start(const ZeroSpans &z, const CountArgs &A, hipStream_t st) {
  int64_t most = 1;
  for (int k = 0; k < z.n; ++k) most = std::max(most, z.words[k]);
  const int64_t blocks =
      std::max<int64_t>(A.n_cols, std::min<int64_t>((most + 255) / 256, 1024));
  hipLaunchKernelGGL(count_start_kernel, dim3((unsigned)blocks, (unsigned)z.n + 1),
                     dim3(256), 0, st, z, A);
  return hipGetLastError();
}

hipError_t launch_count(const CountArgs &A, int n_wg, int max_bins, int max_items,
                        int max_stride, hipStream_t st) {
  hipLaunchKernelGGL(count_partition_kernel, dim3(n_wg, A.n_cols), dim3(kCntThreads),
                     (size_t)max_stride * 2, st, A);
  hipLaunchKernelGGL(count_plan_kernel, dim3((max_bins + 63) / 64, A.n_cols), dim3(64),
                     0, st, A);
  hipLaunchKernelGGL(count_items_kernel, dim3((max_items + kXcds - 1) / kXcds * kXcds, A.n_cols), dim3(kCntThreads),
                     0, st, A);
  hipLaunchKernelGGL(count_emit_kernel,
                     dim3(max_bins * (kCntBinKeys / kEmitKeys), A.n_cols),
                     dim3(kEmitThreads), 0, st, A);
  return hipGetLastError();
}

hipError_t launch_weighted_scan(const WeightedArgs &W, size_t lds, hipStream_t st) {
  hipLaunchKernelGGL(weighted_scan_kernel, dim3(W.slots), dim3(kBuildThreads), lds, st, W);
  return hipGetLastError();
}

}  // namespace compass
