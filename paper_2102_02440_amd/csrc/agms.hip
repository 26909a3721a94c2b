// agms.hip -- the AGMS baseline (Section 4.1) that Fast-AGMS improves on.
//
//  agms_build_kernel  fused selection scan; for every qualifying row, every
//                     one of the K = r * b basic sketches adds the product
//                     over the table's joins of that join's +-1 variable of
//                     the row's key (the composed sketch of a table in a
//                     multi-way join).  A tile's survivors are compacted
//                     (the same ballot compaction as the Fast-AGMS scan) and
//                     their key field elements staged in LDS; lane (c, part)
//                     owns basic sketch c (its seeds in registers) and every
//                     parts-th survivor, reading keys by LDS broadcast.  The
//                     cost is K sign evaluations per join per row -- the
//                     update cost that makes AGMS impractical (Section 4.1.4).
//  agms_start / agms_signs / agms_gather  large tables without predicates
//                     whose keys repeat: the signs of every key of a
//                     column's range are evaluated once, K bits per key
//                     (joins on one column multiplied, i.e. xor-ed), and a
//                     row's K products are the xor of its keys' words; the
//                     bits are counted per sketch in bit-sliced counters.
//                     18M rows of three joins on two columns (1.25M and 2M
//                     keys), K = 112: 6 G sign evaluations, 8.4 ms, become
//                     0.5 G and two 16-byte gathers per row, 0.70 ms.  Rows
//                     with a key outside the range the sample gave are
//                     evaluated one by one.
//  agms_estimate      basic estimate (i, j) = product of the tables' counters;
//                     exact 128-bit row sums, averages over b, median over r.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "agms_params.hpp"
#include "device_math.hpp"
#include "scan_common.hpp"

namespace compass {

struct AgmsJob {
  const AgmsParams &P;
  __device__ int n_preds() const { return P.n_preds; }
  __device__ const PredDev &pred(int q) const { return P.preds[q]; }
};

// +-1 variable of one field element under one basic sketch's seeds
// (the lanes of a wave mostly share the key: the width test is nearly
// always uniform)
__device__ __forceinline__ int32_t agms_xi(uint64_t x, const RowSeeds &s) {
  uint64_t v;
  if ((x >> 31) == 0) {
    const uint32_t x32 = (uint32_t)x;
    v = madd61_x31(s.a3, x32, s.a2);
    v = madd61_x31(v, x32, s.a1);
    v = madd61_x31(v, x32, s.a0);
  } else if ((x >> 32) == 0) {
    const uint32_t x32 = (uint32_t)x;
    v = madd61_x32(s.a3, x32, s.a2);
    v = madd61_x32(v, x32, s.a1);
    v = madd61_x32(v, x32, s.a0);
  } else {
    v = madd61_x61(s.a3, x, s.a2);
    v = madd61_x61(v, x, s.a1);
    v = madd61_x61(v, x, s.a0);
  }
  // parity as add-with-carry plus bit extract, then doubled | 1
  uint32_t lr = low_of_residue(v);
  __asm__("" : "+v"(lr));
  int32_t par = __builtin_amdgcn_sbfe((int32_t)lr, 0, 1);
  __asm__("" : "+v"(par));
  return (int32_t)((uint32_t)par << 1) | 1;
}

// ---------------------------------------------------------------------
// sign tables
// ---------------------------------------------------------------------
__device__ __forceinline__ uint64_t agms_raw(const KeyDev &k, int64_t row) {
  return k.dtype == kDtI32
             ? (uint64_t)(int64_t)reinterpret_cast<const int32_t *>(k.col)[row]
             : reinterpret_cast<const uint64_t *>(k.col)[row];
}

// One workgroup: 1024 keys of every column, spread over its rows.  The range
// of a column ends past the largest key seen (of those its table can hold);
// bad when more than 16 keys cannot be held, or when the signs to evaluate
// would cost more than P.tab.most_lanes.
__global__ __launch_bounds__(1024) void agms_start_kernel(const AgmsParams P) {
  __shared__ uint32_t s_max[kAgmsMaxJoins], s_out[kAgmsMaxJoins];
  if (threadIdx.x < kAgmsMaxJoins) s_max[threadIdx.x] = s_out[threadIdx.x] = 0;
  const int64_t row = P.n_rows * (int64_t)threadIdx.x / 1024;
  uint64_t x[kAgmsMaxJoins];
#pragma unroll
  for (int c = 0; c < kAgmsMaxJoins; ++c)
    if (c < P.tab.n_cols) x[c] = agms_raw(P.tab.col[c], row);
  __syncthreads();
#pragma unroll
  for (int c = 0; c < kAgmsMaxJoins; ++c) {
    if (c >= P.tab.n_cols) break;
    const bool in = x[c] < P.tab.cap[c];
    const uint32_t out = 64 - (uint32_t)__popcll(__ballot(in));
    uint32_t m = in ? (uint32_t)x[c] + 1 : 0u;
#pragma unroll
    for (int d = 32; d; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d));
    if ((threadIdx.x & 63) == 0) {
      atomicMax(&s_max[c], m);
      atomicAdd(&s_out[c], out);
    }
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  AgmsState st;
  memset(&st, 0, sizeof st);
  int64_t lanes = 0;
  for (int c = 0; c < P.tab.n_cols; ++c) {
    st.range[c] = s_max[c];
    lanes += (int64_t)s_max[c] * P.tab.col_joins[c] * ((P.K + 63) / 64 * 64);
    if (s_out[c] > 16) st.bad = 1;
  }
  if (lanes > P.tab.most_lanes) st.bad = 1;
  *P.tab.st = st;
}

// Signs of the keys of [0, range).  A lane owns one basic sketch, a wave 64 of
// them and runs of kSignRun consecutive keys: the sign polynomial is of degree
// three, so its value at the next key is three additions of finite differences
// (mod p) away, and the wave's ballot of the parities is the 64 sketches' word
// of the key.  Bound by the adds: 19 VALU instructions per key, join and
// sketch; 0.5 G signs (and an eighth of idle lanes at K = 112) take 300 us,
// 1.9 T per second, against 380 us by Horner's rule with a lane per key.
// Residues r are held as 8 r, or biased as 8 r + 8, in 64 bits: plain + biased
// carries out of the word exactly when the sum reaches p, and is then already
// reduced, so every value is the canonical one.
constexpr int kSignThreads = 256;
constexpr int kSignRun = 128;

// v with lane `lane` replaced by the wave-uniform x
extern "C" __device__ uint32_t write_lane(uint32_t x, uint32_t lane, uint32_t v) __asm(
    "llvm.amdgcn.writelane.i32");

__device__ __forceinline__ uint64_t horner3(const RowSeeds &s, uint32_t x) {
  uint64_t v = madd61_x31(s.a3, x, s.a2);
  v = madd61_x31(v, x, s.a1);
  return canon61(madd61_x31(v, x, s.a0));
}

__device__ __forceinline__ uint64_t sub61(uint64_t a, uint64_t b) {
  return a >= b ? a - b : a + kP61 - b;
}

// residue of the sum of a plain and a biased value, plain / biased
__device__ __forceinline__ uint64_t add_plain(uint64_t a, uint64_t b) {
  unsigned long long t;
  const bool c = __builtin_add_overflow((unsigned long long)a, (unsigned long long)b, &t);
  return t - (c ? 0u : 8u);
}
__device__ __forceinline__ uint64_t add_biased(uint64_t a, uint64_t b) {
  unsigned long long t;
  const bool c = __builtin_add_overflow((unsigned long long)a, (unsigned long long)b, &t);
  return t + (c ? 8u : 0u);
}

__global__ __launch_bounds__(kSignThreads) void agms_signs_kernel(const AgmsParams P) {
  const AgmsTables &T = P.tab;
  if (T.st->bad) return;
  const int lane = threadIdx.x & 63;
  const int halves = (P.K + 63) / 64;
  uint32_t u = blockIdx.x * (kSignThreads / 64) + (threadIdx.x >> 6);
  const uint32_t stride = gridDim.x * (kSignThreads / 64);
  for (int c = 0; c < T.n_cols; ++c) {
    const uint32_t runs = (T.st->range[c] + kSignRun - 1) / kSignRun;
    const uint32_t units = runs * halves;
    for (; u < units; u += stride) {
      const uint32_t run = u / halves;
      const int h = u - run * halves;
      const uint32_t x0 = run * kSignRun;
      const int k = min(64 * h + lane, P.K - 1);
      uint32_t klo[kSignRun / 64], khi[kSignRun / 64];
#pragma unroll
      for (int j = 0; j < kSignRun / 64; ++j) klo[j] = khi[j] = 0;
      for (int e = 0; e < T.col_joins[c]; ++e) {
        const RowSeeds s = P.seeds[(size_t)T.join[c][e] * P.K + k];
        const uint64_t h0 = horner3(s, x0), h1 = horner3(s, x0 + 1);
        const uint64_t h2 = horner3(s, x0 + 2), h3 = horner3(s, x0 + 3);
        const uint64_t e0 = sub61(h1, h0), e1 = sub61(h2, h1), e2 = sub61(h3, h2);
        const uint64_t f0 = sub61(e1, e0), f1 = sub61(e2, e1);
        uint64_t v = h0 << 3, d1 = (e0 << 3) + 8, d2 = f0 << 3;
        const uint64_t d3 = (sub61(f1, f0) << 3) + 8;
#pragma unroll 1
        for (int j = 0; j < kSignRun / 64; ++j) {
          uint32_t lo = 0, hi = 0;   // lane i: the word of key x0 + 64 j + i
#pragma unroll
          for (int i = 0; i < 64; ++i) {
            const uint64_t m = __ballot(((uint32_t)v & 8u) != 0);
            lo = write_lane((uint32_t)m, i, lo);
            hi = write_lane((uint32_t)(m >> 32), i, hi);
            v = add_plain(v, d1);
            d1 = add_biased(d1, d2);
            d2 = add_plain(d2, d3);
          }
#pragma unroll
          for (int q = 0; q < kSignRun / 64; ++q) {
            klo[q] ^= q == j ? lo : 0u;
            khi[q] ^= q == j ? hi : 0u;
          }
        }
      }
      uint2 *out = reinterpret_cast<uint2 *>(T.signs[c]) +
                   (size_t)(h >> 1) * T.cap[c] * 2 + (h & 1);
#pragma unroll
      for (int j = 0; j < kSignRun / 64; ++j) {
        const uint32_t x = x0 + 64 * j + lane;
        if (x < T.cap[c]) out[(size_t)x * 2] = make_uint2(klo[j], khi[j]);
      }
    }
    u -= units;
  }
}

// Bit-sliced counters: plane p of a word holds bit p of the 32 counts.
constexpr int kPlanes = 12;              // up to 4095 rows per lane
constexpr int kGatherThreads = 512;
constexpr int kGatherRows = 8;           // rows per lane and round
constexpr int kGatherMax = (1 << kPlanes) - 1;

// (a, b, c) -> sum bit into a, carry bit returned
__device__ __forceinline__ uint32_t csa(uint32_t &a, uint32_t b, uint32_t c) {
  const uint32_t x = a ^ b;
  const uint32_t carry = (a & b) | (x & c);
  a = x ^ c;
  return carry;
}

// One workgroup per (chunk of rows, group of 128 sketches).  Bound by the
// gathers: 18M rows of two columns whose tables (20 and 32 MB) exceed an
// XCD's L2 take 390 us, 93 G gathers per second; the counters' carry-save
// adders hide behind them (4 words of 8 rows cost 84 logic instructions).
__global__ __launch_bounds__(kGatherThreads) void agms_gather_kernel(const AgmsParams P,
                                                                     int64_t chunk) {
  __shared__ int32_t s_cnt[kAgmsGroup];
  __shared__ int32_t s_xi[kAgmsGroup];     // sum of the rows evaluated one by one
  __shared__ int32_t s_queue[kGatherThreads * kGatherRows];
  __shared__ int32_t s_qn;
  const AgmsTables &T = P.tab;
  if (T.st->bad) return;
  const int g = blockIdx.y;
  const int64_t row0 = (int64_t)blockIdx.x * chunk;
  const int64_t row1 = min(P.n_rows, row0 + chunk);
  if (threadIdx.x < kAgmsGroup) s_cnt[threadIdx.x] = s_xi[threadIdx.x] = 0;
  if (threadIdx.x == 0) s_qn = 0;
  __syncthreads();
  uint32_t pl[4][kPlanes];
#pragma unroll
  for (int w = 0; w < 4; ++w)
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) pl[w][p] = 0;
  int64_t exceptions = 0;
  constexpr int kRound = kGatherThreads * kGatherRows;
  for (int64_t base = row0; base < row1; base += kRound) {
    const int nt = (int)min((int64_t)kRound, row1 - base);
    uint32_t carry4[2][4];   // weight 4 after each half of the rows
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      constexpr int kH = kGatherRows / 2;
      uint32_t bits[kH][4];
      bool in[kH];
#pragma unroll
      for (int u = 0; u < kH; ++u) {
        in[u] = (int)threadIdx.x + (h * kH + u) * kGatherThreads < nt;
#pragma unroll
        for (int w = 0; w < 4; ++w) bits[u][w] = 0;
      }
      bool out[kH];
#pragma unroll
      for (int u = 0; u < kH; ++u) out[u] = false;
      for (int c = 0; c < T.n_cols; ++c) {   // uniform
        const uint32_t range = T.st->range[c];
        uint32_t key[kH];
#pragma unroll
        for (int u = 0; u < kH; ++u) {
          const int r = (int)threadIdx.x + (h * kH + u) * kGatherThreads;
          const uint64_t x = agms_raw(T.col[c], base + min(r, nt - 1));
          out[u] = out[u] || x >= range;
          key[u] = x < range ? (uint32_t)x : 0u;
        }
        uint4 v[kH];
#pragma unroll
        for (int u = 0; u < kH; ++u) v[u] = T.signs[c][(size_t)g * T.cap[c] + key[u]];
#pragma unroll
        for (int u = 0; u < kH; ++u) {
          bits[u][0] ^= v[u].x;
          bits[u][1] ^= v[u].y;
          bits[u][2] ^= v[u].z;
          bits[u][3] ^= v[u].w;
        }
      }
#pragma unroll
      for (int u = 0; u < kH; ++u) {
        if (in[u] && out[u]) {
          const int r = (int)threadIdx.x + (h * kH + u) * kGatherThreads;
          s_queue[atomicAdd(&s_qn, 1)] = r;
        }
        const bool take = in[u] && !out[u];
#pragma unroll
        for (int w = 0; w < 4; ++w) bits[u][w] = take ? bits[u][w] : 0u;
      }
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t t0 = csa(pl[w][0], bits[0][w], bits[1][w]);
        const uint32_t t1 = csa(pl[w][0], bits[2][w], bits[3][w]);
        carry4[h][w] = csa(pl[w][1], t0, t1);
      }
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      uint32_t k = csa(pl[w][2], carry4[0][w], carry4[1][w]);   // weight 8
#pragma unroll
      for (int p = 3; p < kPlanes; ++p) {
        const uint32_t t = pl[w][p] & k;
        pl[w][p] ^= k;
        k = t;
      }
    }
    // rows with a key outside the ranges: lane k evaluates basic sketch k of
    // the group, a quarter of the workgroup per row
    if (__syncthreads_or(s_qn)) {
      const int n = s_qn;
      const int k = threadIdx.x % kAgmsGroup, c = g * kAgmsGroup + k;
      if (c < P.K) {
        int32_t sum = 0;
        for (int i = threadIdx.x / kAgmsGroup; i < n; i += kGatherThreads / kAgmsGroup) {
          int32_t prod = 1;
          for (int e = 0; e < P.n_joins; ++e)
            prod *= agms_xi(load_field(P.keys[e], base + s_queue[i]),
                            P.seeds[(size_t)e * P.K + c]);
          sum += prod;
        }
        if (sum) atomicAdd(&s_xi[k], sum);
      }
      exceptions += n;
      __syncthreads();
      if (threadIdx.x == 0) s_qn = 0;
      __syncthreads();
    }
  }
  // the lanes' counts summed in their bit-sliced form: first two exchanges
  // split the four words (lane bits 5 and 4 pick the word a lane keeps),
  // the other four leave the word's sums in all 16 lanes of its group
  const int lane = threadIdx.x & 63;
  uint32_t two[2][kPlanes + 1];
  {
    const bool hi = lane & 32;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      uint32_t k = 0;
#pragma unroll
      for (int p = 0; p < kPlanes; ++p) {
        const uint32_t got = __shfl_xor(hi ? pl[w][p] : pl[w + 2][p], 32);
        uint32_t a = hi ? pl[w + 2][p] : pl[w][p];
        k = csa(a, got, k);
        two[w][p] = a;
      }
      two[w][kPlanes] = k;
    }
  }
  uint32_t one[kPlanes + 6];
  {
    const bool hi = lane & 16;
    uint32_t k = 0;
#pragma unroll
    for (int p = 0; p <= kPlanes; ++p) {
      const uint32_t got = __shfl_xor(hi ? two[0][p] : two[1][p], 16);
      uint32_t a = hi ? two[1][p] : two[0][p];
      k = csa(a, got, k);
      one[p] = a;
    }
    one[kPlanes + 1] = k;
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    uint32_t k = 0;
#pragma unroll
    for (int p = 0; p <= kPlanes + 1 + s; ++p) {
      const uint32_t got = __shfl_xor(one[p], 8 >> s);
      k = csa(one[p], got, k);
    }
    one[kPlanes + 2 + s] = k;
  }
  const int word = 2 * (lane >> 5) + ((lane >> 4) & 1);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int bit = 2 * (lane & 15) + u;
    uint32_t n = 0;
#pragma unroll
    for (int p = 0; p < kPlanes + 6; ++p) n |= ((one[p] >> bit) & 1u) << p;
    atomicAdd(&s_cnt[32 * word + bit], (int32_t)n);
  }
  __syncthreads();
  const int c = g * kAgmsGroup + (int)threadIdx.x;
  if (threadIdx.x < kAgmsGroup && c < P.K) {
    // -1 for every set bit, +1 for the others
    const int64_t rows = row1 - row0 - exceptions;
    const int64_t t = rows - 2 * (int64_t)s_cnt[threadIdx.x] + s_xi[threadIdx.x];
    if (t) atomicAdd(reinterpret_cast<unsigned long long *>(P.counters + c),
                     (unsigned long long)t);
  }
  if (g == 0 && threadIdx.x == 0)
    atomicAdd(reinterpret_cast<unsigned long long *>(P.n_selected),
              (unsigned long long)(row1 - row0));
}

__global__ __launch_bounds__(kBuildThreads) void agms_build_kernel(
    const AgmsParams P) {
  extern __shared__ uint64_t xs[];  // [join][kBuildTile] survivor keys
  __shared__ int32_t queue[kBuildTile];
  __shared__ int32_t s_qn;
  __shared__ int64_t red[kBuildThreads];
  const AgmsJob job{P};
  if (P.tab.st && !P.tab.st->bad) return;   // agms_gather_kernel's
  const int K = P.K;
  const int parts = kBuildThreads / K;
  const int c = threadIdx.x % K;
  const int part = threadIdx.x / K;  // parts .. : idle lanes
  const bool lane_on = part < parts;
  RowSeeds sd[kAgmsMaxJoins];
#pragma unroll
  for (int e = 0; e < kAgmsMaxJoins; ++e)
    if (e < P.n_joins && lane_on) sd[e] = P.seeds[(size_t)e * K + c];
  int64_t acc = 0;
  uint64_t sel = 0;
  const int64_t row0 = (int64_t)blockIdx.x * P.rows_per_chunk;
  const int64_t row1 = min(row0 + P.rows_per_chunk, P.n_rows);
  for (int64_t base = row0; base < row1; base += P.tile) {
    const int nt = (int)min((int64_t)P.tile, row1 - base);
    const int qn = compact_tile<AgmsJob, kBuildRowsPerThread>(
        job, base, nt, P.n_preds, queue, &s_qn);
    sel += (uint64_t)qn;
    for (int e = 0; e < P.n_joins; ++e)
      for (int q = threadIdx.x; q < qn; q += kBuildThreads)
        xs[(size_t)e * kBuildTile + q] =
            load_field(P.keys[e], base + (P.n_preds ? queue[q] : q));
    __syncthreads();
    if (lane_on) {
      for (int q = part; q < qn; q += parts) {
        int32_t prod = 1;
#pragma unroll
        for (int e = 0; e < kAgmsMaxJoins; ++e)
          if (e < P.n_joins) prod *= agms_xi(xs[(size_t)e * kBuildTile + q], sd[e]);
        acc += prod;
      }
    }
    __syncthreads();  // xs, queue and s_qn are reused by the next tile
  }
  red[threadIdx.x] = lane_on ? acc : 0;
  __syncthreads();
  if (threadIdx.x < K) {
    int64_t t = 0;
    for (int p = 0; p < parts; ++p) t += red[p * K + threadIdx.x];
    if (t) atomicAdd(reinterpret_cast<unsigned long long *>(P.counters + threadIdx.x),
                     (unsigned long long)t);
  }
  if (P.count_selected && threadIdx.x == 0 && sel)
    atomicAdd(reinterpret_cast<unsigned long long *>(P.n_selected),
              (unsigned long long)sel);
}

hipError_t launch_agms_build(const AgmsParams &P, int n_blocks, int n_cu,
                             hipStream_t st) {
  if (P.tab.st) {
    hipLaunchKernelGGL(agms_start_kernel, dim3(1), dim3(1024), 0, st, P);
    hipLaunchKernelGGL(agms_signs_kernel, dim3((unsigned)(8 * n_cu)),
                       dim3(kSignThreads), 0, st, P);
    // one wave of workgroups (two per CU), whole rounds, the lanes' counts
    // below the planes' limit
    constexpr int64_t kRound = kGatherThreads * kGatherRows;
    constexpr int64_t kMost = kGatherMax / kGatherRows * kRound;
    const int64_t want = std::max<int64_t>(1, 2 * n_cu / P.tab.n_groups);
    int64_t chunk = ((P.n_rows + want - 1) / want + kRound - 1) / kRound * kRound;
    chunk = std::min(chunk, kMost);
    hipLaunchKernelGGL(agms_gather_kernel,
                       dim3((unsigned)((P.n_rows + chunk - 1) / chunk),
                            (unsigned)P.tab.n_groups),
                       dim3(kGatherThreads), 0, st, P, chunk);
  }
  const size_t lds = (size_t)P.n_joins * kBuildTile * 8;
  hipLaunchKernelGGL(agms_build_kernel, dim3(n_blocks), dim3(kBuildThreads),
                     lds, st, P);
  return hipGetLastError();
}

// One workgroup: a lane per basic estimate, then a lane per row's sum.
constexpr int kAgmsEstThreads = 256;

__global__ __launch_bounds__(kAgmsEstThreads) void agms_estimate_kernel(
    AgmsEstArgs a, uint64_t *row_sums, double *est, int32_t *flag) {
  __shared__ double avg[64];
  __shared__ u128 basic[kAgmsMaxCounters];
  const int r = a.r, b = a.b;
  for (int k = threadIdx.x; k < r * b; k += kAgmsEstThreads) {
    int64_t v[16];
#pragma unroll
    for (int t = 0; t < 16; ++t)
      if (t < a.n_tables) v[t] = a.sk[t][k];
    u128 x = 1;
#pragma unroll
    for (int t = 0; t < 16; ++t)
      if (t < a.n_tables) x = mul_u128(x, s64_to_u128(v[t]));
    basic[k] = x;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < r; i += blockDim.x) {
    u128 sum = 0;
    for (int j = 0; j < b; ++j) sum += basic[i * b + j];
    if (row_sums) {
      row_sums[2 * i] = (uint64_t)sum;
      row_sums[2 * i + 1] = (uint64_t)(sum >> 64);
    }
    avg[i] = i128_to_double(sum) / (double)b;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int i = 1; i < r; ++i) {  // insertion sort of r <= 64 averages
    const double v = avg[i];
    int k = i - 1;
    while (k >= 0 && avg[k] > v) {
      avg[k + 1] = avg[k];
      --k;
    }
    avg[k + 1] = v;
  }
  *est = (r & 1) ? avg[r / 2] : (avg[r / 2 - 1] + avg[r / 2]) * 0.5;
  // product of the selected rows below 2^127 (no division: in 128 bits it is
  // a loop over the bits, 8 us per table)
  const u128 lim = (u128)1 << 127;
  u128 p = 1;
  bool ok = true;
  for (int t = 0; t < a.n_tables && ok; ++t) {
    const int64_t n = *a.n_sel[t];
    const uint64_t f = n < 0 ? 0 : (uint64_t)n;
    if (f == 0) {
      p = 0;
      break;
    }
    const u128 hi = mul_u64_full((uint64_t)(p >> 64), f);
    const u128 lo = mul_u64_full((uint64_t)p, f);
    const u128 mid = hi + (lo >> 64);
    if (mid > (lim >> 64))
      ok = false;
    else
      p = (mid << 64) | (uint64_t)lo, ok = p <= lim;
  }
  *flag = ok && p < lim ? 1 : 0;
}

hipError_t launch_agms_estimate(const AgmsEstArgs &a, uint64_t *row_sums,
                                double *est, int32_t *flag, hipStream_t st) {
  hipLaunchKernelGGL(agms_estimate_kernel, dim3(1), dim3(kAgmsEstThreads), 0, st, a,
                     row_sums, est, flag);
  return hipGetLastError();
}

}  // namespace compass
