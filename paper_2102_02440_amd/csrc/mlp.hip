// mlp.hip -- learned correction of sketch estimates (gfx950 kernels).
//
// A small MLP (n_in -> H -> ... -> H -> 1, ReLU) maps per-row sketch
// estimates, selected sizes and sub-plan shape to a correction of the log
// cardinality: y = ln(1 + max(raw, 0)) + net(x), so the zero network is the
// raw median estimate, which stays the fallback.  Weights are kept in fp32
// (master, Adam state) and in bfloat16 (the copy the products read); every
// layer rounds its input activations to bfloat16 and accumulates in fp32.
//
// Kernels: a workgroup takes 16 samples, a wave 16 of a layer's outputs, the
// products on the matrix cores in fp32 (v_mfma_f32_16x16x4_f32: each result
// is the chain of fused multiply-adds over the inputs in ascending order,
// the same bits as a scalar loop; measured on random, cancelling and tiny
// values).  A step is 0.04 GFLOP, so its latency counts: the weights are
// kept a second time as float images in the order of the fragments, both
// ways round, and go from memory to registers in one round of loads.
// 512-sample steps of the 20-64-64-64-1 network: 64 us with staged weight
// tiles and scalar products, 18 us so (step 14, sum and Adam 4).  Every sum keeps one order
// (inputs ascending, samples ascending within groups of 8, groups
// ascending), in fp32.
//   mlp_fwd_kernel     forward pass, tiles walked by a persistent grid
//   mlp_step_kernel    forward and backward, partial gradients of every
//                      8 samples (deterministic slab)
//   mlp_reduce_adam_kernel  sums the slab in a fixed order, then Adam on
//                      the fp32 masters and the weight images
//   mlp_features_kernel  sub-plan features from the 128-bit row estimates
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "compass.h"
#include "device_math.hpp"

namespace compass {

constexpr int kMlpMaxDim = 64;
constexpr int kMlpMaxLayers = 8;
constexpr int kMlpPart = 8;        // samples of one gradient partial
constexpr int kMlpTile = 16;       // samples per workgroup
constexpr int kMlpThreads = 256;   // a wave per 16 outputs

// Images of a layer's weights, rounded to bfloat16: row o holds input i at
// mlp_slot(i) (and the other way round: row i holds output o), 64 x 64 with
// zeros where the layer is narrower; then its biases (fp32, 64).
constexpr int kMlpImage = kMlpMaxDim * kMlpMaxDim;
__device__ __host__ constexpr int mlp_slot(int i) { return (i & 3) * 16 + (i >> 2); }
// rows of activations and deltas in LDS (words): 16-byte aligned, 4 words off
// a multiple of the banks
constexpr int kMlpRow = kMlpMaxDim + 4;

struct MlpShape {
  int32_t n_layers;                  // weight layers (hidden + output)
  int32_t dim[kMlpMaxLayers + 1];    // dim[0] = n_in ... dim[n_layers] = 1
  int32_t woff[kMlpMaxLayers];       // offset of W_l in the flat parameters
  int32_t boff[kMlpMaxLayers];       // offset of b_l
  int32_t n_params;
};

__device__ __forceinline__ float bf16_to_f(uint16_t h) {
  return __uint_as_float((uint32_t)h << 16);
}

// round-to-nearest-even to bfloat16 (finite inputs)
__device__ __forceinline__ uint16_t f_to_bf16(float f) {
  const uint32_t u = __float_as_uint(f);
  const uint32_t lsb = (u >> 16) & 1u;
  return (uint16_t)((u + 0x7FFFu + lsb) >> 16);
}

__device__ __forceinline__ float round_bf16(float f) {
  return bf16_to_f(f_to_bf16(f));
}

__device__ __forceinline__ float lane_value(float v, int i) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), i));
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// 16 words of one lane in chunks of four, as many as `k` inputs need: lane
// (n = lane & 15, q = lane >> 4) of a fragment holds inputs 4 s + q at word s.
struct Frag {
  f32x4 v[4];
  __device__ __forceinline__ void load(const float *row, int k) {
    const int q = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      v[c] = f32x4{0, 0, 0, 0};
      if (16 * c < k) v[c] = *reinterpret_cast<const f32x4 *>(row + 16 * q + 4 * c);
    }
  }
};

// D = A B, the inputs in ascending order: A's rows the samples (row = lane &
// 15), B's columns the outputs; lane (n, q) gets samples 4 q + r of column n.
__device__ __forceinline__ f32x4 mlp_product(const Frag &a, const Frag &b, int k) {
  f32x4 acc = {0, 0, 0, 0};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if (16 * c >= k) break;   // uniform
#pragma unroll
    for (int u = 0; u < 4; ++u)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[c][u], b.v[c][u], acc, 0, 0, 0);
  }
  return acc;
}

// The weights of a wave's 16 columns of every layer and their biases.
struct MlpWeights {
  Frag w[kMlpMaxLayers];
  float bias[kMlpMaxLayers];
  __device__ __forceinline__ void load(const MlpShape &S, const float *__restrict__ img) {
    const int col = 16 * (threadIdx.x >> 6) + (threadIdx.x & 15);
#pragma unroll
    for (int l = 0; l < kMlpMaxLayers; ++l) {
      if (l >= S.n_layers) break;
      w[l].load(img + (size_t)l * kMlpImage + col * kMlpMaxDim,
                16 * (threadIdx.x >> 6) < S.dim[l + 1] ? S.dim[l] : 0);
      bias[l] = img[(size_t)2 * S.n_layers * kMlpImage + l * kMlpMaxDim + col];
    }
  }
};

// Rounded inputs of the tile's samples (row idx[s] of x, row s when idx is
// null; zeros past the last) to LDS.  All lanes call it.
__device__ __forceinline__ void mlp_load_inputs(const float *__restrict__ x,
                                                const int32_t *__restrict__ idx, int s0, int n,
                                                int n_in, float *a) {
  // a wave takes four samples, a lane one input
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  float v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int s = min(s0 + 4 * wave + u, n - 1);
    const size_t r = idx ? (size_t)idx[s] : (size_t)s;
    v[u] = x[r * n_in + min(lane, n_in - 1)];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const bool in = s0 + 4 * wave + u < n && lane < n_in;
    a[(4 * wave + u) * kMlpRow + mlp_slot(lane)] = in ? round_bf16(v[u]) : 0.f;
  }
}

__global__ __launch_bounds__(kMlpThreads) void mlp_fwd_kernel(
    MlpShape S, const float *__restrict__ img, const float *__restrict__ x,
    const float *__restrict__ base, int32_t n, float *__restrict__ y) {
  __shared__ __align__(16) float s_a[2][kMlpTile * kMlpRow];
  MlpWeights W;
  W.load(S, img);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = lane & 15, q = lane >> 4, col = 16 * wave + m;
  const int tiles = (n + kMlpTile - 1) / kMlpTile;
  for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int s0 = t * kMlpTile;
    mlp_load_inputs(x, nullptr, s0, n, S.dim[0], s_a[0]);
    __syncthreads();
#pragma unroll
    for (int l = 0; l < kMlpMaxLayers; ++l) {
      if (l >= S.n_layers) break;
      const int di = S.dim[l], dout = S.dim[l + 1];
      float *next = s_a[(l + 1) & 1];
      if (16 * wave < dout) {
        Frag a;
        a.load(s_a[l & 1] + m * kMlpRow, di);
        const f32x4 z = mlp_product(a, W.w[l], di);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = z[r] + W.bias[l];
          if (l == S.n_layers - 1) {
            const int s = s0 + 4 * q + r;
            if (col == 0 && s < n) y[s] = base[s] + v;
          } else {
            next[(4 * q + r) * kMlpRow + mlp_slot(col)] = round_bf16(v > 0.f ? v : 0.f);
          }
        }
      }
      __syncthreads();
    }
  }
}

// Forward and backward of the workgroup's samples (sample s reads row idx[s]
// of x, base and t, row s when idx is null): dL/dy = 2 (y - t) / n; the
// gradient partials of its two groups of 8 samples go to slab[group][param],
// the loss partials too.  Layer inputs and deltas of all layers stay in LDS
// for the weight gradients, pre-activations in registers.
__global__ __launch_bounds__(kMlpThreads) void mlp_step_kernel(
    MlpShape S, const float *__restrict__ img, const float *__restrict__ x,
    const float *__restrict__ base, const float *__restrict__ t,
    const int32_t *__restrict__ idx, int32_t n, int32_t parts, float *__restrict__ slab,
    float *__restrict__ loss_part) {
  extern __shared__ __align__(16) float lds[];   // [layer][sample][kMlpRow] twice
  __shared__ float s_r2[kMlpTile];
  constexpr int kLayer = kMlpTile * kMlpRow;
  float *ars = lds, *dzs = lds + S.n_layers * kLayer;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int m = lane & 15, q = lane >> 4, col = 16 * wave + m;
  const int s0 = blockIdx.x * kMlpTile;
  // the samples whose results a lane gets, for the last layer
  size_t row[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int s = min(s0 + 4 * q + r, n - 1);
    row[r] = idx ? (size_t)idx[s] : (size_t)s;
  }
  MlpWeights W;
  W.load(S, img);
  Frag wt[kMlpMaxLayers];
#pragma unroll
  for (int l = 1; l < kMlpMaxLayers; ++l) {
    if (l >= S.n_layers) break;
    wt[l].load(img + (size_t)(S.n_layers + l) * kMlpImage + col * kMlpMaxDim,
               16 * wave < S.dim[l] ? S.dim[l + 1] : 0);
  }
  float y0[4], target[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    y0[r] = base[row[r]];
    target[r] = t[row[r]];
  }
  mlp_load_inputs(x, idx, s0, n, S.dim[0], ars);
  __syncthreads();

  f32x4 z[kMlpMaxLayers];
#pragma unroll
  for (int l = 0; l < kMlpMaxLayers; ++l) {
    if (l >= S.n_layers) break;
    const int di = S.dim[l], dout = S.dim[l + 1];
    const bool last = l == S.n_layers - 1;
    z[l] = f32x4{0, 0, 0, 0};
    if (16 * wave < dout) {
      Frag a;
      a.load(ars + l * kLayer + m * kMlpRow, di);
      z[l] = mlp_product(a, W.w[l], di);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool valid = s0 + 4 * q + r < n;
        const float v = z[l][r] + W.bias[l];
        z[l][r] = valid ? v : 0.f;
        if (last) {
          const float res = valid ? y0[r] + v - target[r] : 0.f;
          const float g = valid ? 2.f * res / (float)n : 0.f;
          // (zeros in the other columns: the products take 16 outputs)
          dzs[l * kLayer + (4 * q + r) * kMlpRow + mlp_slot(col)] = col ? 0.f : g;
          if (col == 0) s_r2[4 * q + r] = res * res;
        } else {
          ars[(l + 1) * kLayer + (4 * q + r) * kMlpRow + mlp_slot(col)] =
              valid ? round_bf16(v > 0.f ? v : 0.f) : 0.f;
        }
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < 2 && 2 * blockIdx.x + threadIdx.x < parts) {
    const float *r2 = s_r2 + kMlpPart * threadIdx.x;
    loss_part[2 * blockIdx.x + threadIdx.x] =
        ((r2[0] + r2[4]) + (r2[2] + r2[6])) + ((r2[1] + r2[5]) + (r2[3] + r2[7]));
  }
  // deltas of the layers below: through the weights, where the
  // pre-activation was positive
#pragma unroll
  for (int l = kMlpMaxLayers - 1; l > 0; --l) {
    if (l >= S.n_layers) continue;
    const int di = S.dim[l], dout = S.dim[l + 1];
    if (16 * wave < di) {
      Frag a;
      a.load(dzs + l * kLayer + m * kMlpRow, dout);
      const f32x4 d = mlp_product(a, wt[l], dout);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        dzs[(l - 1) * kLayer + (4 * q + r) * kMlpRow + mlp_slot(col)] =
            z[l - 1][r] > 0.f ? d[r] : 0.f;
    }
    __syncthreads();
  }
  // dW[o][i] = sum_s dz[s][o] a[s][i]: a wave takes 16 rows o, every 16
  // columns i, the two groups of 8 samples apart; db[o] = sum_s dz[s][o].
  // Buffer stores: a lane offset past the end (rows and columns the layer
  // does not have, a group past the last) writes nothing, with no branch.
  // (The scalar offset, 64 c, is below the parameters' bytes wherever it is
  // used: a layer then has more than 16 c inputs.)
  const bool two = 2 * (int)blockIdx.x + 1 < parts;
  float *part0 = slab + (size_t)2 * blockIdx.x * S.n_params;
  __amdgpu_buffer_rsrc_t part[2];
#pragma unroll
  for (int g = 0; g < 2; ++g)
    part[g] = __builtin_amdgcn_make_buffer_rsrc(part0 + (size_t)g * S.n_params, 0,
                                                S.n_params * 4, 0x00027000);
  constexpr int kPast = 0x7FFFFFFF;
#pragma unroll
  for (int l = 0; l < kMlpMaxLayers; ++l) {
    if (l >= S.n_layers) break;
    const int di = S.dim[l], dout = S.dim[l + 1];
    if (16 * wave >= dout) continue;
    // sample 4 u + q, u = 0, 1: the first group; 2, 3: the second
    const float *dz = dzs + l * kLayer + q * kMlpRow + mlp_slot(col);
    const float *ar = ars + l * kLayer + q * kMlpRow + mlp_slot(m);
    float da[4], av[4][4], dbs[kMlpPart];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      da[u] = dz[4 * u * kMlpRow];
      // mlp_slot(16 c + m) = mlp_slot(m) + 4 c
#pragma unroll
      for (int c = 0; c < 4; ++c) av[c][u] = ar[4 * u * kMlpRow + 4 * c];
    }
    // the bias of column `col`: lanes q = 0, 1 take a group each
#pragma unroll
    for (int k = 0; k < kMlpPart; ++k)
      dbs[k] = dzs[l * kLayer + (kMlpPart * (q & 1) + k) * kMlpRow + mlp_slot(col)];
    int off[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int o = 16 * wave + 4 * q + r;
      off[r] = o < dout ? (S.woff[l] + o * di + m) * 4 : kPast;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (16 * c >= di) break;
      const bool in = 16 * c + m < di;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        f32x4 d = {0, 0, 0, 0};
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(da[2 * g], av[c][2 * g], d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(da[2 * g + 1], av[c][2 * g + 1], d, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(d[r]), part[g],
                                                in && (g == 0 || two) ? off[r] : kPast,
                                                64 * c, 0);
      }
    }
    float db = 0.f;
#pragma unroll
    for (int k = 0; k < kMlpPart; ++k) db += dbs[k];
    const int boff = col < dout ? (S.boff[l] + col) * 4 : kPast;
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(db), part[0], q == 0 ? boff : kPast, 0, 0);
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(db), part[1],
                                          q == 1 && two ? boff : kPast, 0, 0);
  }
}

// Gradient = sum of the workgroups' partials (in workgroup order, 32
// partials' loads in flight per lane), then, when `adam`, the Adam update
// of the same parameter (fp32 master, moments, weight images: places `at`,
// the second one -1 for biases).  The last workgroup sums the loss partials.
constexpr int kAdamThreads = 64;

// a parameter's places in the images: weights rounded to bfloat16, both ways
// round; biases as they are
__device__ __forceinline__ void mlp_to_images(float p, int2 at, float *__restrict__ img) {
  if (at.y >= 0) {
    const float w = round_bf16(p);
    img[at.x] = w;
    img[at.y] = w;
  } else {
    img[at.x] = p;
  }
}

__global__ __launch_bounds__(kAdamThreads) void mlp_reduce_adam_kernel(
    const float *__restrict__ slab, int32_t parts, int32_t n_params,
    float *__restrict__ g, const float *__restrict__ loss_part,
    float *__restrict__ loss, float inv_n, int32_t adam, float *__restrict__ p,
    float *__restrict__ m, float *__restrict__ v, float *__restrict__ img,
    const int2 *__restrict__ at, float lr, float b1, float b2, float eps, float c1, float c2) {
  if (blockIdx.x == gridDim.x - 1) {
    if (!loss) return;
    float acc = 0.f;
    for (int b0 = 0; b0 < parts; b0 += kAdamThreads) {
      const int b = b0 + (int)threadIdx.x;
      const float q = b < parts ? loss_part[b] : 0.f;
      for (int u = 0; u < min(kAdamThreads, parts - b0); ++u) acc += lane_value(q, u);
    }
    if (threadIdx.x == 0) *loss = acc * inv_n;  // mean squared error
    return;
  }
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_params) return;
  constexpr int kU = 32;
  float acc = 0.f;
  for (int b0 = 0; b0 < parts; b0 += kU) {
    float t[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u)
      t[u] = b0 + u < parts ? slab[(size_t)(b0 + u) * n_params + k] : 0.f;
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (b0 + u < parts) acc += t[u];
  }
  g[k] = acc;
  if (!adam) return;
  const float mk = b1 * m[k] + (1.f - b1) * acc;
  const float vk = b2 * v[k] + (1.f - b2) * acc * acc;
  m[k] = mk;
  v[k] = vk;
  const float pk = p[k] - lr * (mk / c1) / (sqrtf(vk / c2) + eps);
  p[k] = pk;
  mlp_to_images(pk, at[k], img);
}

__global__ void mlp_images_kernel(const float *__restrict__ p, const int2 *__restrict__ at,
                                  float *__restrict__ img, int32_t n) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) mlp_to_images(p[k], at[k], img);
}

// The query's join graph in kernel arguments (edge endpoints).
struct FeatGraph {
  int32_t n_edges;
  uint8_t u[64], v[64];
};

// Shape of the sub-plan `m` (its tables and the edges between them):
// number of tables, number of edges, diameter (longest shortest path, in
// edges), largest degree, independent cycles (edges - tables + 1).
__device__ void subplan_shape(const FeatGraph &g, uint64_t m, float out[5]) {
  int ne = 0;
  int deg_max = 0;
  const int nt = __popcll(m);
  for (int e = 0; e < g.n_edges; ++e)
    ne += ((m >> g.u[e]) & (m >> g.v[e]) & 1ull) ? 1 : 0;
  int diam = 0;
  for (uint64_t rest = m; rest; rest &= rest - 1) {
    const int t = __ffsll((long long)rest) - 1;
    int deg = 0;
    for (int e = 0; e < g.n_edges; ++e)
      if ((m >> g.u[e]) & (m >> g.v[e]) & 1ull)
        deg += (g.u[e] == t) + (g.v[e] == t);
    deg_max = deg > deg_max ? deg : deg_max;
    // breadth-first levels from t over the sub-plan's edges
    uint64_t seen = 1ull << t, frontier = seen;
    int depth = 0;
    while (true) {
      uint64_t next = 0;
      for (int e = 0; e < g.n_edges; ++e) {
        if (!((m >> g.u[e]) & (m >> g.v[e]) & 1ull)) continue;
        if ((frontier >> g.u[e]) & 1ull) next |= 1ull << g.v[e];
        if ((frontier >> g.v[e]) & 1ull) next |= 1ull << g.u[e];
      }
      next &= ~seen;
      if (!next) break;
      seen |= next;
      frontier = next;
      ++depth;
    }
    diam = depth > diam ? depth : diam;
  }
  out[0] = (float)nt;
  out[1] = (float)ne;
  out[2] = (float)diam;
  out[3] = (float)deg_max;
  out[4] = (float)(ne - nt + 1);
}

// Sub-plan features: 7 order statistics (positions round(k (d-1) / 6)) of
// slog(X_i) = sign * ln(1 + |X_i|) over the sorted row estimates; log2(1 +
// n_sel) of the sub-plan's tables, descending, first 8, zero padded; the 5
// shape statistics of subplan_shape.  base = ln(1 + max(est, 0)).
__global__ void mlp_features_kernel(const u128 *__restrict__ rows, int32_t d,
                                    const double *__restrict__ est,
                                    const uint64_t *__restrict__ masks,
                                    const int64_t *__restrict__ n_sel,
                                    int32_t n_tables, FeatGraph g,
                                    int32_t n, float *__restrict__ x,
                                    float *__restrict__ base) {
  const int sp = blockIdx.x * blockDim.x + threadIdx.x;
  if (sp >= n) return;
  double v[32];
  for (int i = 0; i < d; ++i) {
    const double r = i128_to_double(rows[(size_t)sp * d + i]);
    v[i] = r;
  }
  for (int a = 1; a < d; ++a) {  // sort ascending (by the exact doubles)
    const double t = v[a];
    int b = a - 1;
    while (b >= 0 && v[b] > t) {
      v[b + 1] = v[b];
      --b;
    }
    v[b + 1] = t;
  }
  float *xo = x + (size_t)sp * 20;
  for (int k = 0; k < 7; ++k) {
    const int pos = (int)((k * (d - 1) + 3) / 6);  // round(k (d-1) / 6)
    const double r = v[pos];
    const double s = r < 0 ? -log1p(-r) : log1p(r);
    xo[k] = (float)s;
  }
  double ls[64];
  int cnt = 0;
  const uint64_t m = masks[sp];
  for (int t = 0; t < n_tables; ++t)
    if ((m >> t) & 1ull) ls[cnt++] = log2(1.0 + (double)n_sel[t]);
  for (int k = 0; k < 8 && k < cnt; ++k) {  // 8 largest, descending
    int best = k;
    for (int j = k + 1; j < cnt; ++j)
      if (ls[j] > ls[best]) best = j;
    const double tmp = ls[k];
    ls[k] = ls[best];
    ls[best] = tmp;
  }
  for (int k = 0; k < 8; ++k) xo[7 + k] = k < cnt ? (float)ls[k] : 0.f;
  float sh[5];
  subplan_shape(g, m, sh);
  for (int k = 0; k < 5; ++k) xo[15 + k] = sh[k];
  const double e = est[sp];
  base[sp] = (float)log1p(e > 0 ? e : 0.0);
}

}  // namespace compass

using namespace compass;

namespace compass {
void set_last_error(const std::string &s);
}

static compass_status mfail(compass_status s, const std::string &m) {
  compass::set_last_error(m);
  return s;
}

#define MHIP(expr)                                                        \
  do {                                                                    \
    hipError_t e_ = (expr);                                               \
    if (e_ != hipSuccess)                                                 \
      return mfail(COMPASS_E_HIP,                                         \
                   std::string(#expr) + ": " + hipGetErrorString(e_));    \
  } while (0)

struct compass_mlp_s {
  MlpShape S;
  float *p = nullptr, *m = nullptr, *v = nullptr, *g = nullptr;
  float *img = nullptr;   // weight images (kMlpImage)
  int2 *at = nullptr;     // every parameter's places in them
  float *slab = nullptr, *loss_part = nullptr;
  int32_t cap = 0;     // samples the training buffers hold
  int64_t step = 0;
};

extern "C" compass_status compass_mlp_create(int32_t n_in, int32_t hidden,
                                             int32_t n_hidden_layers,
                                             const float *init,
                                             compass_mlp *out) {
  if (!out || !init) return mfail(COMPASS_E_ARG, "null pointer argument");
  if (n_in < 1 || n_in > kMlpMaxDim || hidden < 1 || hidden > kMlpMaxDim ||
      n_hidden_layers < 1 || n_hidden_layers + 1 > kMlpMaxLayers)
    return mfail(COMPASS_E_ARG, "MLP shape outside [1, 64] x [1, 7] layers");
  compass_mlp_s *M = new compass_mlp_s();
  MlpShape &S = M->S;
  memset(&S, 0, sizeof S);
  S.n_layers = n_hidden_layers + 1;
  S.dim[0] = n_in;
  for (int l = 1; l <= n_hidden_layers; ++l) S.dim[l] = hidden;
  S.dim[S.n_layers] = 1;
  int off = 0;
  for (int l = 0; l < S.n_layers; ++l) {
    S.woff[l] = off;
    off += S.dim[l] * S.dim[l + 1];
    S.boff[l] = off;
    off += S.dim[l + 1];
  }
  S.n_params = off;
  const size_t b = sizeof(float) * off;
  const size_t img_words = (size_t)S.n_layers * (2 * kMlpImage + kMlpMaxDim);
  auto bad = [&](hipError_t e) {
    if (e != hipSuccess) {
      delete M;
      return true;
    }
    return false;
  };
  if (bad(hipMalloc(&M->p, b)) || bad(hipMalloc(&M->m, b)) ||
      bad(hipMalloc(&M->v, b)) || bad(hipMalloc(&M->g, b)) ||
      bad(hipMalloc(&M->img, sizeof(float) * img_words)) ||
      bad(hipMalloc(&M->at, sizeof(int2) * off)))
    return mfail(COMPASS_E_HIP, "hipMalloc failed");
  std::vector<int2> at(off);
  for (int l = 0; l < S.n_layers; ++l) {
    const int di = S.dim[l], dout = S.dim[l + 1];
    for (int o = 0; o < dout; ++o) {
      for (int i = 0; i < di; ++i)
        at[S.woff[l] + o * di + i] =
            make_int2(l * kMlpImage + o * kMlpMaxDim + mlp_slot(i),
                      (S.n_layers + l) * kMlpImage + i * kMlpMaxDim + mlp_slot(o));
      at[S.boff[l] + o] = make_int2(2 * S.n_layers * kMlpImage + l * kMlpMaxDim + o, -1);
    }
  }
  MHIP(hipMemcpy(M->at, at.data(), sizeof(int2) * off, hipMemcpyHostToDevice));
  MHIP(hipMemset(M->img, 0, sizeof(float) * img_words));
  MHIP(hipMemcpy(M->p, init, b, hipMemcpyHostToDevice));
  MHIP(hipMemset(M->m, 0, b));
  MHIP(hipMemset(M->v, 0, b));
  MHIP(hipMemset(M->g, 0, b));
  hipLaunchKernelGGL(mlp_images_kernel, dim3((off + 255) / 256), dim3(256), 0,
                     0, M->p, M->at, M->img, off);
  MHIP(hipGetLastError());
  MHIP(hipDeviceSynchronize());
  *out = M;
  return COMPASS_OK;
}

extern "C" int64_t compass_mlp_n_params(compass_mlp M) {
  return M ? M->S.n_params : 0;
}

extern "C" int64_t compass_mlp_adam_steps(compass_mlp M) {
  return M ? (int64_t)M->step : 0;
}

extern "C" compass_status compass_mlp_forward(compass_mlp M, const float *x,
                                              const float *base, int32_t n,
                                              float *y, hipStream_t st) {
  if (!M || (n > 0 && (!x || !base || !y)) || n < 0)
    return mfail(COMPASS_E_ARG, "bad argument");
  if (n == 0) return COMPASS_OK;
  const int64_t tiles = ((int64_t)n + kMlpTile - 1) / kMlpTile;
  hipLaunchKernelGGL(mlp_fwd_kernel, dim3((unsigned)std::min<int64_t>(tiles, 1024)),
                     dim3(kMlpThreads), 0, st, M->S, M->img, x, base, n, y);
  MHIP(hipGetLastError());
  return COMPASS_OK;
}

// One Adam step on samples idx[0..n) of (x, base, target) (rows 0..n when
// idx is null); grows the gradient slab when n exceeds it.
static compass_status train_batch(compass_mlp M, const float *x,
                                  const float *base, const float *target,
                                  const int32_t *idx, int32_t n, float lr,
                                  float *loss, hipStream_t st) {
  const int parts = (n + kMlpPart - 1) / kMlpPart;
  if (n > M->cap) {
    (void)hipDeviceSynchronize();
    (void)hipFree(M->slab);
    (void)hipFree(M->loss_part);
    M->slab = M->loss_part = nullptr;
    M->cap = 0;
    MHIP(hipMalloc(&M->slab, (size_t)parts * M->S.n_params * sizeof(float)));
    MHIP(hipMalloc(&M->loss_part, (size_t)parts * sizeof(float)));
    M->cap = n;
  }
  const size_t lds = 2 * (size_t)M->S.n_layers * kMlpTile * kMlpRow * sizeof(float);
  hipLaunchKernelGGL(mlp_step_kernel, dim3((n + kMlpTile - 1) / kMlpTile),
                     dim3(kMlpThreads), lds, st, M->S, M->img, x, base, target, idx, n,
                     parts, M->slab, M->loss_part);
  const int np = M->S.n_params;
  if (lr > 0.f) M->step += 1;  // a gradient-only call is not an Adam step
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - powf(b1, (float)M->step);
  const float c2 = 1.f - powf(b2, (float)M->step);
  hipLaunchKernelGGL(mlp_reduce_adam_kernel,
                     dim3((np + kAdamThreads - 1) / kAdamThreads + 1), dim3(kAdamThreads),
                     0, st, M->slab, parts, np, M->g, M->loss_part, loss,
                     1.f / (float)n, lr > 0.f ? 1 : 0, M->p, M->m, M->v, M->img,
                     M->at, lr, b1, b2, 1e-8f, c1, c2);
  MHIP(hipGetLastError());
  return COMPASS_OK;
}

extern "C" compass_status compass_mlp_train_step(compass_mlp M, const float *x,
                                                 const float *base,
                                                 const float *target, int32_t n,
                                                 float lr, float *loss,
                                                 hipStream_t st) {
  if (!M || !x || !base || !target || n < 1)
    return mfail(COMPASS_E_ARG, "bad argument");
  return train_batch(M, x, base, target, nullptr, n, lr, loss, st);
}

extern "C" compass_status compass_mlp_train_epoch(
    compass_mlp M, const float *x, const float *base, const float *target,
    const int32_t *idx, int32_t n_batches, int32_t batch, float lr,
    float *losses, hipStream_t st) {
  if (!M || !x || !base || !target || !idx || !losses || n_batches < 0 ||
      batch < 1 || lr <= 0.f)
    return mfail(COMPASS_E_ARG, "bad argument");
  for (int32_t k = 0; k < n_batches; ++k) {
    const compass_status s = train_batch(M, x, base, target,
                                         idx + (int64_t)k * batch, batch, lr,
                                         losses + k, st);
    if (s != COMPASS_OK) return s;
  }
  return COMPASS_OK;
}

// what: 0 parameters, 1 last gradients, 2 Adam first moments, 3 second
extern "C" compass_status compass_mlp_read(compass_mlp M, int32_t what,
                                           float *host_out) {
  if (!M || !host_out || what < 0 || what > 3)
    return mfail(COMPASS_E_ARG, "bad argument");
  const float *src = what == 0 ? M->p : what == 1 ? M->g : what == 2 ? M->m : M->v;
  MHIP(hipDeviceSynchronize());
  MHIP(hipMemcpy(host_out, src, sizeof(float) * M->S.n_params,
                 hipMemcpyDeviceToHost));
  return COMPASS_OK;
}

extern "C" compass_status compass_mlp_write(compass_mlp M, const float *params,
                                            const float *adam_m,
                                            const float *adam_v, int64_t step) {
  if (!M || !params) return mfail(COMPASS_E_ARG, "bad argument");
  const size_t b = sizeof(float) * M->S.n_params;
  MHIP(hipDeviceSynchronize());
  MHIP(hipMemcpy(M->p, params, b, hipMemcpyHostToDevice));
  if (adam_m) MHIP(hipMemcpy(M->m, adam_m, b, hipMemcpyHostToDevice));
  if (adam_v) MHIP(hipMemcpy(M->v, adam_v, b, hipMemcpyHostToDevice));
  M->step = step;
  hipLaunchKernelGGL(mlp_images_kernel, dim3((M->S.n_params + 255) / 256),
                     dim3(256), 0, 0, M->p, M->at, M->img, M->S.n_params);
  MHIP(hipGetLastError());
  MHIP(hipDeviceSynchronize());
  return COMPASS_OK;
}

extern "C" compass_status compass_mlp_destroy(compass_mlp M) {
  if (!M) return COMPASS_OK;
  (void)hipDeviceSynchronize();
  (void)hipFree(M->p);
  (void)hipFree(M->m);
  (void)hipFree(M->v);
  (void)hipFree(M->g);
  (void)hipFree(M->img);
  (void)hipFree(M->at);
  (void)hipFree(M->slab);
  (void)hipFree(M->loss_part);
  delete M;
  return COMPASS_OK;
}

extern "C" compass_status compass_mlp_features(
    const compass_i128 *row_est, int32_t d, const double *est,
    const uint64_t *masks, const int64_t *n_selected, int32_t n_tables,
    int32_t n_edges, const int32_t *edge_u, const int32_t *edge_v, int32_t n,
    float *x, float *base, hipStream_t st) {
  if (n < 0 || d < 1 || d > 32 || n_tables < 1 || n_tables > 64 ||
      n_edges < 0 || n_edges > 64)
    return mfail(COMPASS_E_ARG, "bad feature arguments");
  if (n_edges > 0 && (!edge_u || !edge_v))
    return mfail(COMPASS_E_ARG, "null edge array");
  FeatGraph g;
  memset(&g, 0, sizeof g);
  g.n_edges = n_edges;
  for (int e = 0; e < n_edges; ++e) {
    if (edge_u[e] < 0 || edge_u[e] >= n_tables || edge_v[e] < 0 ||
        edge_v[e] >= n_tables || edge_u[e] == edge_v[e])
      return mfail(COMPASS_E_GRAPH, "edge with bad endpoints");
    g.u[e] = (uint8_t)edge_u[e];
    g.v[e] = (uint8_t)edge_v[e];
  }
  if (n == 0) return COMPASS_OK;
  if (!row_est || !est || !masks || !n_selected || !x || !base)
    return mfail(COMPASS_E_ARG, "null pointer argument");
  hipLaunchKernelGGL(mlp_features_kernel, dim3((n + 127) / 128), dim3(128), 0, st,
                     reinterpret_cast<const u128 *>(row_est), d, est, masks,
                     n_selected, n_tables, g, n, x, base);
  MHIP(hipGetLastError());
  return COMPASS_OK;
}
