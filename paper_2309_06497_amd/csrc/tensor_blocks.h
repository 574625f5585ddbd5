// Blocks of tensor parameters (Sec. 2.3 of the paper: Shampoo for a tensor of order w keeps one
// factor per dimension and preconditions by mode products; Sec. 4.2.1: merging and blocking).
//
// A block d1 x d2 x d3 (x d4) of a D1 x D2 x D3 (x D4) parameter is strided two or three times
// inside the caller's tensor.  The step therefore works on a block-contiguous copy of the gradient and of the
// parameter (blocks back to back, in row-major order of their block indices), in which
//   * the unfolding along the first dimension is the plain d1 x (d2 d3 ...) matrix,
//   * the unfolding along the last dimension is the plain (d1 d2 ...) x d_last matrix read
//     "rows along k",
//   * the unfolding along a middle dimension k becomes plain once the block, seen as
//     pre x d_k x post, has its first two indices swapped (permute_12_kernel): d_k x (pre post),
// so every factor update and mode product is one of the batched SYRK / GEMM launches of the
// matrix case, and the elementwise kernels see the block as a d1 x (d2 d3) matrix.  The kernels
// here only move data: gather / scatter between the caller's tensor and the copy, and the swap.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "gemm_mfma.h"
#include "group.h"

namespace shampoo {

struct TensorCopyArgs {
  void *tensor;            // the caller's D1 x D2 x D3 x D4 tensor (row-major)
  void *copy;              // the block-contiguous copy
  int64_t D1, D2, D3, D4;  // unused trailing dimensions are 1
  int32_t b;               // block size
  int32_t k2n, k3n, k4n;   // pieces along the second, third and fourth dimension
  int32_t bytes;           // of an element: 4, or 2 (bf16 gradients)
  int32_t first, chunks;   // first workgroup of this tensor; workgroups per block
};
// The tensors of one launch.  A network has dozens of small ones, each worth a few microseconds: one
// launch per 40 of them and direction (that is what fits a kernel's 4 KB of arguments) instead of three
// per tensor, and 32-bit index arithmetic (a block has less than 2^31 elements).  ResNet-50 shapes, 17
// tensors of 11e6 elements in all: 485 -> 96 us a step.
constexpr int TENSOR_COPY_SET = 40;
struct TensorCopySet { TensorCopyArgs t[TENSOR_COPY_SET]; int32_t count; };
static_assert(sizeof(TensorCopySet) <= 4096, "kernel arguments");

constexpr int COPY_U = 4;
// Block index = ((k1 * k2n + k2) * k3n + k3) * k4n + k4.  All pieces before the last one of a
// dimension are full, so the offset of a block inside the copy is
// s1 D2 D3 D4 + d1 s2 D3 D4 + d1 d2 s3 D4 + d1 d2 d3 s4.
template <typename T, bool SCATTER>
__device__ __forceinline__ void tensor_copy(const TensorCopyArgs &g, uint32_t wg) {
  uint32_t blk = wg / (uint32_t)g.chunks;
  const uint32_t chunk = wg - blk * (uint32_t)g.chunks;
  const uint32_t k4 = blk % (uint32_t)g.k4n; blk /= (uint32_t)g.k4n;
  const uint32_t k3 = blk % (uint32_t)g.k3n; blk /= (uint32_t)g.k3n;
  const uint32_t k2 = blk % (uint32_t)g.k2n, k1 = blk / (uint32_t)g.k2n;
  const int64_t s1 = (int64_t)k1 * g.b, s2 = (int64_t)k2 * g.b, s3 = (int64_t)k3 * g.b, s4 = (int64_t)k4 * g.b;
  const int64_t d1 = min((int64_t)g.b, g.D1 - s1), d2 = min((int64_t)g.b, g.D2 - s2), d3 = min((int64_t)g.b, g.D3 - s3),
                d4 = min((int64_t)g.b, g.D4 - s4);
  const int64_t voff = s1 * g.D2 * g.D3 * g.D4 + d1 * (s2 * g.D3 * g.D4) + d1 * d2 * (s3 * g.D4) + d1 * d2 * d3 * s4;
  T *tensor = static_cast<T *>(g.tensor) + ((s1 * g.D2 + s2) * g.D3 + s3) * g.D4 + s4;
  T *copy = static_cast<T *>(g.copy) + voff;
  const uint32_t e4 = (uint32_t)d4, e3 = (uint32_t)d3, e2 = (uint32_t)d2, n = (uint32_t)(d1 * d2 * d3 * d4);
  const int64_t l3 = g.D4, l2 = g.D3 * l3, l1 = g.D2 * l2;
  const uint32_t step = (uint32_t)g.chunks * 256;
  for (uint32_t e0 = chunk * 256 + threadIdx.x; e0 < n; e0 += COPY_U * step) {     // several loads in flight
    int64_t at[COPY_U];
    T v[COPY_U];
#pragma unroll
    for (int u = 0; u < COPY_U; ++u) {
      const uint32_t e = min(e0 + u * step, n - 1);
      const uint32_t q4 = e / e4, i4 = e - q4 * e4, q3 = q4 / e3, i3 = q4 - q3 * e3, i1 = q3 / e2, i2 = q3 - i1 * e2;
      at[u] = i1 * l1 + i2 * l2 + i3 * l3 + i4;
      v[u] = SCATTER ? copy[e] : tensor[at[u]];
    }
#pragma unroll
    for (int u = 0; u < COPY_U; ++u) {
      const uint32_t e = e0 + u * step;
      if (e >= n) continue;
      if (SCATTER) tensor[at[u]] = v[u];
      else copy[e] = v[u];
    }
  }
}
template <bool SCATTER>
__global__ __launch_bounds__(256) void tensor_block_copy_kernel(const TensorCopySet g) {
  int i = 0;
  while (i + 1 < g.count && g.t[i + 1].first <= (int)blockIdx.x) ++i;
  const TensorCopyArgs &t = g.t[i];
  const uint32_t wg = blockIdx.x - t.first;
  if (t.bytes == 4) tensor_copy<uint32_t, SCATTER>(t, wg);
  else tensor_copy<uint16_t, SCATTER>(t, wg);
}

struct PermuteArgs {
  const BlockDesc *desc;        // input through the pointer table (blocks of the copy) ...
  const void *const *table;
  const float *src;             // ... or a dense float32 array [slot][d1][d2][d3]
  float *dst;                   // [slot][d2][d1][d3]
  int32_t d1, d2, d3;
  int32_t chunks, blocks;       // workgroups per block
  int32_t t1, t2, stride;       // tile of i1 and i2 that goes through LDS and its row there; t1 = 0: none
  __device__ __forceinline__ void globals() { to_global(desc, table, src, dst); }
};
constexpr int PERMUTE_TILE = 4608, PERMUTE_LDS = PERMUTE_TILE + 32 * 63;
// The tile of a swap, and its workgroups; `chunks` of them where there is none.  Runs of t2 d3 elements are read and runs of t1 d3
// written; with more than 72 values of i3 the runs as they lie are long enough.  A row's place in LDS is d3 behind the one before modulo
// the 64 banks, so that a run's elements, one from each row in turn, lie in different ones.
inline void permute_shape(PermuteArgs &g, int chunks) {
  g.chunks = chunks; g.t1 = 0; g.t2 = 1; g.stride = 0;
  if (g.d3 > 72) return;
  g.t1 = 32; g.t2 = 16;
  while (g.t1 * g.t2 * g.d3 > PERMUTE_TILE) { if (g.t1 > g.t2) g.t1 /= 2; else g.t2 /= 2; }
  g.stride = g.t2 * g.d3 + ((g.d3 - g.t2 * g.d3) & 63);
  g.chunks = (g.d1 + g.t1 - 1) / g.t1 * ((g.d2 + g.t2 - 1) / g.t2);
}

// dst[slot][i2][i1][i3] = in[slot][i1][i2][i3].  Workgroups: chunks x blocks.  Bound by memory.  Element by element, the 36-byte pieces of a
// 3 x 3 convolution's blocks went to memory by parts of lines: the swaps of ResNet-50's blocks (most of them 128 x 128 x 9, 90 MB
// read and written) took 95 us, 22 through LDS.  Shorter rows of i3, whose tiles leave places empty, lose nothing: steps of 32 blocks of
// 128 x 128 x 2 147 and 143 us, x 3 159 and 154, x 4 165 and 162, x 7 203 and 199.
template <typename T>
__global__ __launch_bounds__(256) void permute_12_kernel(const Group<PermuteArgs> grp) {
  __shared__ float tile[PERMUTE_LDS];
  int wg;
  const PermuteArgs g = group_pick(grp, wg);
  const int slot = wg / g.chunks, chunk = wg - slot * g.chunks;
  if (slot >= g.blocks) return;
  const uint32_t n = (uint32_t)g.d1 * g.d2 * g.d3;
  const T *tin = nullptr;
  if (!g.src) {
    const BlockDesc d = g.desc[slot];
    tin = global_ptr<const T>(g.table[d.param]) + d.offset;
  }
  const float *fin = g.src ? g.src + (int64_t)slot * n : nullptr;
  float *out = g.dst + (int64_t)slot * n;
  const uint32_t d1 = g.d1, d2 = g.d2, d3 = g.d3;   // 32-bit divisions: a block has less than 2^31 elements
  if (g.t1 > 0) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tiles2 = (g.d2 + g.t2 - 1) / g.t2, a = chunk / tiles2, i1 = a * g.t1, i2 = (chunk - a * tiles2) * g.t2;
    const int n1 = min(g.t1, g.d1 - i1), n2 = min(g.t2, g.d2 - i2), run = n2 * g.d3, pieces = (run + 63) / 64;
    const uint32_t over = (65536 + pieces - 1) / pieces, over_d = (65536 + d3 - 1) / d3;   // quotients below 2^16 / divisor
    const int64_t first = ((int64_t)i1 * g.d2 + i2) * g.d3, step = (int64_t)g.d2 * g.d3;
    for (int q0 = wave; q0 < n1 * pieces; q0 += 4 * 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {                  // eight loads in flight
        const int q = min(q0 + 4 * u, n1 * pieces - 1), r1 = (int)((uint32_t)q * over >> 16), x = min((q - r1 * pieces) * 64 + lane, run - 1);
        v[u] = fin ? fin[first + r1 * step + x] : Elem<T>::load1(tin + first + r1 * step + x);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int q = q0 + 4 * u, r1 = (int)((uint32_t)q * over >> 16), x = (q - r1 * pieces) * 64 + lane;
        if (q < n1 * pieces && x < run) tile[r1 * g.stride + x] = v[u];
      }
    }
    __syncthreads();
    for (int r2 = wave; r2 < n2; r2 += 4) {
      float *to = out + ((int64_t)(i2 + r2) * g.d1 + i1) * g.d3;
#pragma unroll 4
      for (int y = lane; y < n1 * g.d3; y += 64) {
        const int r1 = (int)((uint32_t)y * over_d >> 16);
        to[y] = tile[r1 * g.stride + r2 * g.d3 + y - r1 * g.d3];
      }
    }
    return;
  }
  const uint32_t step = g.chunks * 256;
  for (uint32_t e0 = chunk * 256 + threadIdx.x; e0 < n; e0 += COPY_U * step) {
    float v[COPY_U];
#pragma unroll
    for (int u = 0; u < COPY_U; ++u) {
      const uint32_t e = min(e0 + u * step, n - 1);
      v[u] = fin ? fin[e] : Elem<T>::load1(tin + e);
    }
#pragma unroll
    for (int u = 0; u < COPY_U; ++u) {
      const uint32_t e = e0 + u * step, q = e / d3, i3 = e - q * d3, i1 = q / d2, i2 = q - i1 * d2;
      if (e < n) out[(i2 * d1 + i1) * d3 + i3] = v[u];
    }
  }
}

struct NarrowProductArgs {
  const float *src;             // [slot][d2][d1][d]: the block with its two other indices swapped
  const float *root;            // [slot][d][d]
  float *dst;                   // [slot][d1][d2][d]
  float *norm_partial;          // [slot][tiles]
  const float *gmax;            // the result is divided by range_scale of the block's
  int32_t d1, d2, d, tiles2, tiles, blocks;   // tiles2: tiles along d2
  __device__ __forceinline__ void globals() { to_global(src, root, dst, norm_partial, gmax); }
};
constexpr int NARROW_MAX = 16, NARROW_T1 = 32, NARROW_T2 = 16;    // d; a workgroup's share of the other two
inline int narrow_tiles(int64_t d1, int64_t d2) { return (int)((d1 + NARROW_T1 - 1) / NARROW_T1 * ((d2 + NARROW_T2 - 1) / NARROW_T2)); }

// dst[i1][i2] = src[i2][i1] root: the last product of a tensor block with a last dimension of d <= 16, and the swap that
// takes the block back to its own order.  Plain float32 multiply-adds: with d = 9 a tile of the GEMM is 93 % padding.  Bound by memory: chunks of 32 d and
// 16 d values in and out, the exchange in LDS.  The blocks of ResNet-50 (most of them 128 x 128 x 9): 133 us for the GEMM and 34 for the swap before,
// 28 so.  d <= 4 D4.  Workgroups: tiles x blocks.
template <int D4>
__global__ __launch_bounds__(256) void product_narrow_kernel(const Group<NarrowProductArgs> grp) {
  constexpr int T1 = NARROW_T1, T2 = NARROW_T2, LD = 4 * D4 + 1;
  __shared__ float x[T1 * T2 * LD];
  __shared__ __align__(16) float root[NARROW_MAX][4 * D4];        // transposed
  __shared__ float red[4];
  int wg;
  const NarrowProductArgs g = group_pick(grp, wg);
  const int slot = wg / g.tiles, tile = wg - slot * g.tiles;
  if (slot >= g.blocks) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), d = g.d;
  const int t1 = tile / g.tiles2, i1 = t1 * T1, i2 = (tile - t1 * g.tiles2) * T2, n1 = min(T1, g.d1 - i1), n2 = min(T2, g.d2 - i2);
  const int64_t block = (int64_t)slot * g.d1 * g.d2 * d;
  const uint32_t over_d = (65536 + d - 1) / d;                    // e / d for e < 32 d <= 512
  for (int e = tid; e < d * 4 * D4; e += 256) {
    const int j = e / (4 * D4), k = e - j * (4 * D4);
    root[j][k] = k < d ? g.root[(int64_t)slot * d * d + k * d + j] : 0.f;
  }
  float in[T2 / 4][T1 * 4 * D4 / 64];                             // all loads in flight
#pragma unroll
  for (int q = 0; q < T2 / 4; ++q) {
    const int r2 = wave + 4 * q;
    const float *row = g.src + block + ((int64_t)(i2 + min(r2, n2 - 1)) * g.d1 + i1) * d;
#pragma unroll
    for (int t = 0; t < T1 * 4 * D4 / 64; ++t) in[q][t] = row[min(lane + 64 * t, n1 * d - 1)];
  }
#pragma unroll
  for (int q = 0; q < T2 / 4; ++q)
#pragma unroll
    for (int t = 0; t < T1 * 4 * D4 / 64; ++t) {
      const int e = lane + 64 * t, r1 = (int)((uint32_t)e * over_d >> 16), r2 = wave + 4 * q;
      if (e < n1 * d) x[(r1 * T2 + r2) * LD + e - r1 * d] = in[q][t];
    }
  __syncthreads();
  const float inv = 1.f / range_scale(g.gmax[slot]);
  float ss = 0.f;
#pragma unroll
  for (int q = 0; q < T1 * T2 / 256; ++q) {
    const int row = tid + 256 * q;
    if (row / T2 >= n1 || row % T2 >= n2) continue;
    float *own = x + row * LD, v[4 * D4];
#pragma unroll
    for (int k = 0; k < 4 * D4; ++k) v[k] = k < d ? own[k] : 0.f;
    for (int j = 0; j < d; ++j) {
      float s = 0.f;
#pragma unroll
      for (int k = 0; k < 4 * D4; k += 4) {
        const float4 r = *reinterpret_cast<const float4 *>(&root[j][k]);
        s = fmaf(v[k], r.x, s); s = fmaf(v[k + 1], r.y, s); s = fmaf(v[k + 2], r.z, s); s = fmaf(v[k + 3], r.w, s);
      }
      s *= inv;
      own[j] = s;
      ss = fmaf(s, s, ss);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
  if (lane == 0) red[wave] = ss;
  __syncthreads();
  if (tid == 0) g.norm_partial[(int64_t)slot * g.tiles + tile] = (red[0] + red[1]) + (red[2] + red[3]);
#pragma unroll
  for (int q = 0; q < T1 / 4; ++q) {
    const int r1 = wave + 4 * q;
    float *out = g.dst + block + ((int64_t)(i1 + r1) * g.d2 + i2) * d;
    if (r1 < n1)
      for (int e = lane; e < n2 * d; e += 64) {
        const int r2 = (int)((uint32_t)e * over_d >> 16);
        out[e] = x[(r1 * T2 + r2) * LD + e - r2 * d];
      }
  }
}

struct GramReduceArgs {
  const void *partial;    // [slot][splits][d][d]
  float *factor;          // [slot][d][d]
  int32_t d, splits, blocks;
  double alpha, beta;
  __device__ __forceinline__ void globals() { to_global(partial, factor); }
};

struct GramNarrowArgs {
  const BlockDesc *desc;        // [slot][split]: the row ranges of X
  const void *const *table;
  float *partial;               // [slot][split][d][d]
  int32_t d, rows, entries;
  __device__ __forceinline__ void globals() { to_global(desc, table, partial); }
};

// X^T X of a range of rows of a row-major matrix of d <= 16 columns, one wavefront per range: the factor of the last
// dimension of a tensor block (9 columns and 16384 rows for a 3 x 3 convolution at block size 128).  With
// v_mfma_f32_16x16x4_f32 one register of 4 rows is both operands, and 16 rows at a time are summed before they go
// into float64, as in the general SYRK kernel.  That one multiplies 128 x 128 tiles, 99 % of it padding at d = 9:
// 564 -> 25 us for the blocks of ResNet-50 (most of them 128 x 128 x 9).  Bound by the latency of the loads.  Workgroups: ceil(entries / 4), 4 wavefronts.
template <typename T>
__global__ __launch_bounds__(256) void gram_narrow_kernel(const Group<GramNarrowArgs> grp) {
  typedef float narrow_f4 __attribute__((ext_vector_type(4)));
  int wg;
  const GramNarrowArgs g = group_pick(grp, wg);
  const int entry = wg * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4, d = g.d;
  if (entry >= g.entries) return;
  const BlockDesc bd = g.desc[entry];
  const T *x = global_ptr<const T>(g.table[bd.param]) + bd.offset;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
  for (int r0 = 0; r0 < g.rows; r0 += 16) {
    float v[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int r = r0 + 4 * t + lg;
      v[t] = (li < d && r < g.rows) ? Elem<T>::load1(x + (int64_t)r * d + li) : 0.f;
    }
    narrow_f4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) s = __builtin_amdgcn_mfma_f32_16x16x4f32(v[t], v[t], s, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] += (double)s[u];
  }
  float *out = g.partial + (int64_t)entry * d * d;
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (4 * lg + u < d && li < d) out[(4 * lg + u) * d + li] = (float)acc[u];
}

// factor <- beta factor + alpha sum_s partial_s, in float64, fixed order: the Gram matrix of a split
// unfolding.  Workgroups: ceil(d d / 256) x blocks.
template <typename T>
__global__ __launch_bounds__(256) void gram_reduce_kernel(const Group<GramReduceArgs> grp) {
  int wg;
  const GramReduceArgs g = group_pick(grp, wg);
  const int dd = g.d * g.d, per = (dd + 255) / 256, slot = wg / per;
  const int e = (wg - slot * per) * 256 + threadIdx.x;
  if (slot >= g.blocks || e >= dd) return;
  const T *p = static_cast<const T *>(g.partial) + (int64_t)slot * g.splits * dd + e;
  double acc = 0.0;
  int s = 0;
  for (; s + 8 <= g.splits; s += 8) {            // eight loads in flight, summed in order
    T v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[(int64_t)(s + u) * dd];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += (double)v[u];
  }
  for (; s < g.splits; ++s) acc += (double)p[(int64_t)s * dd];
  float *f = g.factor + (int64_t)slot * dd + e;
  *f = (float)(g.beta * (double)*f + g.alpha * acc);
}

}  // namespace shampoo
