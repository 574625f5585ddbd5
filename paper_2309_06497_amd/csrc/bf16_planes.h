// Float32 matrices as three bf16 planes.
//
// x = h + l + m with h = bf16(x), l = bf16(x - h), m = x - h - l: 8 + 8 + 8 bits, exactly the 24 of a float32, and
// with its range of exponents.  So every element keeps its own relative accuracy, however far below the largest one of
// its matrix it is (fp16 planes, scaled per matrix, do not: rows of a gradient 10^-6 and 10^-8 of the largest came out
// of a factor update with errors of 1e-6 and 2e-5 of their own size, and of Lbar G Rbar with 4e-4).  The power of two s
// that the matrix is scaled by puts its largest element near 2^14: l and m then stay normal numbers down to 2^-116 of it.
//
// A product of two such values is  h m' + m h' + l l' + h l' + l h' + h h'  up to 2^-24 of it at worst (2^-28 in the
// mean), each term exact in float32.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "gemm_mfma.h"
#include "group.h"

namespace shampoo {

__device__ __forceinline__ void split3b(float x, uint16_t (&p)[3]) {
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    const __bf16 h = (__bf16)x;
    p[t] = __builtin_bit_cast(uint16_t, h);
    x -= (float)h;                       // exact
  }
}

struct BlockPlanesArgs {
  const BlockDesc *desc;
  const void *const *g_table;
  uint16_t *cols; int64_t plane_stride;  // [plane][slot][n][m]
  uint16_t *rows;                        // the same not transposed, [plane][slot][m][n] (nullptr: not wanted)
  const float *scale;                    // [slot] s
  int32_t m, n, blocks;
  __device__ __forceinline__ void globals() { to_global(desc, g_table, cols, rows, scale); }
};
// The planes of s G_block, transposed and as they lie: operands that are read along k.  Reads 4 and writes 6 (12)
// bytes per element, 16 bytes per lane on both sides; the transposition happens in LDS (rows of 65 words: the 64 lanes
// of a read hit 64 banks).  Requires m % 8 == 0, n % 8 == 0 and 16-byte aligned rows.
// Workgroups: ceil(n / 64) x ceil(m / 64) x blocks, in that order; 256 threads.
__global__ __launch_bounds__(256) void block_planes_kernel(const Group<BlockPlanesArgs> grp) {
  __shared__ float tile[64][65];
  int wg;
  const BlockPlanesArgs g = group_pick(grp, wg);
  const int gx = (g.n + 63) / 64, gy = (g.m + 63) / 64, slot = wg / (gx * gy), ty = (wg - slot * gx * gy) / gx, tx = wg % gx;
  if (slot >= g.blocks) return;
  const BlockDesc d = g.desc[slot];
  const float *src = global_ptr<const float>(g.g_table[d.param]) + d.offset;
  const int i0 = ty * 64, j0 = tx * 64, tid = threadIdx.x;
  const float sc = g.scale[slot];
  float4 v[4];
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const int i = i0 + 16 * h + (tid >> 4), j = j0 + (tid & 15) * 4;
    v[h] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < g.m && j < g.n) v[h] = *reinterpret_cast<const float4 *>(src + (int64_t)i * d.ld + j);
  }
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    float *t = &tile[16 * h + (tid >> 4)][(tid & 15) * 4];
    t[0] = v[h].x * sc; t[1] = v[h].y * sc; t[2] = v[h].z * sc; t[3] = v[h].w * sc;
  }
  __syncthreads();
  auto put = [&](uint16_t *dst, const float (&x)[8]) {
    uint32_t w[3][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint16_t a[3], b[3];
      split3b(x[2 * e], a);
      split3b(x[2 * e + 1], b);
#pragma unroll
      for (int t = 0; t < 3; ++t) w[t][e] = (uint32_t)a[t] | ((uint32_t)b[t] << 16);
    }
#pragma unroll
    for (int t = 0; t < 3; ++t) *reinterpret_cast<uint4 *>(dst + t * g.plane_stride) = make_uint4(w[t][0], w[t][1], w[t][2], w[t][3]);
  };
  const int64_t block = (int64_t)slot * g.m * g.n;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int x = tid + 256 * q, r = x >> 3, c = (x & 7) * 8;
    float t[8];
    if (j0 + r < g.n && i0 + c < g.m) {
#pragma unroll
      for (int e = 0; e < 8; ++e) t[e] = tile[c + e][r];
      put(g.cols + block + (int64_t)(j0 + r) * g.m + i0 + c, t);
    }
    if (g.rows && i0 + r < g.m && j0 + c < g.n) {
#pragma unroll
      for (int e = 0; e < 8; ++e) t[e] = tile[r][c + e];
      put(g.rows + block + (int64_t)(i0 + r) * g.n + j0 + c, t);
    }
  }
}

}  // namespace shampoo
