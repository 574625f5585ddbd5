// Batched float32 GEMM / SYRK on the CDNA4 matrix cores, for operands as they lie in memory (any shape, stride and
// alignment; the products on planes made beforehand are gemm_f16x2.h and syrk_bf16.h).
//
// One workgroup (256 threads = 4 wavefronts of 64) computes a 128 x 128 tile of
// C = alpha * A * B (+ beta * C), or a 64 x 64 one (TILE) where there are few of those.  Each wavefront owns a quadrant as
// 2 x 2 MFMA tiles of 32 x 32, or one; tiles that hold nothing (ragged edges, above the diagonal) are passed over.  Slabs of
// 32 values of k go through LDS, the loads of the next one in flight meanwhile.  Operands may be float32 or bfloat16 in
// memory.
//
// A product is six v_mfma_f32_32x32x16_bf16 of operands split into three bf16 terms (bf16_terms.h): 192 cycles for 16
// values of k, 512 on the float32 matrix cores; a bf16 operand is one term and leaves three products, or one.  The terms are
// made once, on the way into LDS (22 vector instructions per thread, operand and 4 values; made on the way out, by both
// wavefronts that read an operand, the vector instructions took longer than the matrix cores).  The five small
// products have accumulators of their own, so that only h h' is rounded at full size.  FP32 keeps
// v_mfma_f32_32x32x2_f32 on float32 slabs for callers that ask for it.
// 64 symmetric products of 1024 (36 of 64 tiles), operands along k / along rows: 530 / 650 us, 700 on the float32 matrix
// cores; that is 0.87 PFLOP/s of bf16 products, where gemm_f16x2.h reaches 1.1 on planes made beforehand.
//
// The operands of the Shampoo step (Sec. 2.3, 3.1.1 of the paper) map onto it as
//   L <- beta2 L + (1-beta2) G G^T   A(i,k) = G[i][k]   B(k,j) = G[j][k]   (both k-contiguous)
//   R <- beta2 R + (1-beta2) G^T G   A(i,k) = G[k][i]   B(k,j) = G[k][j]   (both row-contiguous)
//   T = Lbar G                       A(i,k) = Lbar[k][i] (symmetric)  B(k,j) = G[k][j]
//   P = T Rbar                       A(i,k) = T[i][k]   B(k,j) = Rbar[k][j]
//   X = Q f(Lambda) Q^T              A(i,k) = f_k Qt[k][i]  B(k,j) = Qt[k][j]
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "bf16_terms.h"
#include "group.h"

namespace shampoo {

constexpr int BM = 128;
constexpr int BN = 128;
constexpr int BK = 32;          // k-slab depth
constexpr int GEMM_LDK = BK + 4;      // FP32, rows of a slab [row][k] and [k][row], floats: 16-byte aligned, four banks apart
constexpr int GEMM_SMALL = 64;        // the smaller tile
// Planes: rows of 32 values of k, 20 words apart; where four rows at a time are written (ROW_CONTIG), every fourth row lies beside
// the next, and the four groups are 16 banks apart.  The 16 lanes that are served at a time then cover the 64 banks, in
// 16-byte reads and in 8-byte writes.
constexpr int GEMM_PK = BK / 2 + 4;
template <int ROWS> struct GemmSlab {
  static constexpr int LDR = ROWS + 4, FLOATS = ROWS * GEMM_LDK;   // FLOATS: the larger of the two layouts
  static constexpr int PGROUP = ROWS / 4 * GEMM_PK + 16, PLANE = 4 * PGROUP;   // words
  static constexpr int PASSES = ROWS * BK / 1024;                  // ROWS x BK floats = 256 threads x PASSES float4
  static_assert(BK * LDR <= FLOATS && ROWS * GEMM_PK <= PLANE, "slab");
};
constexpr int GEMM_THREADS = 256;
constexpr int NUM_XCD = 8;

// How element (row, k) of an operand is laid out in memory.
//   K_CONTIG:   ptr[row * ld + k]     (a row-major matrix used as A, or B given transposed)
//   ROW_CONTIG: ptr[k * ld + row]     (a row-major matrix used as B, or A given transposed)
enum { K_CONTIG = 0, ROW_CONTIG = 1 };

// where a row of a plane begins; row + 32 i lies i plane_tile() words further
template <int ORIENT, int ROWS> __device__ __forceinline__ int plane_row(int row) {
  return ORIENT == K_CONTIG ? row * GEMM_PK : (row & 3) * GemmSlab<ROWS>::PGROUP + (row >> 2) * GEMM_PK;
}
template <int ORIENT> constexpr int plane_tile() { return ORIENT == K_CONTIG ? 32 * GEMM_PK : 8 * GEMM_PK; }

enum { EPI_STORE = 0, EPI_STORE_NORM = 1, EPI_SYRK = 2 };

// One block of a 2-D parameter (Sec. 4.2.1 blocking): where it sits inside the
// caller's row-major tensor.
struct BlockDesc {
  int32_t param;   // index into the pointer table
  int32_t ld;      // columns of the parameter
  int64_t offset;  // row0 * ld + col0 (elements)
  int64_t state_offset;  // offset of the parameter inside the A / M state arrays, plus `offset`
};

// Where an operand of batch entry b lives.
struct Operand {
  const void *base;      // used when !from_table
  int64_t batch_stride;  // elements
  int32_t ld;
  int32_t from_table;    // 1: pointer = ptr_table[desc[b].param] + desc[b].offset, ld = desc[b].ld
};

struct GemmArgs {
  Operand a, b;
  float *c;
  int64_t c_batch_stride;
  int32_t ldc;
  int32_t M, N, K;
  float alpha, beta;
  double alpha_d, beta_d;       // used instead of alpha, beta by the ACC64 kernels
  const BlockDesc *desc;
  const void *const *ptr_table;
  const float *kscale;          // per-k multiplier of A (length K per batch entry), or nullptr
  int64_t kscale_stride;
  const int32_t *skip;          // per batch entry: nonzero = leave C untouched, or nullptr
  float *norm_partial;          // EPI_STORE_NORM: [batch][tiles] sums of squares of the stored tile
  int32_t tiles_m, tiles_n, tiles;  // tiles = tiles per batch entry (triangular count for SYRK)
  int32_t tile0;                // EPI_SYRK: the first of them (rows of tiles in front of it stay as they are)
  int32_t batch;
  int32_t ksplit, krange;       // EPI_SYRK, ksplit > 1: batch entry b is the range b % ksplit, of krange values of k, of operand b / ksplit;
  double *c64;                  // its plain sum goes here, in float64 like c (ACC64 kernels)
  const float *gmax;            // largest element of a block of gradients, per gmax_per operand entries (nullptr: none):
  int32_t gmax_per;             // A and B are multiplied by range_scale of it where scale_a and scale_b say so, and
  int32_t scale_a, scale_b;     // the result is divided by its power unscale
  int32_t unscale;
  __device__ __forceinline__ void globals() { to_global(a.base, b.base, c, desc, ptr_table, kscale, skip, norm_partial, c64, gmax); }
};

__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
  return __uint_as_float(((uint32_t)h) << 16);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static __device__ __forceinline__ void load4(const float *p, float v[4]) {
    const float4 t = *reinterpret_cast<const float4 *>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  }
  static __device__ __forceinline__ float load1(const float *p) { return *p; }
};
template <> struct Elem<uint16_t> {
  static __device__ __forceinline__ void load4(const uint16_t *p, float v[4]) {
    const uint2 t = *reinterpret_cast<const uint2 *>(p);
    v[0] = __uint_as_float(t.x << 16);
    v[1] = __uint_as_float(t.x & 0xffff0000u);
    v[2] = __uint_as_float(t.y << 16);
    v[3] = __uint_as_float(t.y & 0xffff0000u);
  }
  static __device__ __forceinline__ float load1(const uint16_t *p) { return bf16_to_f32(*p); }
};

// Four consecutive elements at any address of the element type's alignment: global loads and stores of 8 and 16 bytes
// need no alignment of their own.
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint16_t ushort4u __attribute__((ext_vector_type(4), aligned(2)));
template <typename GT>
__device__ __forceinline__ void load_u4(const GT *p, float (&v)[4]) {
  if constexpr (sizeof(GT) == 2) {
    const ushort4u x = *reinterpret_cast<const ushort4u *>(p);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = bf16_to_f32(x[e]);
  } else {
    const float4u x = *reinterpret_cast<const float4u *>(p);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = x[e];
  }
}
__device__ __forceinline__ void store_u4(float *p, const float (&v)[4]) { *reinterpret_cast<float4u *>(p) = float4u{v[0], v[1], v[2], v[3]}; }

// Fetches one 128 x BK operand slab into registers (4 * LOAD_PASSES floats per thread)
// and later writes it into LDS as [row][k] (K_CONTIG) or [k][row].  Whatever is read lies inside the matrix: rows past its
// last one read that again (what they reach is never stored), values of k past the end are zero, and of four rows that
// cross the end the last four of the matrix are read and moved into place.
// BITS (bf16 operands): fetched as they lie, two elements to a word, and made floats by unpack().
template <int ORIENT, typename T, int ROWS, bool BITS = false>
struct TileLoader {
  typedef GemmSlab<ROWS> S;
  static constexpr int PASSES = S::PASSES, QUADS = ROWS / 4;   // QUADS threads side by side along the rows, PASSES values of k each
  const T *ptr;     // operand origin for this batch entry, already offset to the tile's first row
  int ld;
  int rows_left;    // valid rows from the tile's first row
  int K;
  int lane_row;     // ROW_CONTIG: the first of the four rows that are read
  int back;         // ROW_CONTIG: how far they lie in front of their place
  float r[PASSES][4];

  __device__ __forceinline__ void init(const T *p, int ld_, int rows_left_, int K_, int tid) {
    ptr = p; ld = ld_; rows_left = rows_left_; K = K_;
    const int r4 = (tid % QUADS) * 4;
    lane_row = min(r4, max(rows_left - 4, 0));
    back = r4 < rows_left ? r4 - lane_row : 0;
  }

  __device__ __forceinline__ void fetch(int k0, int tid) {
    if constexpr (BITS) { fetch_bits(k0, tid); return; }
    const bool whole = k0 + BK <= K;             // uniform
    if (ORIENT == K_CONTIG) {
      constexpr int TPR = BK / 4, RPP = GEMM_THREADS / TPR;   // threads per row, rows per pass
      const int row = tid / TPR, kq = k0 + (tid % TPR) * 4;
#pragma unroll
      for (int h = 0; h < PASSES; ++h) {
        const T *p = ptr + (int64_t)min(row + RPP * h, rows_left - 1) * ld + kq;
        if (whole) {
          load_u4<T>(p, r[h]);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) r[h][j] = kq + j < K ? Elem<T>::load1(p + j) : 0.f;
        }
      }
    } else {
      const int kk = k0 + PASSES * (tid / QUADS);        // PASSES values of k
      if (rows_left >= 4) {                      // uniform
#pragma unroll
        for (int h = 0; h < PASSES; ++h) {
#pragma unroll
          for (int j = 0; j < 4; ++j) r[h][j] = 0.f;
          if (whole || kk + h < K) load_u4<T>(ptr + (int64_t)(kk + h) * ld + lane_row, r[h]);
        }
        if (rows_left < ROWS && (rows_left & 3)) { // uniform
#pragma unroll
          for (int h = 0; h < PASSES; ++h) {
            if (back & 1) { r[h][0] = r[h][1]; r[h][1] = r[h][2]; r[h][2] = r[h][3]; }
            if (back & 2) { r[h][0] = r[h][2]; r[h][1] = r[h][3]; }
          }
        }
      } else {
        const int r4 = (tid % QUADS) * 4;
#pragma unroll
        for (int h = 0; h < PASSES; ++h)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            r[h][j] = (kk + h < K && r4 + j < rows_left) ? Elem<T>::load1(ptr + (int64_t)(kk + h) * ld + r4 + j) : 0.f;
      }
    }
  }

  // Values that are converted here are waited for here, ahead of the products that are to hide the loads, which the float32 matrix
  // cores take long over: T = Lbar G of 96 bf16 blocks of 1024 there 2356 us so, 1943 with the bits.
  __device__ __forceinline__ void fetch_bits(int k0, int tid) {
    typedef uint32_t pair __attribute__((ext_vector_type(2)));
    const bool whole = k0 + BK <= K;             // uniform
    auto put = [&](int h, uint32_t x, uint32_t y) { r[h][0] = __uint_as_float(x); r[h][1] = __uint_as_float(y); };
    auto four = [&](int h, const T *p) { const pair x = __builtin_bit_cast(pair, *reinterpret_cast<const ushort4u *>(p)); put(h, x[0], x[1]); };
    auto some = [&](int h, const T *p, auto exists) {
      uint32_t x[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = exists(j) ? p[j] : 0;
      put(h, x[0] | x[1] << 16, x[2] | x[3] << 16);
    };
    if (ORIENT == K_CONTIG) {
      constexpr int TPR = BK / 4, RPP = GEMM_THREADS / TPR;
      const int row = tid / TPR, kq = k0 + (tid % TPR) * 4;
#pragma unroll
      for (int h = 0; h < PASSES; ++h) {
        const T *p = ptr + (int64_t)min(row + RPP * h, rows_left - 1) * ld + kq;
        if (whole) four(h, p); else some(h, p, [&](int j) { return kq + j < K; });
      }
    } else {
      const int kk = k0 + PASSES * (tid / QUADS), r4 = (tid % QUADS) * 4;
#pragma unroll
      for (int h = 0; h < PASSES; ++h) {
        const T *p = ptr + (int64_t)(kk + h) * ld;
        if (rows_left < 4) some(h, p + r4, [&](int j) { return kk + h < K && r4 + j < rows_left; });
        else if (whole) four(h, p + lane_row);
        else { put(h, 0, 0); if (kk + h < K) four(h, p + lane_row); }
      }
    }
  }
  // once behind a fetch, ahead of all that works on the values
  __device__ __forceinline__ void unpack() {
    if constexpr (BITS) {
#pragma unroll
      for (int h = 0; h < PASSES; ++h) {
        const uint32_t x = __float_as_uint(r[h][0]), y = __float_as_uint(r[h][1]);
        r[h][0] = __uint_as_float(x << 16); r[h][1] = __uint_as_float(x & 0xffff0000u);
        r[h][2] = __uint_as_float(y << 16); r[h][3] = __uint_as_float(y & 0xffff0000u);
      }
      if (ORIENT == ROW_CONTIG && rows_left >= 4 && rows_left < ROWS && (rows_left & 3)) // uniform
#pragma unroll
        for (int h = 0; h < PASSES; ++h) {
          if (back & 1) { r[h][0] = r[h][1]; r[h][1] = r[h][2]; r[h][2] = r[h][3]; }
          if (back & 2) { r[h][0] = r[h][2]; r[h][1] = r[h][3]; }
        }
    }
  }

  __device__ __forceinline__ void multiply(float s) {
#pragma unroll
    for (int h = 0; h < PASSES; ++h)
#pragma unroll
      for (int j = 0; j < 4; ++j) r[h][j] *= s;
  }

  // kscale: optional per-k multiplier (already offset to this batch entry), k0 = slab origin
  __device__ __forceinline__ void scale(const float *kscale, int k0, int tid) {
    if (ORIENT == K_CONTIG) {
      const int kq = (tid % (BK / 4)) * 4;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float s = (k0 + kq + j < K) ? kscale[k0 + kq + j] : 0.f;
#pragma unroll
        for (int h = 0; h < PASSES; ++h) r[h][j] *= s;
      }
    } else {
      const int kk = PASSES * (tid / QUADS);
#pragma unroll
      for (int h = 0; h < PASSES; ++h) {
        const int k = k0 + kk + h;
        const float s = (k < K) ? kscale[k] : 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) r[h][j] *= s;
      }
    }
  }

  __device__ __forceinline__ void store(float *lds, int tid) const {
    if (ORIENT == K_CONTIG) {
      constexpr int TPR = BK / 4, RPP = GEMM_THREADS / TPR;
      const int row = tid / TPR, kq = (tid % TPR) * 4;
#pragma unroll
      for (int h = 0; h < PASSES; ++h)
        *reinterpret_cast<float4 *>(lds + (row + RPP * h) * GEMM_LDK + kq) = make_float4(r[h][0], r[h][1], r[h][2], r[h][3]);
    } else {
      const int kk = PASSES * (tid / QUADS), r4 = (tid % QUADS) * 4;
#pragma unroll
      for (int h = 0; h < PASSES; ++h)
        *reinterpret_cast<float4 *>(lds + (kk + h) * S::LDR + r4) = make_float4(r[h][0], r[h][1], r[h][2], r[h][3]);
    }
  }
  // the planes of the terms, h first
  __device__ __forceinline__ void store_terms(uint32_t *lds, int tid) {
    constexpr bool ONE = sizeof(T) == 2;
    if (ORIENT == K_CONTIG) {
      constexpr int TPR = BK / 4, RPP = GEMM_THREADS / TPR;
      uint32_t *at = lds + (tid / TPR) * GEMM_PK + (tid % TPR) * 2;
#pragma unroll
      for (int h = 0; h < PASSES; ++h)
#pragma unroll
        for (int t = 0; t < (ONE ? 1 : 3); ++t) {
          const uint32_t x = bf16_round2(r[h][0], r[h][1], !ONE && t < 2), y = bf16_round2(r[h][2], r[h][3], !ONE && t < 2);
          *reinterpret_cast<uint2 *>(at + t * S::PLANE + RPP * h * GEMM_PK) = make_uint2(x, y);
        }
    } else {
      uint32_t *at = lds + (tid % QUADS) * GEMM_PK + PASSES / 2 * (tid / QUADS);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < (ONE ? 1 : 3); ++t) {
          const uint32_t x = bf16_round2(r[0][e], r[1][e], !ONE && t < 2);
          if constexpr (PASSES == 4) {
            const uint32_t y = bf16_round2(r[2][e], r[3][e], !ONE && t < 2);
            *reinterpret_cast<uint2 *>(at + t * S::PLANE + e * S::PGROUP) = make_uint2(x, y);
          } else {
            at[t * S::PLANE + e * S::PGROUP] = x;
          }
        }
    }
  }

  // the MFMA operand of 32 rows: row (of the lane), values k ... k + 7 of the slab
  static __device__ __forceinline__ floatx8 operand(const float *lds, int row, int k) {
    return ORIENT == K_CONTIG ? lds_row8<GEMM_LDK>(lds, row, k) : lds_col8<S::LDR>(lds, k, row);
  }
  // of 32 rows: tile i behind the lane's address, values k ... k + 7 of a half of the slab that the lane's address names
  static __device__ __forceinline__ void terms(const uint32_t *lane, int i, int s, Bf16Terms &x) {
    auto plane = [&](int t) {
      return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(lane + t * S::PLANE + i * plane_tile<ORIENT>() + 8 * s));
    };
    x.h = plane(0);
    if constexpr (sizeof(T) == 4) { x.l = plane(1); x.m = plane(2); }
  }
};

// Consecutive workgroup ids are dealt round-robin to the 8 XCDs, each with its
// own L2.  Re-map so that every XCD works on one contiguous range of tiles:
// tiles that share operand panels then hit the same L2.
__device__ __forceinline__ int xcd_remap(int wg, int total) {
  const int per = (total + NUM_XCD - 1) / NUM_XCD;
  return (wg % NUM_XCD) * per + wg / NUM_XCD;
}

template <typename T>
__device__ __forceinline__ const T *operand_ptr(const Operand &o, const BlockDesc *desc,
                                                const void *const *table, int b, int &ld) {
  if (o.from_table) {
    const BlockDesc d = desc[b];
    ld = d.ld;
    return global_ptr<const T>(table[d.param]) + d.offset;
  }
  ld = o.ld;
  return reinterpret_cast<const T *>(o.base) + (int64_t)b * o.batch_stride;
}

// ACC64: the products of a slab of 32 values of k start from zero accumulators, the small ones first (two roundings of full
// size), and are added into float64 registers; the epilogue (alpha * acc + beta * C) is
// evaluated in float64 before the single rounding to float32.  Used for the
// factor updates: the first root refresh sees L = G G^T of a single gradient,
// whose condition number is the square of G's, and a plain float32 running sum
// over k would perturb its small eigenvalues by more than the parity budget.
template <int AO, int BO, typename TA, typename TB, int EPI, bool KSCALE, bool ACC64 = false, bool FP32 = false, int TILE = BM>
__global__ __launch_bounds__(GEMM_THREADS, TILE == BM ? 2 : 4) void gemm_mfma_kernel(const Group<GemmArgs> grp) {
  static_assert(!(ACC64 && FP32), "float64 sums: bf16 terms");
  typedef GemmSlab<TILE> S;
  typedef TileLoader<AO, TA, TILE, FP32 && sizeof(TA) == 2> LoadA;
  typedef TileLoader<BO, TB, TILE, FP32 && sizeof(TB) == 2> LoadB;
  constexpr int WT = TILE / 64, HALF = TILE / 2;      // a wavefront has WT x WT tiles of 32 x 32
  constexpr int SLAB_A = FP32 ? S::FLOATS : (sizeof(TA) == 2 ? 1 : 3) * S::PLANE, SLAB_B = FP32 ? S::FLOATS : (sizeof(TB) == 2 ? 1 : 3) * S::PLANE;
  constexpr int STAGES = FP32 ? 2 : 1;           // two workgroups per CU either way, four of the smaller tile
  __shared__ __align__(16) uint32_t As[STAGES][SLAB_A];
  __shared__ __align__(16) uint32_t Bs[STAGES][SLAB_B];
  __shared__ float red[4];

  int wg;
  const GemmArgs g = group_pick(grp, wg);
  const int total = g.tiles * g.batch;
  const int logical = xcd_remap(wg, total);
  if (logical >= total) return;
  const int b = logical / g.tiles;
  const int tile = logical - b * g.tiles;
  int ti, tj;
  if (EPI == EPI_SYRK) {
    // lower-triangular tile index: t = ti (ti + 1) / 2 + tj, tj <= ti
    const int t = tile + g.tile0;
    ti = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
    while ((ti + 1) * (ti + 2) / 2 <= t) ++ti;
    while (ti * (ti + 1) / 2 > t) --ti;
    tj = t - ti * (ti + 1) / 2;
  } else {
    ti = tile / g.tiles_n;
    tj = tile - ti * g.tiles_n;
  }
  if (g.skip != nullptr && g.skip[b] != 0) return;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int row0 = ti * TILE, col0 = tj * TILE;

  int lda, ldb, entry = b, K = g.K, kfirst = 0;
  if (EPI == EPI_SYRK && g.ksplit > 1) {
    entry = b / g.ksplit;
    kfirst = (b - entry * g.ksplit) * g.krange;
    K = min(g.krange, g.K - kfirst);
  }
  const TA *pa = operand_ptr<TA>(g.a, g.desc, g.ptr_table, entry, lda);
  const TB *pb = operand_ptr<TB>(g.b, g.desc, g.ptr_table, entry, ldb);
  if (EPI == EPI_SYRK) {
    pa += AO == K_CONTIG ? (int64_t)kfirst : (int64_t)kfirst * lda;
    pb += BO == K_CONTIG ? (int64_t)kfirst : (int64_t)kfirst * ldb;
  }
  LoadA la;
  LoadB lb;
  la.init(pa + (AO == K_CONTIG ? (int64_t)row0 * lda : (int64_t)row0), lda, g.M - row0, K, tid);
  lb.init(pb + (BO == K_CONTIG ? (int64_t)col0 * ldb : (int64_t)col0), ldb, g.N - col0, K, tid);
  const float *ks = KSCALE ? g.kscale + (int64_t)b * g.kscale_stride : nullptr;
  const float sg = g.gmax ? range_scale(g.gmax[entry / g.gmax_per]) : 1.f;
  // which of this wavefront's tiles hold part of the result
  bool on[WT][WT];
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j) {
      const int r = wm * HALF + 32 * i, c = wn * HALF + 32 * j;
      on[i][j] = row0 + r < g.M && col0 + c < g.N && !(EPI == EPI_SYRK && ti == tj && c > r);
    }

  floatx16 acc[WT][WT], rest[ACC64 || FP32 ? 1 : WT][ACC64 || FP32 ? 1 : WT];
  double acc64[ACC64 ? WT : 1][ACC64 ? WT : 1][ACC64 ? 16 : 1];
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        acc[i][j][v] = 0.f;
        if constexpr (!ACC64 && !FP32) rest[i][j][v] = 0.f;
        if constexpr (ACC64) acc64[i][j][v] = 0.0;
      }

  const int nk = (K + BK - 1) / BK;
  auto fetch = [&](int k0) {
    la.fetch(k0, tid);
    lb.fetch(k0, tid);
  };
  auto store = [&](int stage, int k0) {
    if constexpr (FP32 && sizeof(TA) == 2) la.unpack();
    if constexpr (FP32 && sizeof(TB) == 2) lb.unpack();
    if (sg != 1.f) {                     // uniform
      if (g.scale_a) la.multiply(sg);
      if (g.scale_b) lb.multiply(sg);
    }
    if (KSCALE) la.scale(ks, k0, tid);
    if constexpr (FP32) {
      la.store(reinterpret_cast<float *>(As[stage]), tid);
      lb.store(reinterpret_cast<float *>(Bs[stage]), tid);
    } else {
      la.store_terms(As[stage], tid);
      lb.store_terms(Bs[stage], tid);
    }
  };
  fetch(0);
  if constexpr (FP32) {
    store(0, 0);
    __syncthreads();
  }

  const int arow = wm * HALF + (lane & 31);
  const int bcol = wn * HALF + (lane & 31);
  const int khalf = lane >> 5;
  const uint32_t *lane_a = As[0] + plane_row<AO, TILE>(arow) + 4 * khalf, *lane_b = Bs[0] + plane_row<BO, TILE>(bcol) + 4 * khalf;
  constexpr bool AONE = sizeof(TA) == 2, BONE = sizeof(TB) == 2;
  for (int kt = 0; kt < nk; ++kt) {
    if constexpr (!FP32) {
      if (kt > 0) __syncthreads();       // the slab before has been read
      store(0, kt * BK);
      __syncthreads();
    }
    if (kt + 1 < nk) fetch((kt + 1) * BK);
    auto terms_a = [&](int i, int s, Bf16Terms &x) { LoadA::terms(lane_a, i, s, x); };
    auto terms_b = [&](int j, int s, Bf16Terms &x) { LoadB::terms(lane_b, j, s, x); };
    if constexpr (ACC64) {
#pragma unroll
      for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j)
          if (on[i][j]) {
            floatx16 c = {};
            Bf16Terms a, t;
            terms_a(i, 0, a);
            terms_b(j, 0, t);
            const bf16x8 ah = a.h, th = t.h;
            c = bf16_small_products<AONE, BONE>(a, t, c);
            terms_a(i, 1, a);
            terms_b(j, 1, t);
            c = bf16_small_products<AONE, BONE>(a, t, c);
            c = bf16_mfma(ah, th, c);
            c = bf16_mfma(a.h, t.h, c);
#pragma unroll
            for (int v = 0; v < 16; ++v) acc64[i][j][v] += (double)c[v];
          }
    } else if constexpr (FP32) {
#pragma unroll 1
      for (int s = 0; s < 2; ++s) {
        const float *as = reinterpret_cast<const float *>(As[kt & 1]), *bs = reinterpret_cast<const float *>(Bs[kt & 1]);
        floatx8 a[WT], t[WT];
#pragma unroll
        for (int i = 0; i < WT; ++i) {
          a[i] = LoadA::operand(as, arow + 32 * i, 16 * s + 8 * khalf);
          t[i] = LoadB::operand(bs, bcol + 32 * i, 16 * s + 8 * khalf);
        }
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
          for (int j = 0; j < WT; ++j)
            if (on[i][j]) acc[i][j] = fp32_products(a[i], t[j], acc[i][j]);
      }
      if (kt + 1 < nk) store((kt + 1) & 1, (kt + 1) * BK);
      __syncthreads();
    } else {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        Bf16Terms a[WT], t[WT];
#pragma unroll
        for (int i = 0; i < WT; ++i) {
          if (on[i][0] || on[i][WT - 1]) terms_a(i, s, a[i]);
          if (on[0][i] || on[WT - 1][i]) terms_b(i, s, t[i]);
        }
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
          for (int j = 0; j < WT; ++j)
            if (on[i][j]) {
              rest[i][j] = bf16_small_products<AONE, BONE>(a[i], t[j], rest[i][j]);
              acc[i][j] = bf16_mfma(a[i].h, t[j].h, acc[i][j]);
            }
      }
    }
  }
  if constexpr (!ACC64 && !FP32)
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
      for (int j = 0; j < WT; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] += rest[i][j][v];
  // s is up to 2^120, its square in float64
  const float inv_s = 1.f / sg;
  const double unscale = g.unscale == 2 ? (double)inv_s * (double)inv_s : g.unscale == 1 ? (double)inv_s : 1.0;
  const double alpha_d = g.alpha_d * unscale;
  const float alpha = g.unscale ? g.alpha * inv_s : g.alpha;

  // ---- epilogue.  Accumulator element v of MFMA tile (mi, ni) is
  //      row = wm*HALF + mi*32 + 8*(v/4) + 4*(lane/32) + v%4, col = wn*HALF + ni*32 + lane%32.
  float *c = g.c + (int64_t)b * g.c_batch_stride;
  const int ldc = g.ldc;
  // The mirror image of four rows of a lane is four consecutive columns: one store, in 16-byte aligned rows (64 symmetric products of
  // 1024: 535 us with four, 520 so).  Small tiles of bf16 operands that lie along k are kept at their five wavefronts per SIMD instead, which
  // the four values would make four (200 of 301 rows to 202 of 202: 65 us with, 62 without; along rows 70.5 and 72.5).
  const bool mirror4 = EPI == EPI_SYRK && (TILE == BM || sizeof(TA) == 4 || AO != K_CONTIG) && (ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(c) & 15) == 0;
  float ss = 0.f;
#pragma unroll
  for (int mi = 0; mi < WT; ++mi)
#pragma unroll
    for (int ni = 0; ni < WT; ++ni) {
      const int j = col0 + wn * HALF + ni * 32 + (lane & 31);
      // EPI_SYRK with a nonzero beta: the 16 old values of an MFMA tile are requested before
      // its first store.  The mirrored stores may alias later loads, so interleaved they
      // would cost one memory round trip per element instead of one per tile.
      float old[EPI == EPI_SYRK ? 16 : 1];
      if (EPI == EPI_SYRK) {
        const bool need = ACC64 ? (g.beta_d != 0.0 && g.ksplit <= 1) : (g.beta != 0.f);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int i = row0 + wm * HALF + mi * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
          old[EPI == EPI_SYRK ? v : 0] = (need && i < g.M && j <= i) ? c[(int64_t)i * ldc + j] : 0.f;
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int ibase = row0 + wm * HALF + mi * 32 + 8 * q + 4 * (lane >> 5);
        float below[4];                  // the lane's four elements, where all lie below the diagonal
        const bool four = mirror4 && j < ibase && ibase + 3 < g.M;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = ibase + e;
          float v = ACC64 && EPI != EPI_SYRK ? (float)(alpha_d * acc64[ACC64 ? mi : 0][ACC64 ? ni : 0][ACC64 ? 4 * q + e : 0])
                                             : alpha * acc[mi][ni][4 * q + e];
          if (i < g.M && j < g.N) {
            if (EPI == EPI_SYRK) {
              // only the lower triangle is computed; its mirror image is written with the
              // same bits so the factor stays exactly symmetric
              if (j <= i) {
                const float o = old[EPI == EPI_SYRK ? 4 * q + e : 0];
                if (ACC64 && g.ksplit > 1) {
                  double *c64 = g.c64 + (int64_t)b * g.c_batch_stride;
                  const double sum = unscale * acc64[ACC64 ? mi : 0][ACC64 ? ni : 0][ACC64 ? 4 * q + e : 0];
                  c64[(int64_t)i * ldc + j] = sum;
                  if (j < i) c64[(int64_t)j * ldc + i] = sum;
                  continue;
                }
                if (ACC64) v = (float)(alpha_d * acc64[ACC64 ? mi : 0][ACC64 ? ni : 0][ACC64 ? 4 * q + e : 0] + g.beta_d * (double)o);
                else v += g.beta * o;
                c[(int64_t)i * ldc + j] = v;
                below[e] = v;
                if (j < i && !four) c[(int64_t)j * ldc + i] = v;
              }
            } else {
              c[(int64_t)i * ldc + j] = v;
              if (EPI == EPI_STORE_NORM) ss += v * v;
            }
          }
        }
        if (EPI == EPI_SYRK && four && !(ACC64 && g.ksplit > 1)) 
          *reinterpret_cast<float4 *>(c + (int64_t)j * ldc + ibase) = make_float4(below[0], below[1], below[2], below[3]);
      }
    }
  if (EPI == EPI_STORE_NORM) {
    // fixed-order reduction: lanes by xor-shuffle, then the 4 wavefronts in order
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
    if (lane == 0) red[wave] = ss;
    __syncthreads();
    if (tid == 0) g.norm_partial[(int64_t)b * g.tiles + tile] = (red[0] + red[1]) + (red[2] + red[3]);
  }
}

}  // namespace shampoo
