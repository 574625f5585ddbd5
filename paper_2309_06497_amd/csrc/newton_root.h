// Coupled inverse Newton iteration for the root inverse (Sec. 3.2.1, item 2 of the paper):
//   A = scale * L + eps I,  c^p = 2 ||A||_F / (p + 1),  X_0 = I / c,  M_0 = A / c^p,
//   T_k = ((p + 1) I - M_k) / p,  X_{k+1} = X_k T_k,  M_{k+1} = T_k^p M_k,
// until ||M_k - I||_inf < tol.  Every iterate is a polynomial in A, hence symmetric, and all
// of them commute: each product is formed on its lower-triangular tiles only and mirrored
// (the SYRK epilogue of the GEMM kernel), 36 of 64 tiles at n = 1024.  The kernels here are
// the small elementwise / reduction steps around those products; convergence is tracked per
// matrix on the device (`done` flags, which the GEMM launches take as their skip list), so
// a refresh needs no host synchronisation.  The host enqueues all iterations up to the cap, and most find every matrix done,
// so launches count: the test on M_k is made by the last workgroup of T_k's launch, a finished matrix is copied out behind the
// last iteration (nothing writes its X any more), and X_1 = T_0 / c is written beside T_0.  64 matrices of 1024 with six launches an
// iteration and X_0 T_0 a product 22.8 ms, with four and without it 21.6.
//
// The last M_k is not formed where it would only be found close enough to I.  With E = M_k - I,
//   M_{k+1} - I = (I - E / p)^p (I + E) - I = - (p + 1) / (2 p) E^2 + ...,
// a polynomial whose coefficients alternate in sign from E^2 on and add up in absolute value to its value at -I, which is 1:
// ||M_{k+1} - I|| <= ||E||^2 for ||E|| <= 1.  So ||E||^2 < tol is in exact arithmetic the paper's test on M_{k+1}, one product
// (X_{k+1} = X_k T_k) for four.  A tolerance below the floor of float32 (next paragraph) a formed M_{k+1} might not pass; such a matrix would
// go on until its norm no longer halves, now it ends at k + 1.
// 64 matrices of 1024 (9 iterations): 20.8 -> 19.35 ms.  For 129 ... 1024, p of 1 ... 8, condition numbers of 1.6 to above 1e6 and a tolerance of
// 1e-6 (n 2^-24: 7.7e-6 and more) neither a number of iterations changed nor an error against float64 by more than 1 %.
//
// Arithmetic is float32: operands as three bf16 terms, products summed in float32 (gemm_mfma.h).  ||M_k - I||_inf cannot fall below
// about n * 2^-24 * (a few) in that arithmetic, so besides the paper's test the iteration of
// a matrix also ends when the norm, once below 0.1 (quadratic regime), fails to halve.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include "bf16_terms.h"
#include "group.h"

namespace shampoo {

struct NewtonArgs {
  const float *a;        // [batch][n][n] input matrices
  int64_t a_stride;
  float *M, *X, *T;      // [batch][n][n] work matrices
  float *X1;             // X_1, where the iterate is X_0; otherwise nullptr
  double *rowpart;       // [batch][ceil(n / 32)] sums of squares of A by block rows
  float *err;            // [batch] ||M - I||_inf of the current iterate (atomic max, cleared by the test)
  int32_t *arrived;      // [batch] workgroups whose rows are in err (cleared by the test)
  float *prev;           // [batch] the norm one iteration earlier
  int32_t *done;         // [batch] M is not needed any more (converged, stalled, capped or failed)
  int32_t *xdone;        // [batch] nor is X_k T_k
  int32_t *failed;       // [batch] not finite: the caller keeps the previous root
  int32_t *iters;        // [batch] number of iterations taken
  int32_t n, p, k, max_iter;
  float epsilon, scale, tol;
};

constexpr int NEWTON_TILE = 32;
// Elements (i, j), (i, j + step) ... of an n x n matrix, four of them, zeros past its edges.  step 1 is one 16-byte access, where rows are
// whole pieces of 16 bytes (the sizes of blocks); a caller's may be any, and then neighbouring lanes take neighbouring elements.  With four
// in a row of each lane, one by one, newton_prep_kernel took 22 us a launch for 64 matrices of 1023 (mean of all 101 of a call), 16 so.
__device__ __forceinline__ void newton_get4(const float *a, int n, int step, int i, int j, float (&x)[4]) {
  const float *p = a + (int64_t)i * n + j;
  if (step == 1) {
    const float4 q = i < n && j < n ? *reinterpret_cast<const float4 *>(p) : make_float4(0.f, 0.f, 0.f, 0.f);
    x[0] = q.x; x[1] = q.y; x[2] = q.z; x[3] = q.w;
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = i < n && j + step * e < n ? p[step * e] : 0.f;
}
__device__ __forceinline__ void newton_put4(float *a, int n, int step, int i, int j, const float (&x)[4]) {
  float *p = a + (int64_t)i * n + j;
  if (step == 1) {
    if (i < n && j < n) *reinterpret_cast<float4 *>(p) = make_float4(x[0], x[1], x[2], x[3]);
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (i < n && j + step * e < n) p[step * e] = x[e];
}
__device__ __forceinline__ bool newton_quads(const float *a, int n) { return n % 4 == 0 && reinterpret_cast<uintptr_t>(a) % 16 == 0; }

// Block row I of A = scale * sym(L) + eps I from the tiles (I, J) and (J, I), J <= I: f(J, r, c, step, x) has row r of the tile, its columns
// c, c + step ... and their values (step: a constant, known only at run time it cost newton_init_kernel 30 of 207 us for 64 matrices of 1024).
// Read along rows; the mirror image goes through LDS.  Read down its columns it took 360 us for the norm and 460 for M_0 and X_0 of 64
// matrices of 1024, 92 and 207 so; of 1023 380 and 490, 129 and 473 so.  256 threads.
template <typename F> __device__ __forceinline__ void newton_block_row(const float *a, int n, int I, float scale, float eps, int &bad, F f) {
  __shared__ float mirror[NEWTON_TILE][NEWTON_TILE + 1];
  const auto tiles = [&](auto step_) {
    constexpr int step = decltype(step_)::value;
    const int r = threadIdx.x >> 3, c = (threadIdx.x & 7) * (step == 1 ? 4 : 1), i = I * NEWTON_TILE + r, mj = I * NEWTON_TILE + c;
    for (int J = 0; J <= I; ++J) {
      const int j = J * NEWTON_TILE + c, mi = J * NEWTON_TILE + r;
      float x[4], y[4];
      newton_get4(a, n, step, i, j, x);
      newton_get4(a, n, step, mi, mj, y);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (!(fabsf(x[e]) <= 3.0e38f) || !(fabsf(y[e]) <= 3.0e38f)) bad = 1;
      }
      __syncthreads();                   // the tile before has been read
#pragma unroll
      for (int e = 0; e < 4; ++e) mirror[r][c + step * e] = y[e];
      __syncthreads();
      double v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = (double)scale * 0.5 * ((double)x[e] + (double)mirror[c + step * e][r]);
        if (i == j + step * e) v[e] += (double)eps;
      }
      f(J, r, c, step_, v);
    }
  };
  if (newton_quads(a, n)) tiles(std::integral_constant<int, 1>{});
  else tiles(std::integral_constant<int, 8>{});
}

// grid (ceil(n / 32), batch): a block row's part of the sum of squares, non-finite check.
__global__ __launch_bounds__(256) void newton_norm_kernel(const NewtonArgs g) {
  __shared__ double red[4];
  const int I = blockIdx.x, b = blockIdx.y, n = g.n, tid = threadIdx.x;
  double ss = 0.0;
  int bad = 0;
  newton_block_row(g.a + (int64_t)b * g.a_stride, n, I, g.scale, g.epsilon, bad, [&](int J, int r, int c, auto step, const double (&v)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (I * NEWTON_TILE + r < n && J * NEWTON_TILE + c + step * e < n) ss += (J < I ? 2.0 : 1.0) * (v[e] * v[e]);
  });
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) { ss += __shfl_xor(ss, off, 64); bad |= __shfl_xor(bad, off, 64); }
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  if (bad && (tid & 63) == 0) atomicOr(&g.failed[b], 1);
  __syncthreads();
  if (tid == 0) g.rowpart[(int64_t)b * gridDim.x + I] = (red[0] + red[1]) + (red[2] + red[3]);
}

// grid (ceil(n / 32), batch): block row I of M_0 = A / c^p and X_0 = I / c, up to the diagonal, and its mirror image; the Frobenius norm is
// summed from the parts in a fixed order by every workgroup.
__global__ __launch_bounds__(256) void newton_init_kernel(const NewtonArgs g) {
  __shared__ double red[4];
  __shared__ float tile[NEWTON_TILE][NEWTON_TILE + 1];
  const int I = blockIdx.x, b = blockIdx.y, n = g.n, tid = threadIdx.x;
  if (g.failed[b]) {
    if (I == 0 && tid == 0) { g.done[b] = 1; g.xdone[b] = 1; g.iters[b] = 0; }
    return;
  }
  double ss = 0.0;
  for (int j = tid; j < (int)gridDim.x; j += 256) ss += g.rowpart[(int64_t)b * gridDim.x + j];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  const double fro = sqrt((red[0] + red[1]) + (red[2] + red[3]));
  const double cp = 2.0 * fro / ((double)g.p + 1.0);           // c^p
  const bool ok = cp > 0.0 && cp <= 1.0e300;
  const double inv_cp = ok ? 1.0 / cp : 0.0;
  const float inv_c = ok ? (float)pow(cp, -1.0 / (double)g.p) : 0.f;
  float *M = g.M + (int64_t)b * n * n, *X = g.X + (int64_t)b * n * n;
  int bad = 0;
  // M and X start 256-byte aligned: where A's rows are whole pieces of 16 bytes, so are theirs
  newton_block_row(g.a + (int64_t)b * g.a_stride, n, I, g.scale, g.epsilon, bad, [&](int J, int r, int c, auto step, const double (&v)[4]) {
    const int i = I * NEWTON_TILE + r, j = J * NEWTON_TILE + c, mi = J * NEWTON_TILE + r, mj = I * NEWTON_TILE + c;
    float x[4], id[4], mirror[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[e] = (float)(v[e] * inv_cp);
      id[e] = i == j + step * e ? inv_c : 0.f;
      tile[r][c + step * e] = x[e];      // its last readers are behind a barrier of the next tile's
    }
    newton_put4(M, n, step, i, j, x);
    newton_put4(X, n, step, i, j, id);
    __syncthreads();
    if (J == I) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) { mirror[e] = tile[c + step * e][r]; id[e] = 0.f; }
    newton_put4(M, n, step, mi, mj, mirror);
    newton_put4(X, n, step, mi, mj, id);
  });
  if (I == 0 && tid == 0) {
    g.done[b] = g.xdone[b] = ok ? 0 : 1;
    if (!ok) g.failed[b] = 1;      // zero or non-finite norm
    g.iters[b] = 0; g.err[b] = 0.f; g.prev[b] = 3.0e38f; g.arrived[b] = 0;
  }
}

// The termination test on M_k (k = g.k), and on M_{k+1} where M_k decides it; e = ||M_k - I||_inf.  One thread
__device__ __forceinline__ void newton_check(const NewtonArgs &g, int b, float e) {
  const float pv = g.prev[b];
  int stop = 0, more = 0;
  if (!(e <= 3.0e38f)) { g.failed[b] = 1; stop = 1; }
  else if (e < g.tol) stop = 1;                               // the paper's criterion
  else if (g.k >= g.max_iter) stop = 1;                       // iteration cap
  else if (pv < 0.1f && e > 0.5f * pv) stop = 1;              // float32 floor reached
  else if (e <= 1.f && e * e < g.tol) more = 1;               // the criterion holds for M_{k+1}
  if (stop) g.xdone[b] = 1;
  if (stop || more) { g.done[b] = 1; g.iters[b] = g.k + more; }
  g.prev[b] = e;
}

// T = ((p + 1) I - M) / p and ||M - I||_inf; the last workgroup of a matrix makes the test.  grid (ceil(n / NEWTON_ROWS), batch), a
// wavefront per row at a time.
// The host enqueues all max_iter iterations, and most of them find every matrix done: with a workgroup per row
// 64 matrices of 1024 cost 60 us for each such launch, now about 5 (root of 64 such matrices: 38.6 -> 32.1 ms).
// Otherwise it is bound by memory: 512 MB in 157 us with 4-byte loads, 118 so.
constexpr int NEWTON_ROWS = 32;
__global__ __launch_bounds__(256) void newton_prep_kernel(const NewtonArgs g) {
  const int b = blockIdx.y, n = g.n, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (g.done[b]) {
    if (blockIdx.x == 0 && threadIdx.x == 0) g.xdone[b] = 1;   // X_k T_k of the launch before was its last
    return;
  }
  const float pp = (float)g.p, inv_p = 1.f / pp;
  const bool quads = newton_quads(g.M, n);                   // T and X_1 lie a multiple of 256 bytes further
  const int c = quads ? 4 * lane : lane, step = quads ? 1 : 64;
  const int last = min((int)(blockIdx.x + 1) * NEWTON_ROWS, n);
  float worst = 0.f;
  for (int i = blockIdx.x * NEWTON_ROWS + w; i < last; i += 4) {
    const int64_t row = ((int64_t)b * n + i) * n;
    const float *M = g.M + row;
    float *T = g.T + row, *X1 = g.X1 ? g.X1 + row : nullptr;
    const float inv_c = X1 ? g.X[row + i] : 0.f;
    float rs = 0.f;
#pragma unroll 4
    for (int j = c; j < n; j += 256) {
      float m[4], t[4];
      newton_get4(M, n, step, 0, j, m);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float id = i == j + step * e ? 1.f : 0.f;
        t[e] = ((pp + 1.f) * id - m[e]) * inv_p;
        rs += fabsf(m[e] - id);
      }
      newton_put4(T, n, step, 0, j, t);
      if (X1) {
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] *= inv_c;
        newton_put4(X1, n, step, 0, j, t);
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) rs += __shfl_xor(rs, off, 64);
    if (!(rs <= 3.0e38f)) rs = __int_as_float(0x7f800000);   // NaN / inf -> +inf, which orders above everything
    worst = fmaxf(worst, rs);
  }
  // Only the norm passes between workgroups, by atomics: each is waited for ahead of the count.  A fence would write T back from
  // the caches, 400 us.
  if (lane == 0) {
    const int before = atomicMax(reinterpret_cast<int *>(g.err + b), __float_as_int(worst));   // >= 0: int order = float order
    asm volatile("" :: "v"(before) : "memory");
  }
  __syncthreads();
  if (threadIdx.x == 0 && atomicAdd(g.arrived + b, 1) == (int)gridDim.x - 1) {
    const float e = __int_as_float(atomicExch(reinterpret_cast<int *>(g.err + b), 0));
    g.arrived[b] = 0;
    newton_check(g, b, e);
  }
}

struct NewtonFinishArgs {
  const float *X[2]; float *x; int64_t x_stride;       // X_k of even k and of odd k
  const int32_t *failed; int32_t *failed_out; unsigned long long *fail_count;
  const int32_t *iters; int32_t *iters_out;
  int32_t n;
};

// grid (ceil(n / NEWTON_ROWS), batch), behind the last iteration: a matrix whose iteration ended at k
// copies X_k into the output (unless it failed) and reports its status.
__global__ __launch_bounds__(256) void newton_finish_kernel(const NewtonFinishArgs g) {
  const int b = blockIdx.y, n = g.n, tid = threadIdx.x;
  const int bad = g.failed[b], k = g.iters[b];
  if (blockIdx.x == 0 && tid == 0) {
    if (g.failed_out) g.failed_out[b] = bad;
    if (g.iters_out) g.iters_out[b] = k;
    if (bad && g.fail_count) atomicAdd(g.fail_count, 1ull);
  }
  if (bad) return;
  const int64_t first = (int64_t)blockIdx.x * NEWTON_ROWS * n, last = min(first + (int64_t)NEWTON_ROWS * n, (int64_t)n * n);
  const float *X = g.X[k & 1] + (int64_t)b * n * n;
  float *x = g.x + (int64_t)b * g.x_stride;
#pragma unroll 4
  for (int64_t e = first + tid; e < last; e += 256) x[e] = X[e];
}


// Matrices of up to 128: the whole iteration in one launch, a workgroup per matrix and a wavefront per 32 x 32 tile on or
// below the diagonal.  Launch by launch such a root is 400 launches whatever its size (2.4 ms), nine of ten of them for
// nothing.  M and X stay in registers, as tiles of MFMA results; the operands of a product go through LDS, mirrored and along
// k (two matrices of 128 fill it).  With E = (I - M) / p, which is exact, X' = X + X E and M' = M + ((I + E)^p - I) M: a product rounds
// at the size of E, not of T = I + E.  Products on the float32 matrix cores, in two accumulators that take turns.  From 97 on ten wavefronts leave
// 168 registers to each, 35 too few: they spill between the products, not in them (with four accumulators 90; 2048 of 128 2.3 ms, 1.6 so).
// One matrix of 64 x 64 2.37 ms in 400 launches, 0.056 so, of 128 x 128 2.36 and 0.18 ms; 2048 of them 3.02 and 0.33, 7.8 and 1.6 ms.
// Bound by the chain of four products an iteration, which many matrices of 64 and all larger ones make on matrix cores that
// are not evenly loaded (10 tiles on 4 SIMDs).  Errors against float64 0.14 to 0.77 of those of the launches.  From 129 on
// two matrices do not fit into LDS.
struct NewtonSmallArgs {
  const float *a; float *x;             // [batch][n][n]
  int32_t *iters_out, *failed_out; unsigned long long *fail_count;      // any may be nullptr
  int32_t n, p, max_iter;
  float epsilon, scale, tol;
};
// A call that allows a single iteration gains too: one matrix of 128 61 -> 37 us, 2048 of them 744 -> 382, 2048 of 32 110 -> 24.
constexpr int NEWTON_SMALL = 128;

// NB = ceil(n / 32).  Workgroups: matrices.
template <int NB> __global__ __launch_bounds__(32 * NB * (NB + 1)) void newton_small_kernel(const NewtonSmallArgs g) {
  constexpr int W = NB * (NB + 1) / 2, NR = 32 * NB, LD = NR + 4;       // rows of a matrix in LDS four banks apart
  __shared__ __align__(16) float sh[2][NR * LD];
  __shared__ float rows[(NB + 1) * NR];
  __shared__ double red[W];
  __shared__ int bads[W];
  const int b = blockIdx.x, n = g.n, tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int ti = 0;
  while (w >= (ti + 1) * (ti + 2) / 2) ++ti;
  const int tj = w - ti * (ti + 1) / 2, half = lane >> 5, l32 = lane & 31;
  // element v of a lane's tile: row i0 + 8 (v / 4) + v % 4, column j
  const int i0 = 32 * ti + 4 * half, j = 32 * tj + l32;
  auto row_of = [&](int v) { return i0 + 8 * (v >> 2) + (v & 3); };
  // The tile and its mirror image into LDS.  A tile on the diagonal reads its own back, and what lies above the diagonal becomes what
  // lies below.
  auto put = [&](float *s, float (&x)[16]) {
    float *down = s + i0 * LD + j, *across = s + j * LD + i0;
#pragma unroll
    for (int v = 0; v < 16; ++v) down[(8 * (v >> 2) + (v & 3)) * LD] = x[v];
    if (ti != tj) {
#pragma unroll
      for (int q = 0; q < 4; ++q) *reinterpret_cast<float4 *>(across + 8 * q) = make_float4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]);
      return;
    }
    wavefront_order();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 t = *reinterpret_cast<const float4 *>(across + 8 * q);
      const float m[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) x[4 * q + e] = i0 + 8 * q + e >= j ? x[4 * q + e] : m[e];
    }
    wavefront_order();
#pragma unroll
    for (int v = 0; v < 16; ++v) down[(8 * (v >> 2) + (v & 3)) * LD] = x[v];
  };
  // The tile of A B, both symmetric.  A lane's four values of k are those of four MFMAs.
  const int steps = (n + 7) / 8;         // zeros behind
  auto product = [&](const float *A, const float *B, float (&out)[16]) {
    const float *pa = A + (32 * ti + l32) * LD + 4 * half, *pb = B + (32 * tj + l32) * LD + 4 * half;
    floatx16 acc[2];
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[e][v] = 0.f;
    for (int q = 0; q < steps; ++q) {
      const float4 x = *reinterpret_cast<const float4 *>(pa + 8 * q), y = *reinterpret_cast<const float4 *>(pb + 8 * q);
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, y.x, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, y.y, acc[1], 0, 0, 0);
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.z, y.z, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.w, y.w, acc[1], 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) out[v] = acc[0][v] + acc[1][v];
  };

  // A = scale * sym(L) + eps I, its norm, M_0 and X_0 as newton_init_kernel
  const float *a = g.a + (int64_t)b * n * n;
  int bad = 0;
  for (int i = w; i < NR; i += W)
    for (int c = lane; c < NR; c += 64) {
      const float x = i < n && c < n ? a[(int64_t)i * n + c] : 0.f;
      if (!(fabsf(x) <= 3.0e38f)) bad = 1;
      sh[0][i * LD + c] = x;
    }
  __syncthreads();
  float M[16], X[16], E[16];             // E = (I - M) / p = T - I
  double val[16], ss = 0.0;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int i = row_of(v);
    val[v] = (double)g.scale * 0.5 * ((double)sh[0][i * LD + j] + (double)sh[0][j * LD + i]);
    if (i == j && i < n) val[v] += (double)g.epsilon;
    ss += (i > j ? 2.0 : i == j ? 1.0 : 0.0) * (val[v] * val[v]);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) { ss += __shfl_xor(ss, off, 64); bad |= __shfl_xor(bad, off, 64); }
  if (lane == 0) { red[w] = ss; bads[w] = bad; }
  __syncthreads();
  double fro = 0.0;
  bad = 0;
#pragma unroll
  for (int i = 0; i < W; ++i) { fro += red[i]; bad |= bads[i]; }
  fro = sqrt(fro);
  const double cp = 2.0 * fro / ((double)g.p + 1.0);           // c^p
  int failed = bad || !(cp > 0.0 && cp <= 1.0e300), iters = 0;
  if (!failed) {
    const double inv_cp = 1.0 / cp;
#pragma unroll
    for (int v = 0; v < 16; ++v) M[v] = (float)(val[v] * inv_cp);
    __builtin_amdgcn_sched_barrier(0);
    const float inv_c = (float)pow(cp, -1.0 / (double)g.p), pp = (float)g.p, inv_p = 1.f / pp;
    float prev = 3.0e38f;
#pragma unroll
    for (int v = 0; v < 16; ++v) X[v] = row_of(v) == j && j < n ? inv_c : 0.f;
    for (int k = 0;; ++k) {
#pragma unroll
      for (int v = 0; v < 16; ++v) E[v] = ((row_of(v) == j && j < n ? 1.f : 0.f) - M[v]) * inv_p;
      __syncthreads();                   // the reads before
      put(sh[0], E);
      put(sh[1], X);
      __syncthreads();
      // ||M - I||_inf = p ||E||_inf: NB + 1 threads a row, then all rows in every wavefront, so that all of them decide alike
      const int r = tid % NR, part = tid / NR;
      float rs = 0.f;
      for (int c = part; c < NR / 4; c += NB + 1) {
        const float4 q = *reinterpret_cast<const float4 *>(sh[0] + r * LD + 4 * c);
        rs += (fabsf(q.x) + fabsf(q.y)) + (fabsf(q.z) + fabsf(q.w));
      }
      rows[part * NR + r] = rs;
      __syncthreads();
      float e = 0.f;
#pragma unroll
      for (int i = lane; i < NR; i += 64) {
        float sum = 0.f;
#pragma unroll
        for (int q = 0; q <= NB; ++q) sum += rows[q * NR + i];
        if (!(sum <= 3.0e38f)) sum = __int_as_float(0x7f800000);
        e = fmaxf(e, sum);
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) e = fmaxf(e, __shfl_xor(e, off, 64));
      e *= pp;
      // the tests of newton_check
      failed = !(e <= 3.0e38f);
      iters = k;
      if (failed || e < g.tol || k >= g.max_iter || (prev < 0.1f && e > 0.5f * prev)) break;
      prev = e;
      float out[16];
      if (k > 0) product(sh[1], sh[0], out);
#pragma unroll
      for (int v = 0; v < 16; ++v) X[v] += k > 0 ? out[v] : inv_c * E[v];
      if (e <= 1.f && e * e < g.tol) { iters = k + 1; break; }
      if (g.p == 1) {
        __syncthreads();
        put(sh[1], M);
      } else {
        product(sh[0], sh[0], out);
#pragma unroll
        for (int v = 0; v < 16; ++v) E[v] = 2.f * E[v] + out[v];          // (I + E)^2 - I, and so on
        __syncthreads();
        put(sh[1], E);
        put(sh[0], M);
        for (int q = 4; q <= g.p; q *= 2) {
          __syncthreads();
          product(sh[1], sh[1], out);
#pragma unroll
          for (int v = 0; v < 16; ++v) E[v] = 2.f * E[v] + out[v];
          __syncthreads();
          put(sh[1], E);
        }
      }
      __syncthreads();
      product(sh[1], sh[0], out);
#pragma unroll
      for (int v = 0; v < 16; ++v) M[v] += out[v];
    }
  }
  if (tid == 0) {
    if (g.failed_out) g.failed_out[b] = failed;
    if (g.iters_out) g.iters_out[b] = iters;
    if (failed && g.fail_count) atomicAdd(g.fail_count, 1ull);
  }
  if (failed) return;
  __syncthreads();
  put(sh[0], X);
  __syncthreads();
  float *x = g.x + (int64_t)b * n * n;
  for (int i = w; i < n; i += W)
    for (int c = lane; c < n; c += 64) x[(int64_t)i * n + c] = sh[0][i * LD + c];
}

inline void launch_newton_small(const NewtonSmallArgs &g, int batch, hipStream_t s) {
  const dim3 grid(batch);
  switch ((g.n + 31) / 32) {
    case 1: hipLaunchKernelGGL(newton_small_kernel<1>, grid, dim3(64), 0, s, g); break;
    case 2: hipLaunchKernelGGL(newton_small_kernel<2>, grid, dim3(192), 0, s, g); break;
    case 3: hipLaunchKernelGGL(newton_small_kernel<3>, grid, dim3(384), 0, s, g); break;
    default: hipLaunchKernelGGL(newton_small_kernel<4>, grid, dim3(640), 0, s, g); break;
  }
}

}  // namespace shampoo
