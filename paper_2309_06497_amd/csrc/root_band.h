// Root inverse of matrices of 128 < n <= 2048 without eigenvectors, batched.
//
//   A = Q B Q^T       blocked Householder reduction to a symmetric band matrix B of 32-wide blocks, in
//                     float64 on the fp64 matrix cores: per panel a QR factorisation (one workgroup per
//                     matrix, panel in registers), Z = W V, Y = Z T - V (T^T V^T Z T) / 2 and
//                     W <- W - V Y^T - Y V^T
//   F = f(B)          f(x) = (x - min(lambda_min, 0) + eps)^-r as a sum of inverses of B + sigma_j
//                     (root_rational.h).  B is block tridiagonal, so an inverse is one elimination along
//                     the blocks (a wavefront per matrix and shift), and every block row of it runs from
//                     its diagonal block to the left by one 32 x 32 product per block
//   X = Q F Q^T       the same reflectors from both sides, last panel first, four panels at a time as one
//                     block reflector of 128 columns: on the way back all of them are known, and a pass over
//                     F then costs 128 multiply-adds per element read instead of 32.  Products with the
//                     batched float32 GEMM (gemm_mfma.h)
//
// The block Jacobi solver (eigh_jacobi.h) needs 10 ... 13 sweeps of 6 n^3 multiply-adds for the
// eigenvectors; this takes about 2 n^3 for the reduction, 1 n^3 for F and 2 n^3 on the way back, and
// nothing in it iterates except the bisection of a negative or tiny smallest eigenvalue.  Jacobi
// still serves callers that want eigenvalues or keep eigenvectors between calls, larger matrices, and
// exponents without a rational fit.
//
// Accuracy: the reduction is backward stable in float64 (eigenvalues move by 1e-16 of the largest, as
// in the float64 sweeps), the inverses are float64; F, the reflectors of the way back and the results of its products
// are float32, like the accumulated rotations and the reconstruction of the Jacobi path, the sums in them float64 (but for
// the update of F from n = 513 on).
//
// Layouts of v_mfma_f64_16x16x4_f64: lane l supplies A(l % 16, l / 16) and B(l / 16, l % 16), element v
// of the result is D(l / 16 + 4 v, l % 16); v_mfma_f32_16x16x4_f32: the same operands, D(4 (l / 16) + v,
// l % 16).  The order of k inside a sum is free, so a result can be the B operand of the next product as
// it stands (step v takes the rows that element v holds), and a symmetric one the A operand too.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "gemm_mfma.h"
#include "group.h"
#include "lds_dma.h"
#include "root_rational.h"
#include "root_tridiag.h"

namespace shampoo {

constexpr int BAND = 32;                 // block size: half bandwidth of B
constexpr int BAND_MAX_N = 2048;
constexpr int BAND_SHIFTS = 32;          // shifts tried per round of the bisection
constexpr int BAND_ROUNDS = 12;          // 33^11 covers 2^53
constexpr int BAND_ROWS = 128;           // rows per workgroup of Y and of the rank-64 update
constexpr int BAND_ZROWS = 64;           // rows per workgroup of Z = W V
constexpr int BAND_COLS = 128;           // columns per workgroup of the rank-64 update
constexpr int BAND_GROUP = 4;            // panels per block reflector of the way back
constexpr int BAND_GW = BAND_GROUP * BAND;   // its columns
constexpr int BAND_PLD = 3 * BAND_GW;    // row of its work array: Z, later Y | V | Y
constexpr int BAND_SLOTS = RAT_MAX_POLES + 1;   // eliminations of B + shift: one per pole and one for the eigenvector

typedef double band_d4 __attribute__((ext_vector_type(4)));
typedef float band_f4 __attribute__((ext_vector_type(4)));

struct BandMeta {
  double dec_min, hi, amax;              // smallest diagonal entry of the rows that stand alone; bounds of the spectrum of B
  double lo[2], up[2];                   // bracket of the smallest eigenvalue of B, by parity of the round
  double base, low, shift, f1, lam;      // eps - shift; lower end of the rational sum's range; min(lambda_min, 0); f(lam); lambda_min of B
  int32_t skip;                          // 0: go on; 1: failed; 2: not asked for
  int32_t coupled, cls, poles, deflate;
  int32_t active[2];                     // bisection still running, by parity of the round
};

struct BandArgs {
  const float *a; int32_t n, np, nb;     // input [n][n]; padded size, number of blocks
  float eps, r, scale;
  float *x; int32_t *failed_user; unsigned long long *fail_count; const int32_t *only;
  BandMeta *meta;
  double *w;        // [np][np]: the matrix being reduced, in the 32 x 32 blocks on and below the diagonal
  float *f;         // [np][np], in the memory of w: F, then X
  double *vp, *z, *y, *t, *part;         // current panel: V, Z, Y [np][32], T [32][32], partial sums of V^T Z [np / 64][32][32]
  float *vall, *tall;                    // all panels: V [np][np], panel k in columns 32 k ...; T [nb - 1][32][32]
  double *dblk, *cblk;                   // B: diagonal blocks [nb][32][32], transposed sub-diagonal blocks [nb][32][32]
  double *kf, *gf;                       // per slot and block: -K^T (A operand order) and weight * G (D order), [BAND_SLOTS][nb][1024]
  double *v1;                            // [np]: eigenvector handled by itself
  int32_t *ok;                           // [2][BAND_SHIFTS]: verdicts of the bisection, by parity of the round
  int32_t *dec;                          // [np]: row is coupled to no other
  int32_t *skip;                         // meta->skip != 0, back to back for the products of the way back
};
// Matrices of one size in a launch (group.h): several sizes go through the same launches, each at its own panel.
struct BandJob {
  BandArgs g;
  int32_t k, cnt;                        // panel, group of panels or round; number of matrices
  __device__ __forceinline__ void globals() {
    to_global(g.a, g.x, g.failed_user, g.fail_count, g.only, g.meta, g.w, g.f, g.vp, g.z, g.y, g.t, g.part, g.vall, g.tall, g.dblk, g.cblk, g.kf, g.gf,
              g.v1, g.ok, g.dec, g.skip);
  }
};
constexpr int BAND_TABLE_RESERVE = sizeof(RatTable) + 16;      // of a launch's arguments, where the weights go along
typedef Group<BandJob> BandJobs;
typedef Group<BandJob, BAND_TABLE_RESERVE> BandTableJobs;
// the job of a workgroup, the matrix and the workgroup's index among the PER of a matrix
#define BAND_PICK(PER)                                                     \
  int wg;                                                                  \
  const BandJob job = group_pick(grp, wg);                                 \
  BandArgs g = job.g;                                                      \
  const int k = job.k, per_ = (PER), b = wg / per_, bx = wg - b * per_;    \
  (void)k; (void)bx;                                                       \
  if (b >= job.cnt) return;
// rows and workgroups of a panel's products
__host__ __device__ inline int band_left(const BandArgs &g, int k) { return g.np - (k + 1) * BAND; }
__host__ __device__ inline int band_row_wgs(const BandArgs &g, int k) { const int m = band_left(g, k); return (m + BAND_ROWS - 1) / BAND_ROWS; }
__host__ __device__ inline int band_z_wgs(const BandArgs &g, int k) { const int m = band_left(g, k); return (m + BAND_ZROWS - 1) / BAND_ZROWS; }
__host__ __device__ inline int band_col_wgs(const BandArgs &g, int k) { const int m = band_left(g, k); return (m + BAND_COLS - 1) / BAND_COLS; }
__host__ __device__ inline int band_groups(const BandArgs &g) { return (g.nb - 1 + BAND_GROUP - 1) / BAND_GROUP; }
// Arrays of the way back, in the memory of kf and gf, which nothing reads any more by then: the work array
// [np][BAND_PLD] of a group of panels; [T^T; -T M T^T / 2] as a [256][128] matrix; T [groups][128][128].
__host__ __device__ inline float *band_p(const BandArgs &g) { return reinterpret_cast<float *>(g.kf); }
__host__ __device__ inline float *band_ts(const BandArgs &g) { return reinterpret_cast<float *>(g.gf); }
__host__ __device__ inline float *band_tg(const BandArgs &g) { return band_ts(g) + 2 * BAND_GW * BAND_GW; }
__host__ __device__ inline int64_t band_p_stride(const BandArgs &g) { return (int64_t)g.nb * 1024 * BAND_SLOTS * 2; }   // matrix to matrix, floats
// room for them: 1536 of 9472 bytes per row, and (2 + groups) 64 KB of 9472 bytes per row from 5 blocks on
static_assert(BAND_PLD * 4 <= 32 * 8 * BAND_SLOTS && (2 + 2) * BAND_GW * BAND_GW * 4 <= 5 * 1024 * 8 * BAND_SLOTS, "way back");

// from the arrays of matrix 0 of the batch to those of matrix b (failed_user and only stay: they are indexed)
__host__ __device__ inline void band_select(BandArgs &g, int b) {
  const int64_t np = g.np, nb = g.nb;
  g.a += (int64_t)b * g.n * g.n; g.x += (int64_t)b * g.n * g.n;
  g.meta += b;
  g.w += b * np * np; g.f += b * np * np * 2;
  g.vp += b * np * BAND; g.z += b * np * BAND; g.y += b * np * BAND; g.t += (int64_t)b * 1024;
  const int64_t parts = (np + BAND_ZROWS - 1) / BAND_ZROWS;
  g.part += b * parts * 1024;
  g.vall += b * np * np; g.tall += b * nb * 1024;
  g.dblk += b * nb * 1024; g.cblk += b * nb * 1024;
  g.kf += b * nb * 1024 * BAND_SLOTS; g.gf += b * nb * 1024 * BAND_SLOTS;
  g.v1 += b * np; g.ok += b * 2 * BAND_SHIFTS; g.dec += b * np; g.skip += b;
}

__device__ __forceinline__ band_d4 band_mfma(double a, double b, band_d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ __forceinline__ band_f4 band_mfma(float a, float b, band_f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ int band_row(int lg, int v) { return lg + 4 * v; }   // of element v of a band_d4

// ---------------------------------------------------------------------------
// W = pad(sym(scale A)); which rows stand alone.  workgroups: np / 32 per matrix, 256 threads
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void band_init_kernel(const BandJobs grp) {
  __shared__ float Xs[BAND][BAND + 1], Ys[BAND][BAND + 1];
  __shared__ int coupled[BAND];
  BAND_PICK(g.nb)
  const int br = bx, tid = threadIdx.x, r = tid >> 3, c4 = (tid & 7) * 4;
  const int32_t *only = g.only;
  band_select(g, b);
  if (only && only[b] == 0) {
    if (br == 0 && tid == 0) g.meta->skip = 2;
    return;
  }
  const int n = g.n, np = g.np;
  if (tid < BAND) coupled[tid] = 0;
  {                                      // rows above a panel's first are zero in V
    float4 *v = reinterpret_cast<float4 *>(g.vall + (int64_t)br * BAND * np);
    for (int e = tid; e < BAND * np / 4; e += 256) v[e] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  const int gi = br * BAND + r;
  int bad = 0, any = 0;
  for (int bc = 0; bc < g.nb; ++bc) {
    const int yi = bc * BAND + r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int xj = bc * BAND + c4 + e, yj = br * BAND + c4 + e;
      const float x = (gi < n && xj < n) ? g.a[(int64_t)gi * n + xj] : 0.f;
      const float y = (yi < n && yj < n) ? g.a[(int64_t)yi * n + yj] : 0.f;
      if (!(fabsf(x) <= 3.0e38f)) bad = 1;
      Xs[r][c4 + e] = x;
      Ys[r][c4 + e] = y;
    }
    __syncthreads();
    double v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = (double)g.scale * (0.5 * ((double)Xs[r][c4 + e] + (double)Ys[c4 + e][r]));
      if (gi != bc * BAND + c4 + e && v[e] != 0.0) any = 1;
    }
    if (bc <= br) {
      double2 *dst = reinterpret_cast<double2 *>(g.w + (int64_t)gi * np + bc * BAND + c4);
      dst[0] = make_double2(v[0], v[1]); dst[1] = make_double2(v[2], v[3]);
    }
    __syncthreads();
  }
  if (any) coupled[r] = 1;
  if (bad) g.meta->skip = 1;
  __syncthreads();
  if (tid < BAND) g.dec[br * BAND + tid] = coupled[tid] ? 0 : 1;
}

// A row that is coupled to no other is an eigenvector by itself: its entry of the result is f of its
// diagonal entry.  It goes through the reduction, like the padding, with a diagonal entry from inside
// the spectrum of the rest.  a workgroup of 256 threads per matrix
__global__ __launch_bounds__(256) void band_alone_kernel(const BandJobs grp) {
  __shared__ double red[2][4];
  BAND_PICK(1)
  band_select(g, b);
  if (g.meta->skip) return;
  const int tid = threadIdx.x, n = g.n, np = g.np;
  double dmin = 1.0e300, fill = -1.0e300;
  for (int i = tid; i < n; i += 256) {
    const double v = g.w[(int64_t)i * np + i];
    if (g.dec[i]) dmin = fmin(dmin, v); else fill = fmax(fill, v);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) { dmin = fmin(dmin, __shfl_xor(dmin, off, 64)); fill = fmax(fill, __shfl_xor(fill, off, 64)); }
  if ((tid & 63) == 0) { red[0][tid >> 6] = dmin; red[1][tid >> 6] = fill; }
  __syncthreads();
  dmin = fmin(fmin(red[0][0], red[0][1]), fmin(red[0][2], red[0][3]));
  fill = fmax(fmax(red[1][0], red[1][1]), fmax(red[1][2], red[1][3]));
  const bool coupled = fill > -1.0e300;
  if (!coupled) fill = 1.0;
  for (int i = tid; i < np; i += 256)
    if (i >= n || g.dec[i]) g.w[(int64_t)i * np + i] = fill;
  if (tid == 0) { g.meta->dec_min = dmin; g.meta->coupled = coupled ? 1 : 0; }
}

// ---------------------------------------------------------------------------
// QR of panel k (rows 32 (k + 1) ... np - 1 of columns 32 k ... 32 k + 31): V, T, R; and D_k as it now is.
// One workgroup of 8 wavefronts per matrix, 16 columns at a time: lane (c = l % 16, ph = l / 16) of
// wavefront w holds rows 32 t + 4 w + ph of column c, t < TT, so that the entry of the pivot column of
// a row reaches the row's 16 columns by a DPP broadcast, which a multiply-add takes as an operand: one instruction per
// register for the scalar products of a column, one for the update.  So that the update is that simple, the pivot column
// stays as it is and becomes the reflector, by one factor, when all 16 are done.  The entries are MFMA operands as they lie.
// Per column one barrier.  Two wavefronts per SIMD: the panel of 2048 rows takes 128 of 256 registers (four
// wavefronts with half as many rows each spilled up to 247 of 128).
// 8 panels of 2016 rows beside 8 others: 287 us with 16 wavefronts, 126 with 8, 96 with the next reads of V on their way and the first
// reflectors applied on the matrix cores (44 of the 126 us, 22 of the 96); 32 of 992 rows 152, 90 and 67 us.  With 4
// wavefronts, one per SIMD, and twice the rows in each, the columns take as long and the reads longer.
// The other matrices of the batch run beside it, other sub-chunks' products too.
// ---------------------------------------------------------------------------
constexpr int BAND_QR_WAVES = 8, BAND_QR_THREADS = 64 * BAND_QR_WAVES;

// d[i] += (lane J of the row's x[i]) * x[i], i < 4.  A register that the DPP operand reads must not have been written by
// the two instructions before.
template <int J> __device__ __forceinline__ void row16_dot4(double (&d)[4], double x0, double x1, double x2, double x3) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %4, %4 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %5, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %6, %6 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %7, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf"
      : "+v"(d[0]), "+v"(d[1]), "+v"(d[2]), "+v"(d[3]) : "v"(x0), "v"(x1), "v"(x2), "v"(x3), "n"(J));
}
// x[i] += (lane J of the row's y[i]) * q; y may be x itself
template <int J> __device__ __forceinline__ void row16_update4(double &x0, double &x1, double &x2, double &x3, double q) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %0, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %1, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %3, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
      : "+v"(x0), "+v"(x1), "+v"(x2), "+v"(x3) : "v"(q), "n"(J));
}
template <int J> __device__ __forceinline__ void row16_fma(double &x, double y, double q) {
  asm("s_nop 1\n\tv_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(x) : "v"(y), "v"(q), "n"(J));
}
template <int J> __device__ __forceinline__ double row16_bcast(double x) { return dpp_fetch<0x150 + J>(x); }

// Elements of a lane in an array of `count` elements: lane address and scalar step.  With a step inside the array, what a lane
// asks for past its end is read as zero.
struct BandColumn {
  __amdgpu_buffer_rsrc_t r;
  int lane;
  __device__ __forceinline__ BandColumn(const void *base, int lane_, int count, int size)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(uniform_ptr(base)), 0, count * size, 0x00020000)), lane(lane_ * size) {}
  __device__ __forceinline__ double get(int at) const {
    typedef uint32_t pair __attribute__((ext_vector_type(2)));
    const pair x = __builtin_amdgcn_raw_buffer_load_b64(r, lane, at * 8, 0);
    return __hiloint2double((int)x[1], (int)x[0]);
  }
  __device__ __forceinline__ band_d4 get4(int at) const {         // at a multiple of 16 bytes
    const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, lane, at * 8, 0), y = __builtin_amdgcn_raw_buffer_load_b128(r, lane + 16, at * 8, 0);
    return (band_d4){__hiloint2double((int)x[1], (int)x[0]), __hiloint2double((int)x[3], (int)x[2]), __hiloint2double((int)y[1], (int)y[0]),
                     __hiloint2double((int)y[3], (int)y[2])};
  }
  __device__ __forceinline__ void put(int at, double v) const {
    typedef uint32_t pair __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(pair{(uint32_t)__double2loint(v), (uint32_t)__double2hiint(v)}, r, lane, at * 8, 0);
  }
  __device__ __forceinline__ void put(int at, float v) const { __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, lane, at * 4, 0); }
};

struct BandQrShared {
  double red[2][BAND_QR_WAVES][16], prow[2][16], tau[BAND];
  double big[BAND_QR_WAVES][256];        // one 16 x 16 tile per wavefront
  double s[16][17], t[2][16][17], g01[16][17];
};

template <int TT>
__global__ __launch_bounds__(BAND_QR_THREADS) void band_qr_kernel(const BandJobs grp) {
  static_assert(TT % 4 == 0, "registers by fours");
  __shared__ BandQrShared sh;
  BAND_PICK(1)
  band_select(g, b);
  if (g.meta->skip) return;
  const int np = g.np, tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 15, ph = lane >> 4;
  const int r0 = (k + 1) * BAND, m = np - r0;
  for (int x = tid; x < 1024; x += BAND_QR_THREADS) g.dblk[(int64_t)k * 1024 + x] = g.w[(int64_t)(k * BAND + (x >> 5)) * np + k * BAND + (x & 31)];
  if (m <= 0) return;
  const int tt = m / BAND;               // row blocks of 32: np is a multiple
  const int rel0 = 4 * w + ph;           // row of register t: rel0 + 32 t
  // The panel's columns in W, V and all of V: a lane's address, plus a scalar that steps from register to register (64 vector
  // addresses, held over both halves, cost more registers than the panel).  Of V also the rows of four registers as an MFMA
  // operand (row c of those 16, four columns).
  const BandColumn wcol(g.w + (int64_t)r0 * np + k * BAND, rel0 * np + c, m * np - k * BAND, 8),
      vcol(g.vp + (int64_t)r0 * BAND, rel0 * BAND + c, m * BAND, 8), vrow(g.vp + (int64_t)r0 * BAND, ((c >> 2) * BAND + 4 * w + (c & 3)) * BAND + 4 * ph, m * BAND, 8),
      acol(g.vall + (int64_t)r0 * np + k * BAND, rel0 * np + c, m * np - k * BAND, 4);
  double P[TT];
  int buf = 0;

  // f(batch, what load(batch) returned) for the batches of four registers that hold rows, the next DEPTH batches' loads ahead of it.
  // With one batch at a time, and none ahead, this kernel spent half of its time here (2048 rows).
  auto by_fours = [&](auto load, auto f) {
    constexpr int B = TT / 4, DEPTH = 2;
    decltype(load(0)) x[DEPTH + 1];
#pragma unroll
    for (int q = 0; q < DEPTH; ++q) if (q < B && 4 * q < tt) x[q] = load(q);
    for_each_block<B>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      if (4 * q < tt) {
        if constexpr (q + DEPTH < B) if (4 * (q + DEPTH) < tt) x[(q + DEPTH) % (DEPTH + 1)] = load(q + DEPTH);
        __builtin_amdgcn_sched_barrier(0);
        f(qc, x[q % (DEPTH + 1)]);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
  };
  auto v0_of = [&](int q) {
    band_d4 x;
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = vcol.get(min(4 * q + u, tt - 1) * BAND * BAND);   // rows past the end meet a zero in P
    return x;
  };
  // sum over the wavefronts of a 16 x 16 tile held as MFMA results: to sum[i][j]
  auto tile_sum = [&](band_d4 acc, double (*sum)[17]) {
#pragma unroll
    for (int v = 0; v < 4; ++v) sh.big[w][(ph + 4 * v) * 16 + c] = acc[v];
    __syncthreads();
    if (tid < 256) {
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < BAND_QR_WAVES; ++i) s += sh.big[i][tid];
      sum[tid >> 4][tid & 15] = s;
    }
    __syncthreads();
  };

#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      P[t] = 0.0;
      if (t < tt) P[t] = wcol.get(t * BAND * np + 16 * h);
    }
    if (h == 1) {                        // the reflectors of the first 16 columns:  C <- C - V0 (T0^T V0^T C)
      band_d4 acc = {0.0, 0.0, 0.0, 0.0};
      by_fours(v0_of, [&](auto qc, const band_d4 &v) {
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = band_mfma(v[u], P[4 * decltype(qc)::value + u], acc);
      });
      tile_sum(acc, sh.s);
      double sw[4];                      // -T0^T V0^T C, rows 4 ph ...
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        double e = 0.0;
#pragma unroll 4
        for (int l = 0; l < 16; ++l) e -= sh.t[0][l][4 * ph + u] * sh.s[l][c];
        sw[u] = e;
      }
      by_fours([&](int q) { return vrow.get4(4 * q * BAND * BAND); }, [&](auto qc, const band_d4 &v) {
        constexpr int t = 4 * decltype(qc)::value;
        band_d4 x = {P[t], P[t + 1], P[t + 2], P[t + 3]};
#pragma unroll
        for (int u = 0; u < 4; ++u) x = band_mfma(v[u], sw[u], x);
#pragma unroll
        for (int u = 0; u < 4; ++u) P[t + u] = x[u];
      });
    }
    double mine = 0.0;                   // the factor that makes a reflector of this lane's column
    for_each_block<16>([&](auto jj) {
      constexpr int J = decltype(jj)::value;
      const int pr = 16 * h + J;         // pivot row
      double d[4] = {0.0, 0.0, 0.0, 0.0};
      {
        const double x = rel0 > pr ? P[0] : 0.0;
        row16_dot4<J>(d, x, P[1], P[2], P[3]);
      }
#pragma unroll
      for (int t = 4; t < TT; t += 4)
        if (t < tt) row16_dot4<J>(d, P[t], P[t + 1], P[t + 2], P[t + 3]);
      const double dot = rows_sum((d[0] + d[1]) + (d[2] + d[3]));
      if (lane < 16) sh.red[buf][w][c] = dot;
      if (rel0 == pr) sh.prow[buf][c] = P[0];
      __syncthreads();
      double part[BAND_QR_WAVES];
#pragma unroll
      for (int i = 0; i < BAND_QR_WAVES; ++i) part[i] = sh.red[buf][i][c];
      const double s = ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
      static_assert(BAND_QR_WAVES == 8, "sum");
      const double sj = row16_bcast<J>(s), x0 = sh.prow[buf][J], pc = sh.prow[buf][c];
      buf ^= 1;
      double tau = 0.0;
      if (sj > TRI_NO_COLUMN) {
        // 1 / |v0|, v0 = x0 -+ norm, starts from the estimate of the norm, beside the steps that refine it (as rsqrt_newton and rcp_newton)
        const double nn = sj + x0 * x0, h2 = 0.5 * nn;
        double rn = __builtin_amdgcn_rsq(nn), r0 = __builtin_amdgcn_rcp(fabs(x0) + nn * rn);
        rn = rn * (1.5 - h2 * (rn * rn)); rn = rn * (1.5 - h2 * (rn * rn));
        const double norm = nn * rn, av = fabs(x0) + norm;
        r0 = r0 * (2.0 - av * r0); r0 = r0 * (2.0 - av * r0);
        const double alpha = x0 > 0.0 ? -norm : norm, inv = x0 > 0.0 ? r0 : -r0;
        tau = av * rn;
        const double zc = c > J ? s * inv + pc : 0.0, wc = tau * zc, q = (x0 > 0.0 ? -rn : rn) * zc;    // q = -wc / v0
        if (c == J) mine = inv;
        double x = rel0 > pr ? P[0] : 0.0;
        const double x1 = x;
        row16_fma<J>(x, x1, q);
        P[0] = rel0 > pr ? x : rel0 == pr ? (c == J ? alpha : P[0] - wc) : P[0];
        row16_update4<J>(x, P[1], P[2], P[3], q);      // x: not used any more
#pragma unroll
        for (int t = 4; t < TT; t += 4)
          if (t < tt) row16_update4<J>(P[t], P[t + 1], P[t + 2], P[t + 3], q);
      }
      if (tid == 0) sh.tau[pr] = tau;
    });
    // R (rows up to the pivot's) and V out; what is left in P is V
    g.cblk[(int64_t)k * 1024 + (16 * h + c) * BAND + rel0] = rel0 <= 16 * h + c ? P[0] : 0.0;
    P[0] = rel0 > 16 * h + c ? P[0] * mine : rel0 == 16 * h + c ? 1.0 : 0.0;
    band_d4 acc = {0.0, 0.0, 0.0, 0.0}, acc01 = {0.0, 0.0, 0.0, 0.0};
    by_fours([&](int q) { return h == 1 ? v0_of(q) : (band_d4){0.0, 0.0, 0.0, 0.0}; }, [&](auto qc, const band_d4 &v0) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = 4 * decltype(qc)::value + u;
        const double v = t > 0 ? P[t] * mine : P[0];
        if (h == 1) acc01 = band_mfma(v0[u], v, acc01);
        acc = band_mfma(v, v, acc);
        if (t < tt) {
          vcol.put(t * BAND * BAND + 16 * h, v);
          acol.put(t * BAND * np + 16 * h, (float)v);
        }
      }
    });
    tile_sum(acc, sh.s);
    // T of these 16 columns: T[i][j] = -tau_j sum_{i <= l < j} T[i][l] (v_l . v_j); lane i holds row i
    if (w == 0) {
      const double tau_c = sh.tau[16 * h + c];
      double T[16], e[16], sc[16];       // e[j]: the sum so far; sc[j]: (v_c . v_j)
#pragma unroll
      for (int j = 0; j < 16; ++j) { e[j] = 0.0; sc[j] = sh.s[c][j]; }
      for_each_block<16>([&](auto jc) {
        constexpr int J = decltype(jc)::value;
        const double tj = row16_bcast<J>(tau_c);
        T[J] = c == J ? tj : c < J ? -tj * e[J] : 0.0;
        for_each_block<15 - J>([&](auto d) { constexpr int j = J + 1 + decltype(d)::value; row16_fma<J>(e[j], sc[j], T[J]); });
      });
      if (lane < 16) {
#pragma unroll
        for (int j = 0; j < 16; ++j) sh.t[h][c][j] = T[j];
      }
    }
    __syncthreads();
    if (h == 1) tile_sum(acc01, sh.g01);
  }
  // T = [T0, -T0 (V0^T V1) T1; 0, T1]
  double e = 0.0;
  const int i = tid >> 4, j = tid & 15;
  if (tid < 256)
#pragma unroll
    for (int l = 0; l < 16; ++l) e += sh.g01[i][l] * sh.t[1][l][j];      // T: zeros below the diagonal
  __syncthreads();
  if (tid < 256) sh.s[i][j] = e;
  __syncthreads();
  if (tid < 256) {
    e = 0.0;
#pragma unroll
    for (int l = 0; l < 16; ++l) e -= sh.t[0][i][l] * sh.s[l][j];
    double *t = g.t;
    float *ta = g.tall + (int64_t)k * 1024;
    auto put = [&](int row, int col, double v) { t[row * BAND + col] = v; ta[row * BAND + col] = (float)v; };
    put(i, j, sh.t[0][i][j]); put(i, 16 + j, e); put(16 + i, j, 0.0); put(16 + i, 16 + j, sh.t[1][i][j]);
  }
}

// ---------------------------------------------------------------------------
// The panel products of the reduction: W22 <- H^T W22 H with H = I - V T V^T on rows and columns
// r0 ... np - 1, r0 = 32 (k + 1).
// ---------------------------------------------------------------------------
// Z = W[r0:, r0:] V[r0:] and, per workgroup, its rows' share of V^T Z.
// Workgroups: ceil((np - r0) / 64) per matrix, 8 wavefronts: 2 of 32 rows by 4 quarters of k, which meet in LDS, so that few
// matrices fill the GPU too.  Bound by memory and by the latency of its loads (every element of W is read once for 64
// multiply-adds).  What lies to the right of the diagonal blocks is read from its mirror image below them.
// 8 matrices of 2048 beside 8 others, the average panel: 118 us with 4 wavefronts of 32 rows over all of k, 38 so.
__global__ __launch_bounds__(512) void band_z_kernel(const BandJobs grp) {
  __shared__ double red[8][16 * 64];
  BAND_PICK(band_z_wgs(g, k))
  band_select(g, b);
  if (g.meta->skip) return;
  const int r0 = (k + 1) * BAND;
  const int np = g.np, tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lg = lane >> 4;
  const int rg = w & 1, kq = w >> 1, base = r0 + BAND_ZROWS * bx + BAND * rg;
  band_d4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = (band_d4){0, 0, 0, 0};
  if (base < np) {
    const int steps = (np - r0) / 16, s1 = steps * (kq + 1) / 4, diag = (base + BAND - r0) / 16;
    int s = steps * kq / 4;
    const double *vr = g.vp + (int64_t)(4 * lg) * BAND + li;
    auto product = [&](int k0, const band_d4 &a0, const band_d4 &a1) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double b0 = vr[(int64_t)(k0 + q) * BAND], b1 = vr[(int64_t)(k0 + q) * BAND + 16];
        acc[0][0] = band_mfma(a0[q], b0, acc[0][0]); acc[0][1] = band_mfma(a0[q], b1, acc[0][1]);
        acc[1][0] = band_mfma(a1[q], b0, acc[1][0]); acc[1][1] = band_mfma(a1[q], b1, acc[1][1]);
      }
    };
    const double *row = g.w + (int64_t)(base + li) * np + 4 * lg;         // a lane reads 4 consecutive k of its rows
#pragma unroll 2
    for (const int e = min(s1, diag); s < e; ++s) {
      const int k0 = r0 + 16 * s;
      product(k0, *reinterpret_cast<const band_d4 *>(row + k0), *reinterpret_cast<const band_d4 *>(row + (int64_t)16 * np + k0));
    }
    const double *col = g.w + (int64_t)(4 * lg) * np + base + li;         // or the same elements of a column
#pragma unroll 2
    for (; s < s1; ++s) {
      const int k0 = r0 + 16 * s;
      band_d4 a0, a1;
#pragma unroll
      for (int q = 0; q < 4; ++q) { a0[q] = col[(int64_t)(k0 + q) * np]; a1[q] = col[(int64_t)(k0 + q) * np + 16]; }
      product(k0, a0, a1);
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[w][((2 * i + j) * 4 + v) * 64 + lane] = acc[i][j][v];
  __syncthreads();
  // wavefront (rg, kq): the tile (kq / 2, kq % 2) of its rows, and what it gives to V^T Z
  const int rt = kq >> 1, j = kq & 1;
  band_d4 z, m0 = {0, 0, 0, 0}, m1 = {0, 0, 0, 0};
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int at = (4 * kq + v) * 64 + lane;
    z[v] = (red[rg][at] + red[2 + rg][at]) + (red[4 + rg][at] + red[6 + rg][at]);
  }
  if (base < np)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t at = (int64_t)(base + 16 * rt + band_row(lg, v)) * BAND + li;
      g.z[at + 16 * j] = z[v];
      m0 = band_mfma(g.vp[at], z[v], m0);
      m1 = band_mfma(g.vp[at + 16], z[v], m1);
    }
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    red[2 * rt + rg][band_row(lg, v) * BAND + 16 * j + li] = m0[v];
    red[2 * rt + rg][(16 + band_row(lg, v)) * BAND + 16 * j + li] = m1[v];
  }
  __syncthreads();
  for (int e = tid; e < 1024; e += 512) g.part[(int64_t)bx * 1024 + e] = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
}

// Y = Z T - V (T^T M T) / 2 with M = V^T Z.  Workgroups: ceil((np - r0) / 128) per matrix, 4 wavefronts of 32 rows.
__global__ __launch_bounds__(256) void band_y_kernel(const BandJobs grp) {
  __shared__ double M[BAND][BAND + 1], Tm[BAND][BAND + 1], S[BAND][BAND + 1];
  BAND_PICK(band_row_wgs(g, k))
  band_select(g, b);
  if (g.meta->skip) return;
  const int r0 = (k + 1) * BAND;
  const int np = g.np, tid = threadIdx.x, lane = tid & 63, w = tid >> 6, li = lane & 15, lg = lane >> 4;
  const int base = r0 + BAND_ROWS * bx + BAND * w;
  // The rows' own operands are requested with the first of the sums, eight of which are in flight: 8 matrices of 2048 beside 8 others, the
  // average panel, 17 us with four and the operands behind them, 12 so.
  band_d4 za[2][2], va[2][2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t at = (int64_t)(min(base, np - BAND) + 16 * rt + li) * BAND + 16 * h + 4 * lg;
      za[rt][h] = *reinterpret_cast<const band_d4 *>(g.z + at);
      va[rt][h] = *reinterpret_cast<const band_d4 *>(g.vp + at);
    }
  double tt[4], s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < 4; ++i) tt[i] = g.t[tid + 256 * i];
  for (int q = 0, parts = band_z_wgs(g, k); q < parts; q += 8) {
    double x[8][4];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[u][i] = g.part[(int64_t)min(q + u, parts - 1) * 1024 + tid + 256 * i];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) s[i] += q + u < parts ? x[u][i] : 0.0;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = tid + 256 * i;
    M[e >> 5][e & 31] = s[i];
    Tm[e >> 5][e & 31] = tt[i];
  }
  __syncthreads();
  const int ti = 16 * (w >> 1), tj = 16 * (w & 1);
  band_d4 acc = {0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < 8; ++s) acc = band_mfma(M[ti + li][4 * s + lg], Tm[4 * s + lg][tj + li], acc);
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 4; ++v) M[ti + band_row(lg, v)][tj + li] = acc[v];
  __syncthreads();
  acc = (band_d4){0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < 8; ++s) acc = band_mfma(Tm[4 * s + lg][ti + li], M[4 * s + lg][tj + li], acc);
#pragma unroll
  for (int v = 0; v < 4; ++v) S[ti + band_row(lg, v)][tj + li] = acc[v];
  __syncthreads();
  if (base >= np) return;
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    band_d4 zt[2], vs[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) { zt[j] = (band_d4){0, 0, 0, 0}; vs[j] = (band_d4){0, 0, 0, 0}; }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int kq = 16 * h + 4 * lg + q;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          zt[j] = band_mfma(za[rt][h][q], Tm[kq][16 * j + li], zt[j]);
          vs[j] = band_mfma(va[rt][h][q], S[kq][16 * j + li], vs[j]);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        g.y[(int64_t)(base + 16 * rt + band_row(lg, v)) * BAND + 16 * j + li] = zt[j][v] - 0.5 * vs[j][v];
  }
}

// W <- W - V Y^T - Y V^T on rows and columns r0 ..., up to the diagonal blocks.  workgroups: the square of
// ceil((np - r0) / 128) per matrix, 4 wavefronts of 32 rows, which keep their rows of V and Y in registers and walk along the
// columns together, 16 at a time.  Memory bound.  The whole square, a second copy of every element for Z to read,
// took 78 us for the average panel of 8 matrices of 2048 beside 8 others, this 51; 48 of 1024: 115 and 80.
__global__ __launch_bounds__(256) void band_update_kernel(const BandJobs grp) {
  BAND_PICK(band_row_wgs(g, k) * band_col_wgs(g, k))
  const int rows = band_row_wgs(g, k), by = bx / rows;
  band_select(g, b);
  if (g.meta->skip) return;
  const int r0 = (k + 1) * BAND;
  const int np = g.np, tid = threadIdx.x, lane = tid & 63, w = tid >> 6, li = lane & 15, lg = lane >> 4;
  const int base = r0 + BAND_ROWS * (bx - rows * by) + BAND * w;
  if (base >= np) return;
  const int c0 = r0 + BAND_COLS * by, c1 = min(c0 + BAND_COLS, base + BAND);
  if (c0 >= c1) return;
  band_d4 va[2][2], ya[2][2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int64_t at = (int64_t)(base + 16 * rt + li) * BAND + 16 * kk + 4 * lg;
      ya[rt][kk] = *reinterpret_cast<const band_d4 *>(g.y + at);
      va[rt][kk] = *reinterpret_cast<const band_d4 *>(g.vp + at);
    }
  for (int c = c0; c < c1; c += 16) {
    double *dst = g.w + (int64_t)base * np + c + li;
    double old[2][4];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int v = 0; v < 4; ++v) old[rt][v] = dst[(int64_t)(16 * rt + band_row(lg, v)) * np];
    band_d4 acc[2];
    acc[0] = (band_d4){0, 0, 0, 0}; acc[1] = (band_d4){0, 0, 0, 0};
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int64_t at = (int64_t)(c + li) * BAND + 16 * kk + 4 * lg;
      const band_d4 yb = *reinterpret_cast<const band_d4 *>(g.y + at), vb = *reinterpret_cast<const band_d4 *>(g.vp + at);
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) acc[rt] = band_mfma(va[rt][kk][q], yb[q], acc[rt]);
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) acc[rt] = band_mfma(ya[rt][kk][q], vb[q], acc[rt]);
    }
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int v = 0; v < 4; ++v) dst[(int64_t)(16 * rt + band_row(lg, v)) * np] = old[rt][v] - acc[rt][v];
  }
}

// ---------------------------------------------------------------------------
// The block tridiagonal matrix
// ---------------------------------------------------------------------------
// Gershgorin bounds of B.  a workgroup of 256 threads per matrix
__global__ __launch_bounds__(256) void band_bounds_kernel(const BandJobs grp) {
  __shared__ double red[2][4];
  BAND_PICK(1)
  band_select(g, b);
  if (g.meta->skip) return;
  const int tid = threadIdx.x, np = g.np;
  double hi = -1.0e300, amax = 0.0;
  for (int i = tid; i < np; i += 256) {
    const int blk = i >> 5, r = i & 31;
    const double *d = g.dblk + (int64_t)blk * 1024 + r * BAND;
    double off = 0.0;
    for (int c = 0; c < BAND; ++c) if (c != r) off += fabs(d[c]);
    if (blk > 0) for (int c = 0; c < BAND; ++c) off += fabs(g.cblk[(int64_t)(blk - 1) * 1024 + c * BAND + r]);
    if (blk + 1 < g.nb) for (int c = 0; c < BAND; ++c) off += fabs(g.cblk[(int64_t)blk * 1024 + r * BAND + c]);
    hi = fmax(hi, d[r] + off);
    amax = fmax(amax, fabs(d[r]) + off);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) { hi = fmax(hi, __shfl_xor(hi, off, 64)); amax = fmax(amax, __shfl_xor(amax, off, 64)); }
  if ((tid & 63) == 0) { red[0][tid >> 6] = hi; red[1][tid >> 6] = amax; }
  __syncthreads();
  if (tid == 0) {
    g.meta->hi = fmax(fmax(red[0][0], red[0][1]), fmax(red[0][2], red[0][3]));
    g.meta->amax = fmax(fmax(red[1][0], red[1][1]), fmax(red[1][2], red[1][3]));
  }
}

// Position of element (i, k) of -K^T in its stored order (A operand: lane l holds (l % 16, l / 16 + 4 v))
// and of element (r, c) of a block in result order.
__device__ __forceinline__ int band_a_index(int i, int k) { return ((((i >> 4) * 2 + (k >> 4)) * 4 + ((k & 15) >> 2)) << 6) + ((k & 3) << 4) + (i & 15); }
__device__ __forceinline__ int band_d_index(int r, int c) { return ((((r >> 4) * 2 + (c >> 4)) * 4 + ((r & 15) >> 2)) << 6) + ((r & 3) << 4) + (c & 15); }

// One block of the elimination, all of it in the registers of one wavefront as MFMA results:
//     M  pivot block (D_i + sigma I less what the blocks before took away)   ->  -M^-1
//     K  R^T, R the block that couples i + 1 to i                            ->  K^T = M^-1 R^T
//     S  D_i+1                                                                ->  D_i+1 - R M^-1 R^T
// by 32 pivots of the sweep operator on [M R^T; R S].  S is eliminated pivot by pivot (the stable
// Cholesky way); formed as a product with M^-1 it would lose the condition number of M in accuracy,
// which for a pivot block with a few large eigenvalues and many tiny ones is everything.
// Bound by the latency of a pivot: its row goes through LDS (64 doubles) and its reciprocal is a chain of its own.  So a pivot
// first updates the row of the next one, sends it and requests it; the rest of its update runs meanwhile, the next reciprocal
// in the second half of it, and the next block's D and R are requested half way through this one.
// 16 matrices of 2048, a launch of 256 chains of 64 blocks beside another: 615 us without that, 385 so; a lone chain of 32 blocks 278 and
// 157 us.  Two wavefronts per SIMD instead of three (248 registers) cost less than that gains also where thousands of chains run.
// Returns whether all pivots were positive.
// INVERSE = false: only that answer and S.  The rows that pivots have left behind are not turned into an inverse,
// and of the symmetric M and S only the three tiles on and above the diagonal are kept up: 27 instead of 48
// multiply-adds per lane and pivot.
struct BandElim {
  double M[2][2][4], K[2][2][4], S[2][2][4], nk[2][2][4], ns[2][2][4];   // nk, ns: R^T and D_i+1 of the block to come
  struct Row { double p, c[2], k[2], f[2][4], h[2][4]; };                // a pivot, and its row of [M K] by columns and by rows
  static __device__ __forceinline__ void load(double (&x)[2][2][4], const double *d, int li, int lg) {
    const double *p = d + lg * BAND + li;
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int tj = 0; tj < 2; ++tj)
#pragma unroll
        for (int v = 0; v < 4; ++v) x[ti][tj][v] = p[(16 * ti + 4 * v) * BAND + 16 * tj];
  }
  // d, rt: D and R^T of all nb blocks, row-major
  __device__ __forceinline__ void begin(const double *d, const double *rt, int nb, int li, int lg) {
    load(ns, d, li, lg);
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int tj = 0; tj < 2; ++tj)
#pragma unroll
        for (int v = 0; v < 4; ++v) { S[ti][tj][v] = ns[ti][tj][v]; nk[ti][tj][v] = 0.0; }
    request(d, rt, 0, nb, li, lg);
  }
  __device__ __forceinline__ void request(const double *d, const double *rt, int i, int nb, int li, int lg) {
    if (i + 1 < nb) { load(nk, rt + (int64_t)i * 1024, li, lg); load(ns, d + (int64_t)(i + 1) * 1024, li, lg); }
  }
  // Row PV through LDS.  What a pivot does not need any more is not sent: its wavefront's accesses to LDS keep their order.
  template <bool INVERSE, int PV> __device__ __forceinline__ void fetch(double *row, Row &r, int li, int lg) {
    constexpr int ti = PV / 16, v = PV % 16 / 4, t0 = INVERSE ? 0 : ti;
    wavefront_order();
    if (lg == PV % 4) {
      if (t0 == 0) row[li] = M[ti][0][v];
      row[16 + li] = M[ti][1][v];
      row[32 + li] = K[ti][0][v]; row[48 + li] = K[ti][1][v];
    }
    wavefront_order();
    r.p = row[PV];
    r.c[0] = t0 == 0 ? row[li] : 0.0; r.c[1] = row[16 + li];
    r.k[0] = row[32 + li]; r.k[1] = row[48 + li];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (t >= t0) r.f[t][u] = row[16 * t + lg + 4 * u];
        r.h[t][u] = row[32 + 16 * t + lg + 4 * u];
      }
  }
  // Formed here: moved to where it is used next, an update would keep its operands alive until then.
  static __device__ __forceinline__ void pin(double &x) { asm volatile("" : "+v"(x)); }
  // 1 / pivot, with a floor under it
  static __device__ __forceinline__ double inverse(double p, double tiny, bool &ok) {
    if (!(p > 0.0)) ok = false;
    if (!(p > tiny)) p = tiny;
    return rcp_newton(p);
  }
  template <bool INVERSE = true>
  __device__ __forceinline__ bool step(const double *d, const double *rt, int i, int nb, double sigma, double tiny, double *row, int li, int lg) {
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int tj = 0; tj < 2; ++tj)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          M[ti][tj][v] = S[ti][tj][v] + (ti == tj && lg + 4 * v == li ? sigma : 0.0);
          K[ti][tj][v] = nk[ti][tj][v];
          S[ti][tj][v] = ns[ti][tj][v];
        }
    bool ok = true;
    Row cur;
    fetch<INVERSE, 0>(row, cur, li, lg);
    double inv = inverse(cur.p, tiny, ok);
    for_each_block<32>([&](auto pc) {
      constexpr int PV = decltype(pc)::value, ti = PV / 16, v = PV % 16 / 4, t0 = INVERSE ? 0 : ti;
      constexpr int NT = (PV + 1) / 16, NV = (PV + 1) % 16 / 4;            // where the next pivot's row is
      const double c0 = t0 == 0 ? cur.c[0] * inv : 0.0, c1 = cur.c[1] * inv, k0 = cur.k[0] * inv, k1 = cur.k[1] * inv;
      const bool mine = li == PV % 16;
      // of the pivot's own column remains its row times 1 / pivot
      const double m0 = INVERSE && ti == 0 && mine ? -inv : c0, m1 = INVERSE && ti == 1 && mine ? -inv : c1;
      auto update_mk = [&](int t, int u) {
        if (t < t0 || (!INVERSE && t == ti && u < v)) return;              // rows in front of the pivot are done with
        if (INVERSE) M[t][ti][u] = mine ? 0.0 : M[t][ti][u];
        if (INVERSE || t == 0) M[t][0][u] -= cur.f[t][u] * m0;
        M[t][1][u] -= cur.f[t][u] * m1;
        K[t][0][u] -= cur.f[t][u] * k0;
        K[t][1][u] -= cur.f[t][u] * k1;
        if (INVERSE || t == 0) pin(M[t][0][u]);
        pin(M[t][1][u]); pin(K[t][0][u]); pin(K[t][1][u]);
      };
      auto update_s = [&](int t, int u) {
        if (INVERSE || t == 0) S[t][0][u] -= cur.h[t][u] * k0;
        S[t][1][u] -= cur.h[t][u] * k1;
        if (INVERSE || t == 0) pin(S[t][0][u]);
        pin(S[t][1][u]);
      };
      // the pivot's own row; one that shares its registers with the next pivot's has to be settled first
      auto own = [&]() {
        if (!INVERSE) return;
        const bool row = lg == PV % 4;
        M[ti][0][v] = row ? (ti == 0 && mine ? -inv : c0) : M[ti][0][v];
        M[ti][1][v] = row ? (ti == 1 && mine ? -inv : c1) : M[ti][1][v];
        K[ti][0][v] = row ? k0 : K[ti][0][v];
        K[ti][1][v] = row ? k1 : K[ti][1][v];
      };
      Row next = cur;
      if constexpr (PV < 31) {
        update_mk(NT, NV);
        if (NT == ti && NV == v) own();
        fetch<INVERSE, PV + 1>(row, next, li, lg);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) if (!(PV < 31 && t == NT && u == NV)) update_mk(t, u);
      if (!(PV < 31 && NT == ti && NV == v)) own();
      if constexpr (PV < 31) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) update_s(t, u);
      if constexpr (PV < 31) inv = inverse(next.p, tiny, ok);
      if constexpr (PV == 15) request(d, rt, i + 1, nb, li, lg);
      cur = next;
    });
    return ok;
  }
};

// Round `round` of the search for the smallest eigenvalue: wavefront s tells whether B - shift_s is
// positive definite.  Round 0: a ladder of shifts over all magnitudes; later rounds divide the bracket,
// where the eigenvalue is negative or so small that float64 resolves it only by itself.
// BAND_SHIFTS workgroups per matrix, one wavefront
__device__ __forceinline__ double band_ladder(int s, double amax) {   // 0, amax 2^-48 ... 2^-3, -amax 2^-55 ... 2
  return s == 0 ? 0.0 : s <= 16 ? ldexp(amax, 3 * s - 51) : -2.0 * ldexp(amax, 4 * (s - 31));
}
__device__ __forceinline__ void band_bracket(const BandArgs &g, int round, double &lo, double &up, int &active) {
  // what round - 1 has left behind: its own bracket and its verdicts
  const BandMeta &m = *g.meta;
  const int32_t *ok = g.ok + ((round - 1) & 1) * BAND_SHIFTS;
  if (round == 1) {
    int cnt = 0;
    while (cnt <= 16 && ok[cnt]) ++cnt;
    if (cnt > 0) {
      lo = band_ladder(cnt - 1, m.amax);
      up = cnt <= 16 ? band_ladder(cnt, m.amax) : m.hi;
    } else {
      int s = 17;
      while (s < 31 && !ok[s]) ++s;
      lo = band_ladder(s, m.amax);
      up = s == 17 ? 0.0 : band_ladder(s - 1, m.amax);
    }
    active = m.coupled && (cnt == 0 || lo + (double)g.eps < TRI_DEFLATE_BELOW * (m.hi + (double)g.eps)) ? 1 : 0;
  } else {
    lo = m.lo[(round - 1) & 1]; up = m.up[(round - 1) & 1]; active = m.active[(round - 1) & 1];
    if (active) {
      int cnt = 0;
      while (cnt < BAND_SHIFTS && ok[cnt]) ++cnt;
      const double step = (up - lo) / (BAND_SHIFTS + 1);
      up = cnt < BAND_SHIFTS ? lo + step * (cnt + 1) : up;
      lo = lo + step * cnt;
      if (!(up - lo > 0x1p-53 * m.amax)) active = 0;
    }
  }
}
__global__ __launch_bounds__(64) void band_probe_kernel(const BandJobs grp) {
  __shared__ double row[2 * BAND];
  BAND_PICK(BAND_SHIFTS)
  const int s = bx, round = k;
  band_select(g, b);
  if (g.meta->skip) return;
  const int lane = threadIdx.x, li = lane & 15, lg = lane >> 4;
  double sigma;
  if (round == 0) {
    sigma = band_ladder(s, g.meta->amax);
  } else {
    double lo, up;
    int active;
    band_bracket(g, round, lo, up, active);
    if (s == 0 && lane == 0) { g.meta->lo[round & 1] = lo; g.meta->up[round & 1] = up; g.meta->active[round & 1] = active; }
    if (!active) return;
    sigma = lo + (up - lo) / (BAND_SHIFTS + 1) * (s + 1);
  }
  BandElim e;
  bool ok = true;
  e.begin(g.dblk, g.cblk, g.nb, li, lg);
  for (int i = 0; i < g.nb && ok; ++i) ok = e.step<false>(g.dblk, g.cblk, i, g.nb, -sigma, 1.0e-290, row, li, lg);
  if (lane == 0) g.ok[(round & 1) * BAND_SHIFTS + s] = ok ? 1 : 0;
}

// Range, poles and exceptions of every matrix.  One thread per matrix
__global__ __launch_bounds__(64) void band_plan_kernel(const BandJobs grp) {
  int wg;
  const BandJob job = group_pick(grp, wg);
  BandArgs g = job.g;
  const int b = wg * 64 + threadIdx.x;
  if (b >= job.cnt) return;
  int32_t *failed_user = g.failed_user;
  band_select(g, b);
  BandMeta &m = *g.meta;
  if (m.skip == 2) { *g.skip = 1; return; }
  if (m.skip == 0) {
    double lo, up;
    int active;
    band_bracket(g, BAND_ROUNDS, lo, up, active);
    const double eps = (double)g.eps, r = (double)g.r;
    const double lam_min = m.coupled ? fmin(lo, m.dec_min) : m.dec_min;
    m.shift = fmin(lam_min, 0.0);
    m.lam = lo;
    if (!(pow((lam_min - m.shift) + eps, -r) <= 3.0e38)) m.skip = 1;
    m.base = eps - m.shift;
    const double top = m.hi + m.base, low = fmax(lo + m.base, TRI_LOWEST * top);
    m.deflate = m.coupled && low < TRI_DEFLATE_BELOW * top ? 1 : 0;
    m.cls = rat_class(low, top);
    m.poles = rat_poles(m.cls);
    m.low = ldexp(top, -4 * (m.cls + 1));
    m.f1 = pow((lo - m.shift) + eps, -r);
  }
  *g.skip = m.skip ? 1 : 0;
  if (failed_user) failed_user[b] = m.skip ? 1 : 0;
  if (m.skip && g.fail_count) atomicAdd(g.fail_count, 1ull);
}

// Eliminates B + sigma_j from the first block to the last, then forms the diagonal blocks of the inverse
// from the last to the first.  One wavefront per matrix and pole, BAND_SLOTS workgroups per matrix.  Bound by the
// latency of 32 pivots per block.  The last slot iterates for the eigenvector that is handled by itself, from just below
// its eigenvalue: the smallest pole is near zero on the shifted axis, and where lambda_min is positive that is no nearer
// to it than to the next eigenvalue.
__global__ __launch_bounds__(64) void band_factor_kernel(const BandTableJobs grp, const RatTable table) {
  __shared__ double row[2 * BAND];
  __shared__ double z[BAND_MAX_N + BAND];
  BAND_PICK(BAND_SLOTS)
  const int pole = bx;
  band_select(g, b);
  const BandMeta m = *g.meta;
  const bool vector = pole == RAT_MAX_POLES;
  if (m.skip || (vector ? !m.deflate : pole >= m.poles)) return;
  const int lane = threadIdx.x, li = lane & 15, lg = lane >> 4, nb = g.nb;
  const double sigma = vector ? 0x1p-50 * m.amax - m.lam : m.base + m.low * exp(rat_log_pole(m.cls, pole));
  const double wj = vector ? 0.0 : table.w[rat_offset(m.cls) + pole] * pow(m.low, 1.0 - (double)g.r);
  double *kf = g.kf + (int64_t)pole * nb * 1024, *gf = g.gf + (int64_t)pole * nb * 1024;
  BandElim e;
  e.begin(g.dblk, g.cblk, nb, li, lg);
  for (int i = 0; i < nb; ++i) {
    e.step(g.dblk, g.cblk, i, nb, sigma, 0x1p-60 * m.amax, row, li, lg);
    double *go = gf + (int64_t)i * 1024;
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int tj = 0; tj < 2; ++tj)
#pragma unroll
        for (int v = 0; v < 4; ++v) go[((ti * 2 + tj) * 4 + v) * 64 + lane] = -e.M[ti][tj][v];
    if (i + 1 < nb) {
      double *ko = kf + (int64_t)i * 1024;
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj)
#pragma unroll
          for (int v = 0; v < 4; ++v) ko[band_a_index(16 * ti + lg + 4 * v, 16 * tj + li)] = -e.K[ti][tj][v];
    }
  }
  __syncthreads();
  if (vector) {
    // x <- (B + sigma)^-1 x:  z_i+1 = x_i+1 - K_i z_i,  x_i = pivot_i^-1 z_i - K_i^T x_i+1
    const int a = lane & 31, k0 = 16 * (lane >> 5);
    for (int i = lane; i < g.np; i += 64) z[i] = 1.0 + 0.25 * (double)(((unsigned)i * 2654435761u) >> 24) * 0x1p-8;
    __syncthreads();
    // Chains of 2 nb steps: the next step's entries of K and of the inverse pivots are requested before this one's are used.
    auto k_to = [&](double (&x)[16], int i) {                    // K_i, for z_i
      const double *ko = kf + (int64_t)min(i, max(nb - 2, 0)) * 1024;
#pragma unroll
      for (int q = 0; q < 16; ++q) x[q] = ko[band_a_index(k0 + q, a)];
    };
    auto back_to = [&](double (&x)[16], double (&y)[16], int i) {  // pivot_i^-1, for z_i, and K_i^T, for z_i+1
      const double *go = gf + (int64_t)max(i, 0) * 1024, *ko = kf + (int64_t)max(min(i, nb - 2), 0) * 1024;
#pragma unroll
      for (int q = 0; q < 16; ++q) { x[q] = go[band_d_index(a, k0 + q)]; y[q] = ko[band_a_index(a, k0 + q)]; }
    };
    for (int it = 0; it < 5; ++it) {
      double kx[16], gx[16];
      k_to(kx, 0);
      for (int i = 0; i + 1 < nb; ++i) {
        double next[16], s = 0.0;
        k_to(next, i + 1);
#pragma unroll
        for (int q = 0; q < 16; ++q) s += kx[q] * z[BAND * i + k0 + q];
        s += __shfl_xor(s, 32, 64);
        if (lane < 32) z[BAND * (i + 1) + a] += s;
        wavefront_order();
#pragma unroll
        for (int q = 0; q < 16; ++q) kx[q] = next[q];
      }
      double nrm = 0.0;
      back_to(gx, kx, nb - 1);
      for (int i = nb - 1; i >= 0; --i) {
        double gn[16], kn[16], s = 0.0;
        back_to(gn, kn, i - 1);
#pragma unroll
        for (int q = 0; q < 16; ++q) s += gx[q] * z[BAND * i + k0 + q];
        if (i + 1 < nb) {
#pragma unroll
          for (int q = 0; q < 16; ++q) s += kx[q] * z[BAND * (i + 1) + k0 + q];
        }
        s += __shfl_xor(s, 32, 64);
        wavefront_order();
        if (lane < 32) z[BAND * i + a] = s;
        wavefront_order();
        nrm += lane < 32 ? s * s : 0.0;
#pragma unroll
        for (int q = 0; q < 16; ++q) { gx[q] = gn[q]; kx[q] = kn[q]; }
      }
      nrm = rsqrt_newton(wave64_sum(nrm));
      for (int i = lane; i < g.np; i += 64) z[i] *= nrm;
      wavefront_order();
    }
    for (int i = lane; i < g.np; i += 64) g.v1[i] = z[i];
    return;
  }
  // G_i = pivot_i^-1 + K_i^T G_i+1 K_i; the next block's operands are requested before the products of this one
  double G[2][2][4], P[2][2][4], kn[2][2][4];
  auto get = [&](double (&x)[2][2][4], const double *from) {
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int tj = 0; tj < 2; ++tj)
#pragma unroll
        for (int v = 0; v < 4; ++v) x[ti][tj][v] = from[((ti * 2 + tj) * 4 + v) * 64 + lane];
  };
  get(G, gf + (int64_t)(nb - 1) * 1024);
  if (nb > 1) { get(P, gf + (int64_t)(nb - 2) * 1024); get(kn, kf + (int64_t)(nb - 2) * 1024); }
  for (int i = nb - 1; i >= 0; --i) {
    if (i + 1 < nb) {
      double p[2][2][4], kk[2][2][4];
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj)
#pragma unroll
          for (int v = 0; v < 4; ++v) { p[ti][tj][v] = P[ti][tj][v]; kk[ti][tj][v] = kn[ti][tj][v]; }
      if (i > 0) { get(P, gf + (int64_t)(i - 1) * 1024); get(kn, kf + (int64_t)(i - 1) * 1024); }
      band_d4 H[2][2];
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj) {
          H[ti][tj] = (band_d4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int tk = 0; tk < 2; ++tk)
#pragma unroll
            for (int v = 0; v < 4; ++v) H[ti][tj] = band_mfma(G[tk][ti][v], kk[tj][tk][v], H[ti][tj]);
        }
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj) {
          band_d4 acc = {p[ti][tj][0], p[ti][tj][1], p[ti][tj][2], p[ti][tj][3]};
#pragma unroll
          for (int tk = 0; tk < 2; ++tk)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc = band_mfma(kk[ti][tk][v], H[tk][tj][v], acc);
#pragma unroll
          for (int v = 0; v < 4; ++v) G[ti][tj][v] = acc[v];
        }
    }
    double *go = gf + (int64_t)i * 1024;
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int tj = 0; tj < 2; ++tj)
#pragma unroll
        for (int v = 0; v < 4; ++v) go[((ti * 2 + tj) * 4 + v) * 64 + lane] = wj * G[ti][tj][v];
  }
}

// Block row l of F = sum_j w_j (B + sigma_j)^-1: per pole G_{l,i} = -G_{l,i+1} K_i, held transposed, so that
// a product's result is the next one's operand; the poles are dealt over 8 wavefronts, which meet in
// LDS once per block.  nb workgroups per matrix, 512 threads; the longest rows first.
template <int PW>
__global__ __launch_bounds__(512, 2) void band_rows_kernel(const BandJobs grp) {
  __shared__ float red[2][8][1024];
  BAND_PICK(g.nb)
  band_select(g, b);
  const int poles = g.meta->poles;
  if (g.meta->skip || (poles + 7) / 8 != PW) return;
  const int np = g.np, nb = g.nb, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int l = nb - 1 - bx;
  double gt[PW][2][2][4];                // [pole][rows 16 h ...][tile of columns][v]
#pragma unroll
  for (int p = 0; p < PW; ++p) {
    const int j = w + 8 * p;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          gt[p][h][ti][v] = j < poles ? g.gf[((int64_t)j * nb + l) * 1024 + ((ti * 2 + h) * 4 + v) * 64 + lane] : 0.0;
  }
  for (int i = l; i >= 0; --i) {
    if (i < l) {
#pragma unroll
      for (int p = 0; p < PW; ++p) {
        const int j = w + 8 * p;
        if (j < poles) {
          const double *ko = g.kf + ((int64_t)j * nb + i) * 1024 + lane;
          double kn[2][2][4];
#pragma unroll
          for (int ti = 0; ti < 2; ++ti)
#pragma unroll
            for (int tk = 0; tk < 2; ++tk)
#pragma unroll
              for (int v = 0; v < 4; ++v) kn[ti][tk][v] = ko[((ti * 2 + tk) * 4 + v) * 64];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            band_d4 acc[2];
#pragma unroll
            for (int ti = 0; ti < 2; ++ti) {
              acc[ti] = (band_d4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
              for (int tk = 0; tk < 2; ++tk)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[ti] = band_mfma(kn[ti][tk][v], gt[p][h][tk][v], acc[ti]);
            }
#pragma unroll
            for (int ti = 0; ti < 2; ++ti)
#pragma unroll
              for (int v = 0; v < 4; ++v) gt[p][h][ti][v] = acc[ti][v];
          }
        }
      }
    }
    float *out = red[i & 1][w];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          double s = 0.0;
#pragma unroll
          for (int p = 0; p < PW; ++p) s += gt[p][h][ti][v];
          out[((h * 2 + ti) * 4 + v) * 64 + lane] = (float)s;
        }
    __syncthreads();
    for (int e = tid; e < 1024; e += 512) {
      double sum = 0.0;
#pragma unroll
      for (int q = 0; q < 8; ++q) sum += (double)red[i & 1][q][e];
      const float s = (float)sum;
      const int el = e & 63, v = (e >> 6) & 3, ti = (e >> 8) & 1, h = e >> 9;
      const int r = 16 * h + (el & 15), c = 16 * ti + (el >> 4) + 4 * v;
      g.f[(int64_t)(BAND * l + r) * np + BAND * i + c] = s;
      if (i < l) g.f[(int64_t)(BAND * i + c) * np + BAND * l + r] = s;
    }
  }
}

// The part of F along v1 becomes f1:  F <- F - v q^T - q v^T,  q = F v - (v.F v + f1) / 2 v.
// First kernel: y = F v;  workgroups: np / 32 per matrix, 256 threads.  Second: the update, by as many.
__global__ __launch_bounds__(256) void band_fv_kernel(const BandJobs grp) {
  BAND_PICK(g.nb)
  band_select(g, b);
  if (g.meta->skip || !g.meta->deflate) return;
  const int np = g.np, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int r = bx * BAND + w; r < (bx + 1) * BAND; r += 4) {
    double s = 0.0;
    for (int c = lane; c < np; c += 64) s += (double)g.f[(int64_t)r * np + c] * g.v1[c];
    s = wave64_sum(s);
    if (lane == 0) g.z[r] = s;
  }
}
__global__ __launch_bounds__(256) void band_deflate_kernel(const BandJobs grp) {
  __shared__ double red[4];
  BAND_PICK(g.nb)
  band_select(g, b);
  if (g.meta->skip || !g.meta->deflate) return;
  const int np = g.np, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  double s = 0.0;
  for (int c = tid; c < np; c += 256) s += g.z[c] * g.v1[c];
  s = wave64_sum(s);
  if (lane == 0) red[w] = s;
  __syncthreads();
  const double K = 0.5 * ((red[0] + red[1]) + (red[2] + red[3]) + g.meta->f1);
  for (int r = bx * BAND + w; r < (bx + 1) * BAND; r += 4) {
    const double vr = g.v1[r], qr = g.z[r] - K * vr;
    for (int c = lane; c < np; c += 64) {
      const double vc = g.v1[c], qc = g.z[c] - K * vc;
      g.f[(int64_t)r * np + c] = (float)((double)g.f[(int64_t)r * np + c] - (vr * qc + qr * vc));
    }
  }
}

// ---------------------------------------------------------------------------
// The way back: F <- H F H^T for H = I - V T V^T of a group of 4 panels, as
//     Z = F V,  Y = Z T^T - V (T M T^T) / 2 with M = V^T Z,  F <- F - Y V^T - V Y^T
// The first, the second and the last product are launches of gemm_mfma_kernel on the work array
// [Z V] and [Y V], [V Y]; the last computes the tiles on and below the diagonal and mirrors them.
// 64 matrices of 1024, kernel time summed over four streams: 23.7 ms one panel at a time, 16 ms so (64
// refreshed factors: 19.5 -> 18.1 ms in all); groups of 4 because T and M of 128 columns still fit LDS.
// ---------------------------------------------------------------------------
// T of the groups: T of two neighbours is [T1, -T1 (V1^T V2) T2; 0, T2].  band_groups workgroups per matrix, 16
// wavefronts that share the rows of the 6 products V_a^T V_b; all groups of all matrices in one launch.
__global__ __launch_bounds__(1024) void band_group_t_kernel(const BandJobs grp) {
  __shared__ float red[16][1024], T[BAND_GW][BAND_GW + 1];
  BAND_PICK(band_groups(g))
  band_select(g, b);
  if (g.meta->skip) return;
  const int np = g.np, q = bx, tid = threadIdx.x, lane = tid & 63, w = tid >> 6, li = lane & 15, lg = lane >> 4;
  const int panels = min(BAND_GROUP, g.nb - 1 - BAND_GROUP * q);
  band_f4 acc[6][2][2];
#pragma unroll
  for (int e = 0; e < 6; ++e)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[e][i][j] = (band_f4){0.f, 0.f, 0.f, 0.f};
  const float *v = g.vall + BAND_GW * q + li;
  for (int r = (BAND_GROUP * q + 1) * BAND + 4 * w; r < np; r += 64) {
    float x[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) x[t] = t < 2 * panels ? v[(int64_t)(r + lg) * np + 16 * t] : 0.f;
    int e = 0;
#pragma unroll
    for (int b = 1; b < 4; ++b)
#pragma unroll
      for (int a = 0; a < b; ++a, ++e)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[e][i][j] = band_mfma(x[2 * a + i], x[2 * b + j], acc[e][i][j]);
  }
  int e = 0;
#pragma unroll
  for (int b = 1; b < 4; ++b)
#pragma unroll
    for (int a = 0; a < b; ++a, ++e) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int u = 0; u < 4; ++u) red[w][(16 * i + 4 * lg + u) * BAND + 16 * j + li] = acc[e][i][j][u];
      __syncthreads();
      double s = 0.0;
#pragma unroll
      for (int k = 0; k < 16; ++k) s += (double)red[k][tid];
      T[BAND * a + (tid >> 5)][BAND * b + (tid & 31)] = (float)s;
      T[BAND * b + (tid >> 5)][BAND * a + (tid & 31)] = 0.f;
      __syncthreads();
    }
#pragma unroll
  for (int a = 0; a < 4; ++a)
    T[BAND * a + (tid >> 5)][BAND * a + (tid & 31)] = a < panels ? g.tall[(int64_t)(BAND_GROUP * q + a) * 1024 + tid] : 0.f;
  __syncthreads();
  float *u = red[0];                     // [h][h]: (V1^T V2) T2
  for (int h = BAND; h < BAND_GW; h *= 2)
    for (int o = 0; o < BAND_GW; o += 2 * h) {
      for (int x = tid; x < h * h; x += 1024) {
        const int i = x / h, j = x % h;
        double s = 0.0;
        for (int k = 0; k <= j; ++k) s += (double)T[o + i][o + h + k] * (double)T[o + h + k][o + h + j];
        u[x] = (float)s;
      }
      __syncthreads();
      for (int x = tid; x < h * h; x += 1024) {
        const int i = x / h, j = x % h;
        double s = 0.0;
        for (int k = i; k < h; ++k) s += (double)T[o + i][o + k] * (double)u[k * h + j];
        T[o + i][o + h + j] = (float)-s;
      }
      __syncthreads();
    }
  float *out = band_tg(g) + (int64_t)q * BAND_GW * BAND_GW;
  for (int x = tid; x < BAND_GW * BAND_GW; x += 1024) out[x] = T[x / BAND_GW][x % BAND_GW];
}

// V of group q into the work array (Y = false), or Y into its second place.  np / 8 workgroups per matrix, 256 threads
template <bool Y>
__global__ __launch_bounds__(256) void band_stage_kernel(const BandJobs grp) {
  BAND_PICK(g.np / 8)
  const int q = k;
  band_select(g, b);
  if (g.meta->skip) return;
  const int row = bx * 8 + (threadIdx.x >> 5), c = (threadIdx.x & 31) * 4;
  float *p = band_p(g) + (int64_t)row * BAND_PLD;
  if (Y) {
    *reinterpret_cast<float4 *>(p + 2 * BAND_GW + c) = *reinterpret_cast<const float4 *>(p + c);
  } else {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (BAND_GW * q + c < g.np) v = *reinterpret_cast<const float4 *>(g.vall + (int64_t)row * g.np + BAND_GW * q + c);
    *reinterpret_cast<float4 *>(p + BAND_GW + c) = v;
  }
}

// M = V^T Z and M T^T, which goes where Y will be read from.  4 workgroups of 16 wavefronts per matrix: 32 rows of M each, 4
// blocks of 32 columns by 4 quarters of V's rows.  On the fp64 matrix cores: float32 sums here cost more accuracy than the
// roundings of everything else on the way back together.  Bound by them: one workgroup per matrix for this and the next
// kernel's product took 158 us for 32 matrices of 1024 beside 32 others, the two take 78 and 29.
__global__ __launch_bounds__(1024) void band_m_kernel(const BandJobs grp) {
  __shared__ float M[BAND][BAND_GW + 1], T[BAND_GW][BAND_GW + 1];
  __shared__ double red[16][4 * 64];
  BAND_PICK(4)
  const int q = k;
  band_select(g, b);
  if (g.meta->skip) return;
  const int np = g.np, tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lg = lane >> 4;
  const int i0 = 32 * bx, j0 = 32 * (w & 3), kq = w >> 2;
  const float *tg = band_tg(g) + (int64_t)q * BAND_GW * BAND_GW;
  for (int x = tid; x < BAND_GW * BAND_GW; x += 1024) T[x / BAND_GW][x % BAND_GW] = tg[x];
  band_d4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = (band_d4){0.0, 0.0, 0.0, 0.0};
  const float *p = band_p(g) + (int64_t)lg * BAND_PLD + li;
  const int first = (BAND_GROUP * q + 1) * BAND, steps = (np - first) / 16;
  for (int s = steps * kq / 4, e = steps * (kq + 1) / 4; s < e; ++s)
#pragma unroll
    for (int t = 0; t < 16; t += 4) {
      const float *z = p + (int64_t)(first + 16 * s + t) * BAND_PLD, *v = z + BAND_GW;
      const double a0 = v[i0], a1 = v[i0 + 16], b0 = z[j0], b1 = z[j0 + 16];
      acc[0][0] = band_mfma(a0, b0, acc[0][0]); acc[0][1] = band_mfma(a0, b1, acc[0][1]);
      acc[1][0] = band_mfma(a1, b0, acc[1][0]); acc[1][1] = band_mfma(a1, b1, acc[1][1]);
    }
#pragma unroll
  for (int x = 0; x < 4; ++x) {              // tile by tile: the sums of four quarters
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) red[w][u * 64 + lane] = acc[x >> 1][x & 1][u];
    __syncthreads();
    const int at = kq * 64 + lane, jb = w & 3;      // element kq of the tile
    const double sum = (red[jb][at] + red[4 + jb][at]) + (red[8 + jb][at] + red[12 + jb][at]);
    M[16 * (x >> 1) + band_row(lg, kq)][32 * jb + 16 * (x & 1) + li] = (float)sum;
  }
  __syncthreads();
  // 32 x 128 results: a tile of 16 x 16 per wavefront
  const int ti = 16 * (w & 1), tj = 16 * (w >> 1);
  band_d4 n = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
  for (int s = 0; s < BAND_GW / 4; ++s) n = band_mfma((double)M[ti + li][4 * s + lg], (double)T[tj + li][4 * s + lg], n);
  float *out = band_ts(g);
#pragma unroll
  for (int u = 0; u < 4; ++u) out[(BAND_GW + i0 + ti + band_row(lg, u)) * BAND_GW + tj + li] = (float)n[u];
}

// [T^T; -T (M T^T) / 2], the second half in the place of M T^T.  4 workgroups of 4 wavefronts per matrix: 32 columns each.
__global__ __launch_bounds__(256) void band_s_kernel(const BandJobs grp) {
  __shared__ float N[BAND_GW][BAND + 1];
  BAND_PICK(4)
  const int q = k;
  band_select(g, b);
  if (g.meta->skip) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, li = lane & 15, lg = lane >> 4, i0 = 32 * w, j0 = 32 * bx;
  const float *tg = band_tg(g) + (int64_t)q * BAND_GW * BAND_GW;
  float *out = band_ts(g);
  for (int x = tid; x < BAND_GW * BAND; x += 256) {
    const int row = x / BAND, col = x % BAND;
    N[row][col] = out[(BAND_GW + row) * BAND_GW + j0 + col];
    out[(j0 + col) * BAND_GW + row] = tg[row * BAND_GW + j0 + col];
  }
  __syncthreads();
  band_d4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = (band_d4){0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
  for (int s = 0; s < BAND_GW / 4; ++s) {
    const int x = 4 * s + lg;
    const double a0 = tg[(i0 + li) * BAND_GW + x], a1 = tg[(i0 + 16 + li) * BAND_GW + x], b0 = N[x][li], b1 = N[x][16 + li];
    acc[0][0] = band_mfma(a0, b0, acc[0][0]); acc[0][1] = band_mfma(a0, b1, acc[0][1]);
    acc[1][0] = band_mfma(a1, b0, acc[1][0]); acc[1][1] = band_mfma(a1, b1, acc[1][1]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int u = 0; u < 4; ++u)
        out[(BAND_GW + i0 + 16 * i + band_row(lg, u)) * BAND_GW + j0 + 16 * j + li] = (float)(-0.5 * acc[i][j][u]);
}

// x from the lower triangle of F, mirrored; the rows that stand alone.  a workgroup of 256 threads per pair of 32 x 32 tiles and matrix
__global__ __launch_bounds__(256) void band_out_kernel(const BandJobs grp) {
  __shared__ float tile[BAND][BAND + 1];
  BAND_PICK(g.nb * (g.nb + 1) / 2)
  band_select(g, b);
  if (g.meta->skip) return;
  const int n = g.n, np = g.np, tid = threadIdx.x;
  int bi = (int)((sqrtf(8.f * (float)bx + 1.f) - 1.f) * 0.5f);
  while ((bi + 1) * (bi + 2) / 2 <= bx) ++bi;
  while (bi * (bi + 1) / 2 > bx) --bi;
  const int bj = bx - bi * (bi + 1) / 2;
  const int r = tid >> 3, c4 = (tid & 7) * 4;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int i = bi * BAND + r, j = bj * BAND + c4 + e;
    float v = g.f[(int64_t)i * np + j];
    if (i < n && j < n && (g.dec[i] || g.dec[j]))
      v = i == j ? (float)pow(((double)g.scale * (double)g.a[(int64_t)i * n + i] - g.meta->shift) + (double)g.eps, -(double)g.r) : 0.f;
    tile[r][c4 + e] = v;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int c = c4 + e;
    const int i = bi * BAND + r, j = bj * BAND + c;
    if (i < n && j < n) g.x[(int64_t)i * n + j] = (bi == bj && c > r) ? tile[c][r] : tile[r][c];
    const int mi = bj * BAND + r, mj = bi * BAND + c;
    if (bi != bj && mi < n && mj < n) g.x[(int64_t)mi * n + mj] = tile[c][r];
  }
}

// meta and flags start at zero.  One thread per matrix
__global__ __launch_bounds__(256) void band_clear_kernel(const BandJobs grp) {
  int wg;
  const BandJob job = group_pick(grp, wg);
  BandArgs g = job.g;
  const int b = wg * 256 + threadIdx.x;
  if (b >= job.cnt) return;
  band_select(g, b);
  g.meta->skip = 0;
  g.meta->active[0] = g.meta->active[1] = 0;
}

#undef BAND_PICK

}  // namespace shampoo
