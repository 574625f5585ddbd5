// Root inverse of matrices of n <= 128 without eigenvectors, one workgroup per matrix.
//
//   A = Q T Q^T        Householder reduction to tridiagonal form, float64, A in registers
//   F = f(T)           f(x) = (x - min(lambda_min, 0) + eps)^-r as a sum of inverses of shifted T
//                      (root_rational.h): two recurrences per shift, one product chain per row
//   X = Q F Q^T        the same reflectors in reverse order, 16 at a time (up to n = 16 one by one), float64, F in registers
//
// The LDS Jacobi solver (eigh_jacobi.h) does the same job in about eight sweeps of 127 rounds with
// two barriers and a pass over the matrix each; here there are 126 reflections and 8 products of 16.  It still serves
// callers that want the eigenvalues, and exponents that root_rational.h has no fit for.
//
// What bounds it: the latency of a reflection (two barriers, LDS round trips) and the fp64 matrix cores on the way back.  Cycles at
// n = 128, two workgroups per CU: 37000 to read A, 382000 to reduce it, 69000 for bounds and pivots, 103000 for F, 153000 back.
// The matrix itself stays out of LDS: a thread owns rows rg + RG a and columns cl + 16 b (cyclic,
// so that the shrinking part stays spread over all threads), and only the vectors of a reflection go
// through LDS.  At n = 128: 4 wavefronts,
// 128 registers of matrix per lane, 80 KB of LDS, two workgroups per CU.
//
// Accuracy: T comes from a float64 reduction, so eigenvalues move by about 1e-16 of the largest, as
// in the float64 Jacobi; the reflectors are kept as float32 for the way back (orthogonal to 1e-7,
// like accumulated float32 rotations) and the terms of F are float32.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "eigh_jacobi.h"      // SmallRootArgs, rcp_newton
#include "group.h"
#include "root_rational.h"

namespace shampoo {

// The smallest eigenvalue is bisected to float64 accuracy and its eigenvector handled apart from
// the rational sum when it is negative (then f there is exactly eps^-r) or below this fraction of
// the largest: a float64 reduction resolves lambda to 1e-16 of the largest, so that at 2^-32 the
// argument of f still holds to 1e-6.
constexpr double TRI_DEFLATE_BELOW = 0x1p-32;
constexpr double TRI_LOWEST = 0x1p-48;       // the widest range of the rational sum
// A column (squared norm) that is too small to be reflected.  Where columns depend on each other, what a reflection
// leaves of the next one is rounding, 1e-16 of it, and so on: after some ten of them its square is a denormal number with a
// few bits, and a reflector made of it is not orthogonal.  1e-100 is far below the rounding of any float32 matrix.
constexpr double TRI_NO_COLUMN = 1e-200;
constexpr int TRI_TABLE_RESERVE = sizeof(RatTable) + 16;   // of a launch's arguments, for the weights
constexpr int TRI_CHUNK = 16;                // columns of F handed from their makers to their owners at a time

// element of another lane of the same 16
template <int CTRL>
__device__ __forceinline__ double dpp_fetch(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_MIRROR8 = 0x141, DPP_MIRROR16 = 0x140;

__device__ __forceinline__ double row16_sum(double x) {
  x += dpp_fetch<DPP_XOR1>(x);
  x += dpp_fetch<DPP_XOR2>(x);
  x += dpp_fetch<DPP_MIRROR8>(x);
  return x + dpp_fetch<DPP_MIRROR16>(x);
}
__device__ __forceinline__ double lane_value(double x, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane), __builtin_amdgcn_readlane(__double2loint(x), lane));
}
// sum over the 64 lanes, the same bits in all of them
__device__ __forceinline__ double wave64_sum(double x) {
  x = row16_sum(x);
  return (lane_value(x, 0) + lane_value(x, 16)) + (lane_value(x, 32) + lane_value(x, 48));
}

// sum over the four lanes l % 16, in all of them
__device__ __forceinline__ double rows_sum(double x) {
  auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(x), false, false);
  auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(x), false, false);
  x = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
  lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(x), false, false);
  hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(x), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

// The reduction's lanes: 16 columns (lane bits 5, 4, 1, 0) by 4 rows (bits 3, 2), so that the sums over columns begin with the
// swaps of half and quarter wavefronts, which exchange what each side does not keep without a selection.
__device__ __forceinline__ int tri_col(int lane) { return (lane >> 4) * 4 + (lane & 3); }
__device__ __forceinline__ int tri_row(int lane) { return (lane >> 2) & 3; }
__device__ __forceinline__ double tri_rows_sum(double x) { x += dpp_fetch<0x128>(x); return x + dpp_fetch<0x124>(x); }   // row_ror:8, row_ror:4
// lanes < 32: a + a of lane + 32; others b + b of lane - 32
__device__ __forceinline__ double swap32_sum(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// the same between the even and the odd rows of 16 lanes
__device__ __forceinline__ double swap16_sum(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// Sums over the 16 columns of v[P0 ... 7], P0 < 4 or not: a lane ends with value tri_slot<P0>.
template <int P0> __device__ __forceinline__ int tri_slot(int lane) {
  return P0 < 4 ? (lane >> 5) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 1) & 1) : 4 + (lane >> 5) * 2 + ((lane >> 4) & 1);
}
template <int P0> __device__ __forceinline__ double tri_cols_sums(const double (&v)[8], int lane) {
  double x;
  if constexpr (P0 < 4) {
    const double a = swap16_sum(swap32_sum(v[0], v[4]), swap32_sum(v[2], v[6])), b = swap16_sum(swap32_sum(v[1], v[5]), swap32_sum(v[3], v[7]));
    const bool second = (lane & 2) != 0;
    x = (second ? b : a) + dpp_fetch<DPP_XOR2>(second ? a : b);
  } else {
    x = swap16_sum(swap32_sum(v[4], v[6]), swap32_sum(v[5], v[7]));
    x += dpp_fetch<DPP_XOR2>(x);
  }
  return x + dpp_fetch<DPP_XOR1>(x);
}

typedef double tri_d4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ tri_d4 tri_mfma(double a, double b, tri_d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// f(BlockIndex<0>()), ..., f(BlockIndex<COUNT - 1>()): a loop whose index is a constant in the body
template <int I> struct BlockIndex { static constexpr int value = I; };
template <int COUNT, int I = 0, typename F> __device__ __forceinline__ void for_each_block(F &&f) {
  if constexpr (I < COUNT) { f(BlockIndex<I>()); for_each_block<COUNT, I + 1>(f); }
}

// All pivots of T - sigma positive, i.e. sigma < lambda_min
__device__ __forceinline__ bool tri_above(const double *d, const double *e, int n, double sigma) {
  double piv = d[0] - sigma;
  bool ok = piv > 0.0;
  for (int i = 1; i < n; ++i) {
    piv = d[i] - sigma - e[i - 1] * e[i - 1] * rcp_newton(piv);
    ok = ok && piv > 0.0;
  }
  return ok;
}

// The way back: 16 reflectors at a time.  The strides leave no bank conflicts but for a few lanes, along rows and across them.
template <int N> struct TriBack {
  float v[16][N + 20];                       // V^T
  double y[16][N + 18];                      // Z^T, shares of M, Y^T; S = V^T V of all groups, 256 entries each
  double t[N / 16][256];                     // T^T of all groups
};
template <int N> struct TriShared {
  double d[N], e[N], v1[N];                  // T; the eigenvector handled by itself
  double beta[N];                            // reflector k: 0 where there is none
  union {
    struct {
      union {
        struct { double x[N], p[N], s2[4], vav[4]; } step;    // vectors of the current reflection, wavefronts' sums
        struct { double slot[N * RAT_MAX_POLES]; float chunk[TRI_CHUNK][N]; } fun;
        TriBack<N> back;
      };
      float vs[(N - 1) * (N - 2) / 2];       // reflector k: entries k + 2 .. n - 1 (entry k + 1 is 1)
    };
    float out[N][N + 1];
  };
  double bound[2];                           // bracket of the smallest eigenvalue
  int count;
  unsigned char dec[N];                      // row k is coupled to no other
};

// N: the largest n; NT threads = 16 lanes along the columns x RG row groups
template <int N, int NT>
__global__ __launch_bounds__(NT, 2) void rootinv_tridiag_kernel(const Group<SmallRootArgs, TRI_TABLE_RESERVE> grp, const RatTable table) {
  constexpr int RG = NT / 16, RB = N / RG, CB = N / 16;
  static_assert(RB == 8, "rows of a lane");
  constexpr int PQ = RAT_MAX_POLES / 2, PQ_STEP = 6;      // two lanes share a row of F: poles per lane, taken 6 at a time
  static_assert(NT == 2 * N && PQ % PQ_STEP == 0, "two lanes per row");
  int b;
  const SmallRootArgs g = group_pick(grp, b);
  if (b >= g.batch || (g.only && g.only[b] == 0)) return;
  __shared__ __align__(16) TriShared<N> sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, cl = tri_col(lane), rg = tri_row(lane) + 4 * wave;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int n = g.n;
  const float *a = g.a + (int64_t)b * g.a_stride;
  auto wave_sums = [](const double *s) { return NT == 64 ? s[0] : NT == 128 ? s[0] + s[1] : (s[0] + s[1]) + (s[2] + s[3]); };

  // ---- load (symmetrised), find what is not finite and the rows that stand alone ----
  double A[RB][CB];
  int bad = 0;
  // element e is in row e / n: e n < 2^32.  16 loads in flight (one at a time took 42 us for 64 KB)
  const uint32_t over_n = (uint32_t)((1ull << 32) / n) + ((n & (n - 1)) != 0 ? 1u : 0u);
  auto row_of = [&](int e) { return n == 1 ? 0 : (int)__umulhi((uint32_t)e, over_n); };
  for (int e0 = tid; e0 < n * n; e0 += 16 * NT) {
    float v[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) { const int e = e0 + NT * t; v[t] = a[e < n * n ? e : 0]; }
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const int e = e0 + NT * t, i = row_of(e);
      if (e >= n * n) continue;
      if (!(fabsf(v[t]) <= 3.0e38f)) bad = 1;
      sh.out[i][e - i * n] = v[t];
    }
  }
  for (int i = tid; i < N; i += NT) sh.dec[i] = 1;
  __syncthreads();
#pragma unroll
  for (int p = 0; p < RB; ++p) {
    const int r = rg + RG * p, ri = min(r, n - 1);
    bool any = false;
#pragma unroll
    for (int q = 0; q < CB; ++q) {
      const int c = cl + 16 * q, ci = min(c, n - 1);
      const double v = (double)g.scale * (0.5 * ((double)sh.out[ri][ci] + (double)sh.out[ci][ri]));
      A[p][q] = (r < n && c < n) ? v : 0.0;
      any = any || (r != c && A[p][q] != 0.0);
    }
    if (any) sh.dec[r] = 0;
  }
  bad = __syncthreads_or(bad);
  if (bad) {   // Sec. 3.2.3: keep the previous root
    if (tid == 0) {
      if (g.failed) g.failed[b] = 1;
      if (g.fail_count) atomicAdd(g.fail_count, 1ull);
    }
    return;
  }
  // A row that is coupled to no other is an eigenvector by itself: its entry of the result is f of
  // its diagonal entry, and it takes part in the reduction with a diagonal entry from inside the
  // spectrum of the rest, where it changes neither end of it.
#pragma unroll
  for (int p = 0; p < RB; ++p)
#pragma unroll
    for (int q = 0; q < CB; ++q)
      if (rg + RG * p == cl + 16 * q) sh.step.x[rg + RG * p] = A[p][q];
  __syncthreads();
  double dec_min = 1.0e300, fill = -1.0e300;
  for (int i = lane; i < n; i += 64) {
    const double v = sh.step.x[i];
    if (sh.dec[i]) dec_min = fmin(dec_min, v); else fill = fmax(fill, v);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) { dec_min = fmin(dec_min, __shfl_xor(dec_min, off, 64)); fill = fmax(fill, __shfl_xor(fill, off, 64)); }
  const bool coupled = fill > -1.0e300, lone = dec_min < 1.0e300;
  if (!coupled) fill = 1.0;
#pragma unroll
  for (int p = 0; p < RB; ++p)
#pragma unroll
    for (int q = 0; q < CB; ++q) {
      const int r = rg + RG * p, c = cl + 16 * q;
      if (r == c && r < n && sh.dec[r]) A[p][q] = fill;
    }
  __syncthreads();

  // ---- reduction ----
  auto offs = [n](int k) { return k * (n - 2) - k * (k - 1) / 2 - (k + 2); };   // entry i of reflector k: vs[offs(k) + i]
  // Columns 16 KQ .. 16 KQ + 15: the blocks left of and above them are finished and drop out of the
  // code (the whole similarity transform is applied to the others: what it does to finished rows and
  // columns inside them is to turn them into T).
  // Bound by the latency of a reflection.  The update of A that belongs to one is done in the next: its first block column
  // ahead of the barrier behind which the next column can be read, the rest beside the chain from that column's norm to its
  // reflector.  Norm and v^T A v are summed within the wavefronts ahead of the barriers that are there anyway.  3072 matrices of 128 x 128, two
  // workgroups per CU: 3590 cycles per reflection before, 3030 so.
  double vr[RB], qr[RB], vc[CB], qc[CB];         // rows and columns of v and q: A <- A - v q^T - q v^T is to be done
#pragma unroll
  for (int p = 0; p < RB; ++p) vr[p] = qr[p] = 0.0;
#pragma unroll
  for (int q = 0; q < CB; ++q) vc[q] = qc[q] = 0.0;
  auto reduce16 = [&](auto kq) {
    constexpr int KQ = decltype(kq)::value, P0 = 16 * KQ / RG, P1 = P0 + 16 / RG, P2 = P1 + 16 / RG;  // row blocks P0 .. P1 - 1: rows 16 KQ .. 16 KQ + 15
    for (int k = 16 * KQ; k < min(16 * KQ + 16, n - 1); ++k) {
      double *xb = sh.step.x, *pb = sh.step.p;
      double s2 = 0.0;
#pragma unroll
      for (int p = P0; p < RB; ++p) {
        A[p][KQ] = fma(-vr[p], qc[KQ], fma(-qr[p], vc[KQ], A[p][KQ]));
        const double x = (p >= P2 || rg + RG * p > k + 1) ? A[p][KQ] : 0.0;
        s2 = fma(x, x, s2);
      }
      if (cl == (k & 15)) {
#pragma unroll
        for (int p = P0; p < RB; ++p) {
          const int r = rg + RG * p;
          xb[r] = (p >= P1 || r > k) ? A[p][KQ] : 0.0;
          if (p < P1 && r == k) sh.d[k] = A[p][KQ];
        }
      }
      s2 = tri_rows_sum(s2);
      if (lane == ((k & 12) << 2 | (k & 3))) sh.step.s2[wave] = s2;
      __syncthreads();
      s2 = wave_sums(sh.step.s2);
      const double x0 = xb[k + 1];
      // finished rows of A (p < P0) are left as they are
#pragma unroll
      for (int q = KQ + 1; q < CB; ++q)
#pragma unroll
        for (int p = P0; p < RB; ++p) A[p][q] = fma(-vr[p], qc[q], fma(-qr[p], vc[q], A[p][q]));
      const bool none = !(s2 > TRI_NO_COLUMN);       // nothing to reflect
      // 1 / (norm |v0|) starts from the estimate of the norm, beside the steps that refine it (as rsqrt_newton and rcp_newton)
      const double nn = none ? 1.0 : fma(x0, x0, s2), h = 0.5 * nn;
      double rn = __builtin_amdgcn_rsq(nn), bi = __builtin_amdgcn_rcp(fma(nn * rn, fabs(x0), nn));
      rn = rn * (1.5 - h * (rn * rn)); rn = rn * (1.5 - h * (rn * rn));
      const double norm = nn * rn, nv = fma(norm, fabs(x0), nn);          // norm |v0| = norm (norm + |x0|)
      bi = bi * (2.0 - nv * bi); bi = bi * (2.0 - nv * bi);
      const double alpha = x0 > 0.0 ? -norm : norm, v0 = x0 - alpha, beta = none ? 0.0 : bi;
      double part[RB], vav = 0.0;
#pragma unroll
      for (int p = 0; p < RB; ++p) part[p] = 0.0;
#pragma unroll
      for (int q = KQ; q < CB; ++q) {
        vc[q] = xb[cl + 16 * q];
        if (q < KQ + 2 && cl + 16 * q == k + 1) vc[q] = v0;
#pragma unroll
        for (int p = P0; p < RB; ++p) part[p] = fma(A[p][q], vc[q], part[p]);
      }
#pragma unroll
      for (int p = P0; p < RB; ++p) {
        vr[p] = xb[rg + RG * p];
        if (p < P2 && rg + RG * p == k + 1) vr[p] = v0;
        vav = fma(vr[p], part[p], vav);
      }
      pb[rg + RG * tri_slot<P0>(lane)] = tri_cols_sums<P0>(part, lane);
      vav = rows_sum(row16_sum(vav));
      if (lane == 0) sh.step.vav[wave] = vav;
      {
        const double inv = copysign(norm * beta, v0);
        if (tid == 0) { sh.beta[k] = beta; sh.e[k] = none ? x0 : alpha; }
        if (tid > k + 1 && tid < n) sh.vs[offs(k) + tid] = (float)(xb[tid] * inv);
      }
      __syncthreads();
      const double K = 0.5 * beta * (beta * wave_sums(sh.step.vav));       // beta^2 may be too large
#pragma unroll
      for (int q = KQ; q < CB; ++q) qc[q] = fma(beta, pb[cl + 16 * q], -K * vc[q]);
#pragma unroll
      for (int p = P0; p < RB; ++p) qr[p] = fma(beta, pb[rg + RG * p], -K * vr[p]);
    }
  };
  for_each_block<CB>(reduce16);
#pragma unroll
  for (int p = 0; p < RB; ++p)
#pragma unroll
    for (int q = 0; q < CB; ++q)
      if (rg + RG * p == n - 1 && cl + 16 * q == n - 1) sh.d[n - 1] = A[p][q];
  __syncthreads();

  // ---- bounds of the spectrum, smallest eigenvalue ----
  const double eps = (double)g.epsilon, r_exp = (double)g.r;
  double hi = -1.0e300, amax = 0.0;
  for (int i = lane; i < n; i += 64) {
    const double off = (i > 0 ? fabs(sh.e[i - 1]) : 0.0) + (i < n - 1 ? fabs(sh.e[i]) : 0.0);
    hi = fmax(hi, sh.d[i] + off);
    amax = fmax(amax, fabs(sh.d[i]) + off);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) { hi = fmax(hi, __shfl_xor(hi, off, 64)); amax = fmax(amax, __shfl_xor(amax, off, 64)); }
  if (wave == 0) {
    // a ladder of shifts, one per lane: 0, amax 2^-48 ... amax 2^-1, and downwards -2 amax 2^-56 ... -2 amax
    const double sigma = lane == 0 ? 0.0 : lane <= 48 ? ldexp(amax, lane - 49) : -2.0 * ldexp(amax, 4 * (lane - 63));
    const unsigned long long up = __ballot(tri_above(sh.d, sh.e, n, sigma));
    const int cnt = __popcll(up & ((1ull << 49) - 1));
    if (lane == 0) {
      double lo_b, hi_b;
      if (cnt > 0) {
        lo_b = cnt == 1 ? 0.0 : ldexp(amax, cnt - 1 - 49);
        hi_b = cnt == 49 ? hi : ldexp(amax, cnt - 49);
      } else {
        int l = 49;
        while (l < 63 && !((up >> l) & 1)) ++l;
        lo_b = -2.0 * ldexp(amax, 4 * (l - 63));
        hi_b = l == 49 ? 0.0 : -2.0 * ldexp(amax, 4 * (l - 1 - 63));
      }
      sh.bound[0] = lo_b; sh.bound[1] = hi_b; sh.count = cnt;
    }
  }
  __syncthreads();
  double lam = sh.bound[0], lam_up = sh.bound[1];
  const bool deflate = coupled && (sh.count == 0 || lam + eps < TRI_DEFLATE_BELOW * (hi + eps));
  if (deflate) {
    for (int round = 0; round < 12 && lam_up - lam > 0x1p-53 * amax; ++round) {
      const double step = (lam_up - lam) / (NT + 1);
      const int c = __syncthreads_count(tri_above(sh.d, sh.e, n, lam + step * (tid + 1)));
      const double base = lam;
      lam = base + step * c;
      if (c < NT) lam_up = base + step * (c + 1);
    }
  }
  const double lam_min = coupled ? fmin(lam, dec_min) : dec_min;
  const double shift = fmin(lam_min, 0.0);
  // without deflation lam is a lower bound within a factor of two, and only a bound is needed
  const double f_min = pow((lam_min - shift) + eps, -r_exp);
  if (!(f_min <= 3.0e38)) {   // not representable: keep the previous root
    if (tid == 0) {
      if (g.failed) g.failed[b] = 1;
      if (g.fail_count) atomicAdd(g.fail_count, 1ull);
    }
    return;
  }
  if (tid == 0 && g.failed) g.failed[b] = 0;
  const double base = eps - shift, top = hi + base;
  double low = fmax(lam + base, TRI_LOWEST * top);
  const int cls = rat_class(low, top), np = rat_poles(cls);
  low = ldexp(top, -4 * (cls + 1));
  double *slot = sh.fun.slot;
  if (deflate && tid == 0) {
    // the eigenvector of lam by inverse iteration just below it
    const double sg = lam - 0x1p-50 * amax;
    double *piv = slot, *z = sh.v1;
    double pv = sh.d[0] - sg;
    piv[0] = 1.0 / pv;
    for (int i = 1; i < n; ++i) { pv = sh.d[i] - sg - sh.e[i - 1] * sh.e[i - 1] * piv[i - 1]; piv[i] = 1.0 / (pv > 0x1p-60 * amax ? pv : 0x1p-60 * amax); }
    for (int i = n; i < N; ++i) z[i] = 0.0;
    for (int i = 0; i < n; ++i) z[i] = 1.0 + 0.25 * (double)((i * 2654435761u) >> 24) * 0x1p-8;
    for (int it = 0; it < 4; ++it) {
      double zz = z[0];
      for (int i = 1; i < n; ++i) { zz = z[i] - sh.e[i - 1] * piv[i - 1] * zz; z[i] = zz; }
      zz = z[n - 1] * piv[n - 1];
      z[n - 1] = zz;
      double s2 = zz * zz;
      for (int i = n - 2; i >= 0; --i) { zz = piv[i] * (z[i] - sh.e[i] * zz); z[i] = zz; s2 += zz * zz; }
      const double inv = 1.0 / sqrt(s2);
      for (int i = 0; i < n; ++i) z[i] *= inv;
    }
  }
  __syncthreads();

  // ---- F = sum_j w_j (T + sigma_j)^-1: pivots from the top, diagonal of the inverse from the bottom ----
  // slot (i, j): first 1 / pivot, then (-e_i / pivot, w_j G_ii) as float32
  const int half = ((np + 1) / 2 + PQ_STEP - 1) / PQ_STEP * PQ_STEP;     // poles per lane of a row, the last ones with weight 0
  if (tid < 2 * half) {
    const bool real = tid < np;
    const double sg = real ? base + low * exp(rat_log_pole(cls, tid)) : amax + top;
    const double wj = real ? table.w[rat_offset(cls) + tid] * pow(low, 1.0 - r_exp) : 0.0;
    double inv = rcp_newton(sh.d[0] + sg);
    slot[tid] = inv;
    for (int i = 1; i < n; ++i) {
      inv = rcp_newton(sh.d[i] + sg - sh.e[i - 1] * sh.e[i - 1] * inv);
      slot[i * RAT_MAX_POLES + tid] = inv;
    }
    double G = inv, next = n > 1 ? slot[(n - 2) * RAT_MAX_POLES + tid] : 0.0;
    reinterpret_cast<float2 *>(slot)[(n - 1) * RAT_MAX_POLES + tid] = make_float2(0.f, (float)(wj * G));
    for (int i = n - 2; i >= 0; --i) {
      const double pi = next, k = sh.e[i] * pi;
      if (i > 0) next = slot[(i - 1) * RAT_MAX_POLES + tid];
      G = pi + k * k * G;
      reinterpret_cast<float2 *>(slot)[i * RAT_MAX_POLES + tid] = make_float2((float)-k, (float)(wj * G));
    }
  }
  __syncthreads();
  // d has served: f of the rows that stand alone goes there
  for (int i = tid; i < n; i += NT)
    if (sh.dec[i]) sh.d[i] = pow(((double)g.scale * (double)a[(int64_t)i * n + i] - shift) + eps, -r_exp);
  // Row l of F runs from its diagonal entry to the left: G_{l,i} = -(e_i / pivot_i) G_{l,i+1}, every
  // pole by itself, two lanes sharing the poles of a row.  A lane's values are zero until its row begins.
  // F is kept as results of 16 x 16 matrix products: a wavefront has tile columns J = wave and CB - 1 - wave, element (j, I, u) is
  // row 16 I + lg + 4 u, column 16 J_j + li.
  const int lg = lane >> 4, li = lane & 15;
  const int tile[2] = {wave_u, CB - 1 - wave_u};
  tri_d4 F[2][CB];
  {
    const int l = tid >> 1;
    float val[PQ];
#pragma unroll
    for (int q = 0; q < PQ; ++q) val[q] = 0.f;
    const float4 *sl = reinterpret_cast<const float4 *>(slot + (tid & 1) * half);
    for (int ch = (n - 1) / TRI_CHUNK; ch >= 0; --ch) {
      // all 32 rows of a wavefront have begun, or some
      auto columns = [&](auto begun) {
        for (int i = min(n, (ch + 1) * TRI_CHUNK) - 1; i >= ch * TRI_CHUNK; --i) {
          float acc = 0.f;
#pragma unroll
          for (int q0 = 0; q0 < PQ; q0 += PQ_STEP)
            if (q0 < half) {
#pragma unroll
              for (int q = q0; q < q0 + PQ_STEP; q += 2) {
                const float4 s = sl[i * (RAT_MAX_POLES / 2) + q / 2];
                val[q] *= s.x;
                val[q + 1] *= s.z;
                if (!decltype(begun)::value && l == i) { val[q] = s.y; val[q + 1] = s.w; }
                acc += val[q] + val[q + 1];
              }
            }
          acc += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(acc), DPP_XOR1, 0xf, 0xf, true));
          if ((tid & 1) == 0) sh.fun.chunk[i - ch * TRI_CHUNK][l] = acc;
        }
      };
      if (32 * wave_u >= (ch + 1) * TRI_CHUNK) columns(BlockIndex<1>());
      else if (32 * wave_u + 31 >= ch * TRI_CHUNK) columns(BlockIndex<0>());
      __syncthreads();
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int I = 0; I < CB; ++I)
          if (min(I, tile[j]) == ch)             // all of its rows and columns lie in one 16 x 16 block
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int r = 16 * I + lg + 4 * u, c = 16 * tile[j] + li, mn = min(r, c), mx = max(r, c);
              F[j][I][u] = mx < n ? (double)sh.fun.chunk[mn % TRI_CHUNK][mx] : 0.0;
            }
      __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int I = 0; I < CB; ++I)
        if (16 * min(I, tile[j]) >= n) F[j][I] = (tri_d4){0.0, 0.0, 0.0, 0.0};      // no chunk of it
  }

  // ---- the eigenvector that is handled by itself: the part of F along v1 is replaced by f ----
  // F <- F - v q^T - q v^T with p = F v, q = p - (v.p + f) / 2 v
  if (deflate) {
    double *pb = sh.step.p;
    const double *v = sh.v1;
    double p[2] = {0.0, 0.0};
#pragma unroll
    for (int I = 0; I < CB; ++I)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double x = v[16 * I + lg + 4 * u];
        p[0] += F[0][I][u] * x; p[1] += F[1][I][u] * x;
      }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      p[j] += __shfl_xor(p[j], 16, 64); p[j] += __shfl_xor(p[j], 32, 64);
      if (lg == 0) pb[16 * tile[j] + li] = p[j];
    }
    __syncthreads();
    double vp = 0.0;
#pragma unroll
    for (int e = 0; e < (N + 63) / 64; ++e) {
      const int i = lane + 64 * e;
      if (N % 64 == 0 || i < N) vp += v[i] * pb[i];
    }
    const double K = 0.5 * (wave64_sum(vp) + pow((lam - shift) + eps, -r_exp));
    double vc[2], qc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) { vc[j] = v[16 * tile[j] + li]; qc[j] = p[j] - K * vc[j]; }
#pragma unroll
    for (int I = 0; I < CB; ++I)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double vr = v[16 * I + lg + 4 * u], qr = pb[16 * I + lg + 4 * u] - K * vr;
        F[0][I][u] -= vr * qc[0] + qr * vc[0]; F[1][I][u] -= vr * qc[1] + qr * vc[1];
      }
    __syncthreads();
  }

  // ---- X = Q F Q^T, 16 reflectors at a time, on the fp64 matrix cores ----
  // Group q: those with k + 1 in 16 q ... 16 q + 15, which are zero in front of row 16 q.  Their product is I - V T V^T, and
  //   F <- F - Y V^T - V Y^T,   Y = Z T^T - V (T M T^T) / 2,   Z = F V,   M = V^T Z.
  // Five barriers for 16 reflections, and no wavefront sums: one reflection at a time (two barriers, two sums over the lanes)
  // the kernel took 3011 us for 3000 matrices of up to 128 x 128, so 2673.  Lane l supplies A(l % 16, l / 16 + 4 u) and B(l / 16 + 4 u, l % 16) to step u of a product
  // and gets D(l / 16 + 4 u, l % 16): a result is the B operand of the next one as it lies, F also its own A operand.
  TriBack<N> &bk = sh.back;
  // entry (row, reflector 16 q + i - 1) of V
  auto entry = [&](int k, int at, int row) { return row == k + 1 ? 1.f : row > k + 1 && row < n ? sh.vs[at + row] : 0.f; };
  auto exists = [n](int k) { return k >= 0 && k <= n - 3; };
  // A matrix of one tile, in the smallest variant: one reflection at a time, F in 4 registers of the one wavefront and nothing in
  // LDS but the reflectors.  F <- F - v q^T - q v^T with q = tau p - tau^2 (v.p) / 2 v, p = F v, tau = 2 / v.v.  512 matrices of 4, 8, 12 and 16: 21.1,
  // 27.3, 33.6 and 40.0 us by groups of 16, 15.5, 23.3, 31.5 and 39.8 so.
  const bool one_tile = N == 32 && n <= 16;
  if (one_tile) {
    for (int k = n - 3; k >= 0; --k) {
      if (sh.beta[k] == 0.0) continue;
      const int at = offs(k);
      const double vc = (double)entry(k, at, li);
      double vr[4], pr[4], p = 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u) { vr[u] = (double)entry(k, at, lg + 4 * u); p = fma(F[0][0][u], vr[u], p); }
      const double tau = 2.0 * rcp_newton(row16_sum(vc * vc));
      p = rows_sum(p);
#pragma unroll
      for (int u = 0; u < 4; ++u) pr[u] = __shfl(p, lg + 4 * u, 64);
      const double K = 0.5 * tau * row16_sum(vc * p), q = tau * (p - K * vc);
#pragma unroll
      for (int u = 0; u < 4; ++u) F[0][0][u] -= vr[u] * q + tau * (pr[u] - K * vr[u]) * vc;
    }
  } else {
    // S = V^T V, then T by columns: T_jj = 2 / S_jj, T_ij = -T_jj sum_l T_il S_lj.  A wavefront does two groups
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int q = tile[j], k = 16 * q + li - 1, at = exists(k) ? offs(k) : 0;
      tri_d4 s = {0.0, 0.0, 0.0, 0.0};
      for (int r0 = 16 * q; r0 < n; r0 += 16)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double x = exists(k) ? (double)entry(k, at, r0 + lg + 4 * u) : 0.0;
          s = tri_mfma(x, x, s);
        }
      double *S = &bk.y[0][0] + 256 * q;
#pragma unroll
      for (int u = 0; u < 4; ++u) S[(lg + 4 * u) * 16 + li] = s[u];
    }
    __syncthreads();
    if (lg < 2) {
      const int q = lg == 0 ? tile[0] : tile[1];
      const double *S = &bk.y[0][0] + 256 * q;
      double T[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int k = 16 * q + j - 1;
        const bool is = exists(k) && sh.beta[max(k, 0)] != 0.0;
        const double tau = is ? 2.0 * rcp_newton(S[17 * j]) : 0.0;
        double x = 0.0;
#pragma unroll
        for (int l = 0; l < j; ++l) x += T[l] * S[l * 16 + j];
        T[j] = li == j ? tau : li < j ? -tau * x : 0.0;
        bk.t[q][j * 16 + li] = T[j];
      }
    }
  }
  for (int q = one_tile ? -1 : (n - 2) / 16; q >= 0; --q) {
    __syncthreads();                             // T; what the group before has read
    for (int e = tid; e < 16 * N; e += NT) {
      const int i = e / N, row = e % N, k = 16 * q + i - 1;
      bk.v[i][row] = exists(k) ? entry(k, offs(k), row) : 0.f;
    }
    __syncthreads();
    // Z^T, and the share of M of this wavefront's rows
    tri_d4 z[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}}, m = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int I = 0; I < CB; ++I)
      if (I >= q)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double x = (double)bk.v[li][16 * I + lg + 4 * u];
          z[0] = tri_mfma(x, F[0][I][u], z[0]); z[1] = tri_mfma(x, F[1][I][u], z[1]);
        }
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (tile[j] >= q) {
#pragma unroll
        for (int u = 0; u < 4; ++u) bk.y[lg + 4 * u][16 * tile[j] + li] = z[j][u];
        wavefront_order();                       // entries that other lanes of the wavefront have just written
#pragma unroll
        for (int u = 0; u < 4; ++u)
          m = tri_mfma((double)bk.v[li][16 * tile[j] + lg + 4 * u], bk.y[li][16 * tile[j] + lg + 4 * u], m);
      }
    wavefront_order();                           // and read
#pragma unroll
    for (int u = 0; u < 4; ++u) bk.y[lg + 4 * u][16 * tile[0] + li] = m[u];
    __syncthreads();
    // W = T M T^T / 2
    double t[4];
    tri_d4 W = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      t[u] = bk.t[q][(lg + 4 * u) * 16 + li];
      double x = 0.0;
#pragma unroll
      for (int e = 0; e < CB / 2; ++e) x += bk.y[lg + 4 * u][16 * e + li];       // M is symmetric
      W = tri_mfma(x, t[u], W);
    }
    {
      const tri_d4 mt = W;
      W = (tri_d4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int u = 0; u < 4; ++u) W = tri_mfma(t[u], mt[u], W);
    }
    __syncthreads();
    // -Y^T = W V^T - T Z^T, -V^T
    tri_d4 y[2];
    double v[2][4];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      y[j] = (tri_d4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int u = 0; u < 4; ++u) y[j] = tri_mfma(-t[u], z[j][u], y[j]);
#pragma unroll
      for (int u = 0; u < 4; ++u) v[j][u] = -(double)bk.v[lg + 4 * u][16 * tile[j] + li];
      if (tile[j] >= q)
#pragma unroll
        for (int u = 0; u < 4; ++u) y[j] = tri_mfma(-0.5 * W[u], v[j][u], y[j]);
#pragma unroll
      for (int u = 0; u < 4; ++u) bk.y[lg + 4 * u][16 * tile[j] + li] = -y[j][u];
    }
    __syncthreads();
#pragma unroll
    for (int I = 0; I < CB; ++I) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double yi = bk.y[lg + 4 * u][16 * I + li], vi = (double)bk.v[lg + 4 * u][16 * I + li];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if (tile[j] >= q) F[j][I] = tri_mfma(yi, v[j][u], F[j][I]);
          if (I >= q) F[j][I] = tri_mfma(vi, y[j][u], F[j][I]);
        }
      }
    }
  }
  __syncthreads();

  // ---- out: the lower triangle and its mirror image carry the same bits ----
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int e = 0; e < 4 * CB; ++e) {
      const int r = 16 * (e >> 2) + lg + 4 * (e & 3), c = 16 * tile[j] + li;
      if (r < n && c <= r) {
        double v = F[j][e >> 2][e & 3];
        if (lone && (sh.dec[r] || sh.dec[c])) v = r == c ? sh.d[r] : 0.0;
        sh.out[r][c] = (float)v;
      }
    }
  __syncthreads();
  float *x = g.x + (int64_t)b * g.x_stride;
  for (int e = tid; e < n * n; e += NT) {
    const int i = row_of(e), j = e - i * n;
    x[e] = i >= j ? sh.out[i][j] : sh.out[j][i];
  }
}

}  // namespace shampoo
