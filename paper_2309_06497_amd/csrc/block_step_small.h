// Whole optimizer step of one small block (m, n <= 128) in a single workgroup.
//
// For blocks this small the step is bound by HBM traffic and launch count, not
// by the matrix cores: run stage by stage, the gradient block is read four
// times, the intermediate Lbar G makes a round trip through HBM, and a bucket
// costs eight launches.  Here one workgroup of 256 threads keeps the gradient
// block in LDS (68 KB of the 160 KB per CU, two workgroups per CU; 17 KB where all blocks are at
// most 64 x 64) and runs, on a step without root refresh (Sec. 3 complete pseudocode):
//   Gf <- beta1 Gf + (1 - beta1) G  (filtered gradients; otherwise Gf = G)           (Sec. 3.1.1)
//   A <- A + G.^2,  s_g = ||c1 Gf / (sqrt(A) + eps_g)||_F^2                           (Sec. 2.4)
//   L <- beta L + alpha G G^T,  R <- beta R + alpha G^T G                             (Sec. 3.1.1)
//   T = c1 Lbar Gf (kept in LDS, over G),  P_sh = T Rbar,  s_sh = ||P_sh||_F^2        (Sec. 2.3)
//   P = -sqrt(s_g / s_sh) P_sh [- wd W],  M <- mu M + P,  W <- W + lr M               (Sec. 2.4, 3.1.2, 3.1.3)
// Every tensor is read once and written once, of the factors the lower triangle (their upper halves are
// completed by mirror_upper_tiles_kernel when someone asks for them).
//
// Products.  Every operand is split into three bf16 terms in registers (bf16_planes.h: 8 + 8 + 8 bits, all of a float32;
// five or six vector instructions an element) and a product is six v_mfma_f32_32x32x16_bf16, 192 cycles for 16 values of k
// where the float32 matrix cores take 512; an unfiltered bf16 gradient is one term by itself.  The splitting and the
// matrix cores then take about the same time, and together less than the memory traffic.  Sums of the
// factors: those of 32 values of k start from zero, the small products first (two roundings of full size, against sixteen on
// the float32 matrix cores), and go into float64.
// G is scaled by a power of two where its largest element is outside 2^-40 ... 2^40, so that no term underflows.
//
// One step of 512 blocks of 128 x 128, of ResNet-50 in blocks of 128, and of nine blocks of at most 64 x 64, float32 matrix
// cores with slabs of Lbar and Rbar through LDS, and this: 170, 517, 62 us and 126, 382, 19 us.
//
// Lbar and Rbar are read along their rows straight into registers (they are symmetric), RING steps of 16 ahead: no
// slabs, and four barriers in all.  What the next phase needs is requested before the products of the present one.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include "elementwise.h"
#include "gemm_mfma.h"
#include "bf16_terms.h"
#include "lds_dma.h"

namespace shampoo {

constexpr int SB = 128;            // largest block edge handled here
constexpr int SB_HALF = 64;        // the small variant
constexpr int SB_THREADS = 256;
constexpr int SB_POINTERS = 224;   // of parameters that travel with the launch
static_assert(SB_THREADS == EW_THREADS, "chunks of 1-D parameters");

// One block handled by the kernel: where it sits in the caller's tensors and where its state
// sits in the workspace (byte offsets).  Blocks of all small buckets share one launch.
struct SmallBlock {
  BlockDesc d;
  int32_t m, n;
  int64_t off_L, off_R, off_Linv, off_Rinv;   // m x m, n x n float32
  int64_t off_P;                              // m x n: Lbar G Rbar, kept for inspection
  int64_t off_norms;                          // 2 floats
  int32_t filter;                             // the filtered gradient is updated here (otherwise prep_kernel has)
};

struct SmallStepArgs {
  const SmallBlock *blocks;      // one per workgroup, largest first
  unsigned char *ws;
  void *const *w_table;
  const void *const *g_table;
  float *a_state, *m_state;      // m_state nullptr when mu == 0
  float *gf_state;               // filtered gradient (FILT kernels)
  double alpha_d, beta_d;        // factor update weights
  float graft_eps, mu, lr, wd_decoupled;
  float a_decay, a_gain, a_bc;   // grafting state A <- a_decay A + a_gain G.^2, root of a_bc A
  float beta1, gd_scale;         // filter, and its bias correction c1
  int32_t nesterov;
  int32_t fp32;                  // Lbar G Rbar on the float32 matrix cores
  int32_t n_blocks;              // workgroups behind them: chunks of 1-D parameters
  DiagArgs diag;
  // Parameter and gradient pointers of up to SB_POINTERS parameters by value: a step that needs nothing else is one launch
  // (one 256 x 128 weight and a bias: 18.0 us with a launch for the tables and one for the bias, 15.4 us so)
  int32_t by_value;
  void *w_ptr[SB_POINTERS];
  const void *g_ptr[SB_POINTERS];
};
static_assert(sizeof(SmallStepArgs) <= 4096, "kernel arguments");

// sums / maxima over the workgroup in a fixed order; every thread gets the result.  red: 4 floats not in use.
__device__ __forceinline__ float sb_reduce(float v, float *red, int tid) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// A range of memory that is read and written by byte offsets; what lies past its end is read as zero and not written, so
// that the edges of a block need no branches.
typedef __amdgpu_buffer_rsrc_t SbRange;
constexpr int SB_NOWHERE = INT32_MIN;        // an offset past the end of every range
__device__ __forceinline__ SbRange sb_range(const void *p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(uniform_ptr(p)), 0, (int)min(bytes, (int64_t)INT32_MAX), 0x00020000);
}
__device__ __forceinline__ float sb_get(SbRange r, int at) { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, at, 0, 0)); }
__device__ __forceinline__ void sb_put(SbRange r, int at, float x) { __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, at, 0, 0); }
// Eight consecutive floats of a root.  Past the end of a row they are the next one's: the operand that they meet is zero there.
__device__ __forceinline__ floatx8 sb_get8(SbRange r, int at) {
  const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, at, 0, 0), y = __builtin_amdgcn_raw_buffer_load_b128(r, at + 16, 0, 0);
  floatx8 f;
#pragma unroll
  for (int e = 0; e < 4; ++e) { f[e] = __uint_as_float(x[e]); f[4 + e] = __uint_as_float(y[e]); }
  return f;
}

// Rows 32 I .. 32 I + 31, columns 32 J .. (one tile, or two) of F <- beta F + alpha S, on and below the diagonal;
// S = G G^T (WHICH = 0, dim = m, K = n) or G^T G (WHICH = 1, dim = n, K = m).  The old values are requested before the
// products are formed.
template <int WHICH, int LD, bool ONE>
__device__ __forceinline__ void sb_factor(const float *Gs, float *F, int dim, int K, int I, int J, bool two, double alpha, double beta,
                                          int l32, int khalf) {
  const int row0 = 32 * I, col0 = 32 * J, stride = 4 * dim;
  const SbRange f = sb_range(F, (int64_t)dim * stride);
  // element v of tile t: this offset + (8 (v / 4) + v % 4) rows
  int at[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int j = col0 + 32 * t + l32;
    at[t] = j < dim && (t == 0 || two) ? (row0 + 4 * khalf) * stride + 4 * j : SB_NOWHERE;
  }
  // no branch around them, or they would be waited for where it ends
  float old[2][16];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) old[t][v] = sb_get(f, beta != 0.0 ? at[t] + (8 * (v >> 2) + (v & 3)) * stride : SB_NOWHERE);
  double sum[2][16];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[t][v] = 0.0;
  auto operand = [&](int first, int k) {
    return WHICH == 0 ? lds_row8<LD>(Gs, first + l32, k + 8 * khalf) : lds_col8<LD>(Gs, k + 8 * khalf, first + l32);
  };
  // 32 values of k from zero accumulators (G is zero from K on): both sets of small products, then both h h'
#pragma unroll 1
  for (int k = 0; k < K; k += 32) {
    floatx16 acc[2] = {};
    bf16x8 ah[2], bh[2][2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      Bf16Terms a, b0, b1;
      bf16_split<ONE>(operand(row0, k + 16 * s), a);
      if (I == J) b0 = a; else bf16_split<ONE>(operand(col0, k + 16 * s), b0);
      ah[s] = a.h; bh[s][0] = b0.h;
      if constexpr (!ONE) acc[0] = bf16_small_products<false, false>(a, b0, acc[0]);
      if (two) {
        if (I == J + 1) b1 = a; else bf16_split<ONE>(operand(col0 + 32, k + 16 * s), b1);
        bh[s][1] = b1.h;
        if constexpr (!ONE) acc[1] = bf16_small_products<false, false>(a, b1, acc[1]);
      }
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) acc[0] = bf16_mfma(ah[s], bh[s][0], acc[0]);
    if (two)
#pragma unroll
      for (int s = 0; s < 2; ++s) acc[1] = bf16_mfma(ah[s], bh[s][1], acc[1]);
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[0][v] += (double)acc[0][v];
    if (two)
#pragma unroll
      for (int v = 0; v < 16; ++v) sum[1][v] += (double)acc[1][v];
  }
  // not converted to float64 before the products: that would wait for them there
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) asm volatile("" : "+v"(old[t][v]));
  // of a tile on the diagonal the lower half
  const bool diag[2] = {I == J, I == J + 1};
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int i = 8 * (v >> 2) + (v & 3);
      const float x = (float)(alpha * sum[t][v] + beta * (double)old[t][v]);
      sb_put(f, diag[t] && l32 > i + 4 * khalf ? SB_NOWHERE : at[t] + i * stride, x);
    }
}

// The lower triangle of tiles of a factor as jobs of one tile or two beside each other: rows of tiles 3, 3, 2, 1, and the single ones of
// rows 2 and 0.  Of the tiles rows that exist, the job `q` (counted among those of its kind): row, first column.
__device__ __forceinline__ int sb_pairs(int tiles) { return tiles >= 4 ? 4 : tiles == 3 ? 2 : tiles == 2 ? 1 : 0; }
__device__ __forceinline__ int sb_singles(int tiles) { return tiles >= 3 ? 2 : 1; }

// GT: element type of the caller's gradients; CAP: no block is larger; FILT: directions from the filtered gradient.
// grid: one workgroup per entry of g.blocks and per chunk of g.diag.
template <typename GT, int CAP, bool FILT>
__global__ __launch_bounds__(SB_THREADS, 2) void block_step_small_kernel(const SmallStepArgs g) {
  constexpr int LD = CAP + 4;
  constexpr int GV = CAP * CAP / 4 / SB_THREADS;   // vectors of 4 elements of a block per thread
  constexpr int VPR = CAP / 4, RPP = SB_THREADS / VPR;   // vectors per row; rows between a thread's vectors
  constexpr int TT = CAP / 64;                     // tiles of 32 per wavefront and direction, at most
  constexpr int RING = CAP == 128 ? 4 : CAP / 16;
  constexpr bool BF = sizeof(GT) == 2;
  __shared__ __align__(16) float Gs[CAP * LD];     // s G, then s Gf, then T; zero outside m x n
  __shared__ float red[4][4];

  const int slot = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, khalf = lane >> 5;
  auto w_of = [&](int32_t param) { return global_ptr<float>(g.by_value ? g.w_ptr[param] : g.w_table[param]); };
  auto g_of = [&](int32_t param) { return global_ptr<const GT>(g.by_value ? g.g_ptr[param] : g.g_table[param]); };
  if (slot >= g.n_blocks) {
    const DiagChunk c = g.diag.chunks[slot - g.n_blocks];
    diag_chunk<GT>(g.diag, c, w_of(c.param), g_of(c.param));
    return;
  }
  const SmallBlock sbk = g.blocks[slot];
  const int m = sbk.m, n = sbk.n;
  const BlockDesc d = sbk.d;
  float *norms = reinterpret_cast<float *>(g.ws + sbk.off_norms);
  const GT *gp = g_of(d.param) + d.offset;
  float *wp = w_of(d.param) + d.offset;
  float *ap = g.a_state + d.state_offset;
  float *mp = g.m_state ? g.m_state + d.state_offset : nullptr;
  float *fp = FILT ? g.gf_state + d.state_offset : nullptr;
  const int ld = d.ld;

  // ---- G -> LDS, filter, grafting state and graft norm on the way (each element once).  A thread has vectors of four
  // columns of every RPP-th row; the last vector of a row that does not end with it begins earlier, so that it repeats
  // elements of the one before (both store the same values there).  Blocks of less than four columns: element by element.
  float ss = 0.f, gmax = 0.f, fmx = 0.f;
  const int vi = tid / VPR, vj = (tid % VPR) * 4, back = max(0, min(3, vj + 4 - n));     // first column: vj - back; `back` of the four are repeated
  const bool vec = n >= 4, mine = vec && vj < n;
  auto element = [&](float gv, float &fv, float &av, bool fresh) {
    if constexpr (FILT) { if (sbk.filter) fv = g.beta1 * fv + (1.f - g.beta1) * gv; } else fv = gv;
    av = g.a_decay * av + g.a_gain * (gv * gv);
    const float pg = (fv * g.gd_scale) / (sqrtf(g.a_bc * av) + g.graft_eps);
    if (fresh) ss += pg * pg;
    gmax = fmaxf(gmax, fabsf(gv));
    fmx = fmaxf(fmx, fabsf(fv));
  };
  // (x0 x1 x2 x3) without the repeated ones, zeros behind
  auto align = [&](float (&x)[4]) {
    if (back & 1) { x[0] = x[1]; x[1] = x[2]; x[2] = x[3]; x[3] = 0.f; }
    if (back & 2) { x[0] = x[2]; x[1] = x[3]; x[2] = 0.f; x[3] = 0.f; }
  };
  {
    // every load is issued before the first store, so the whole block costs one memory round trip
    float gv[GV][4], av[GV][4];
    const int64_t first = (int64_t)vi * ld + vj - back;
#pragma unroll
    for (int u = 0; u < GV; ++u) {
#pragma unroll
      for (int e = 0; e < 4; ++e) gv[u][e] = 0.f;
      if (mine && vi + RPP * u < m) {
        load_u4<GT>(gp + first + (int64_t)(RPP * u) * ld, gv[u]);
        load_u4<float>(ap + first + (int64_t)(RPP * u) * ld, av[u]);
      }
    }
    wavefront_order();                           // repeated elements: read by both lanes before either stores them
#pragma unroll
    for (int u = 0; u < GV; ++u)
      if (mine && vi + RPP * u < m) {
        float fv[4];
        const int64_t at = first + (int64_t)(RPP * u) * ld;
        if constexpr (FILT) { load_u4<float>(fp + at, fv); wavefront_order(); }
#pragma unroll
        for (int e = 0; e < 4; ++e) element(gv[u][e], fv[e], av[u][e], e >= back);
        if constexpr (FILT) { if (sbk.filter) store_u4(fp + at, fv); }
        store_u4(ap + at, av[u]);
      }
    if (!vec)
      for (int x = tid; x < m * n; x += SB_THREADS) {
        const int64_t at = (int64_t)(x / n) * ld + x % n;
        float fv = 0.f, a = ap[at];
        if constexpr (FILT) fv = fp[at];
        element(Elem<GT>::load1(gp + at), fv, a, true);
        if constexpr (FILT) { if (sbk.filter) fp[at] = fv; }
        ap[at] = a;
      }
    // the scale, known to all before anything is put into LDS
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { gmax = fmaxf(gmax, __shfl_xor(gmax, off, 64)); fmx = fmaxf(fmx, __shfl_xor(fmx, off, 64)); ss += __shfl_xor(ss, off, 64); }
    if (lane == 0) { red[0][wave] = ss; red[1][wave] = gmax; red[2][wave] = fmx; }
    __syncthreads();
    ss = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    gmax = fmaxf(fmaxf(red[1][0], red[1][1]), fmaxf(red[1][2], red[1][3]));
    fmx = fmaxf(fmaxf(red[2][0], red[2][1]), fmaxf(red[2][2], red[2][3]));
    const float sg = range_scale(gmax);
#pragma unroll
    for (int u = 0; u < GV; ++u) {
      align(gv[u]);
      *reinterpret_cast<float4 *>(&Gs[(vi + RPP * u) * LD + vj]) = make_float4(gv[u][0] * sg, gv[u][1] * sg, gv[u][2] * sg, gv[u][3] * sg);
    }
    __syncthreads();
    if (!vec) {
      for (int x = tid; x < m * n; x += SB_THREADS) Gs[(x / n) * LD + x % n] = sg * Elem<GT>::load1(gp + (int64_t)(x / n) * ld + x % n);
      __syncthreads();
    }
    if (tid == 0) norms[0] = ss;
  }
  const int mt = (m + 31) >> 5, nt = (n + 31) >> 5;

  // ---- factor updates (Gs is read-only here): the pairs of tiles of L, those of R, then the single tiles, dealt out in turn
  {
    float *Lp = reinterpret_cast<float *>(g.ws + sbk.off_L), *Rp = reinterpret_cast<float *>(g.ws + sbk.off_R);
    const double inv_s = 1.0 / (double)range_scale(gmax), alpha = g.alpha_d * (inv_s * inv_s);
    const int pl = sb_pairs(mt), pr = sb_pairs(nt), sl = sb_singles(mt), total = pl + pr + sl + sb_singles(nt);
    for (int q = wave; q < total; q += 4) {
      const bool two = q < pl + pr;
      int k = two ? q : q - pl - pr;
      const bool right = k >= (two ? pl : sl);
      if (right) k -= two ? pl : sl;
      const int t = right ? nt : mt;
      // pairs (3, 0) (3, 2) (2, 0) (1, 0); singles (2, 2) (0, 0)
      const int p = k + 4 - sb_pairs(t), I = two ? (p < 2 ? 3 : 4 - p) : (t >= 3 && k == 0 ? 2 : 0), J = two ? (p == 1 ? 2 : 0) : I;
      if (!right) sb_factor<0, LD, BF>(Gs, Lp, m, n, I, J, two, alpha, g.beta_d, l32, khalf);
      else sb_factor<1, LD, BF>(Gs, Rp, n, m, I, J, two, alpha, g.beta_d, l32, khalf);
    }
  }

  // ---- how the wavefronts share an m x n result: 2 x 2 of them with up to 2 x 2 tiles each, or all four along the
  // longer side where the other has two tiles or one
  int r0, c0;
  bool r_two = false, c_two = false;
  if (TT == 1 || (mt <= 2 && nt <= 2)) { r0 = 32 * (wave >> 1); c0 = 32 * (wave & 1); }
  else if (nt <= 2) { r0 = 32 * wave; c0 = 0; c_two = nt == 2; }
  else if (mt <= 2) { r0 = 0; c0 = 32 * wave; r_two = mt == 2; }
  else { r0 = 64 * (wave >> 1); c0 = 64 * (wave & 1); r_two = r0 + 32 < m; c_two = c0 + 32 < n; }
  const bool active = r0 < m && c0 < n;


  // ---- the filtered gradient takes the place of G; every thread reads back what it has written itself
  const float sf = FILT ? range_scale(fmx) : range_scale(gmax);
  if constexpr (FILT) {
    float fv[GV][4];
#pragma unroll
    for (int u = 0; u < GV; ++u) {
#pragma unroll
      for (int e = 0; e < 4; ++e) fv[u][e] = 0.f;
      if (mine && vi + RPP * u < m) { load_u4<float>(fp + (int64_t)(vi + RPP * u) * ld + vj - back, fv[u]); align(fv[u]); }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < GV; ++u)
      *reinterpret_cast<float4 *>(&Gs[(vi + RPP * u) * LD + vj]) = make_float4(fv[u][0] * sf, fv[u][1] * sf, fv[u][2] * sf, fv[u][3] * sf);
    __syncthreads();
    if (!vec) {
      for (int x = tid; x < m * n; x += SB_THREADS) Gs[(x / n) * LD + x % n] = sf * fp[(int64_t)(x / n) * ld + x % n];
      __syncthreads();
    }
  }

  floatx16 acc[TT][TT];
  floatx8 ring[RING][TT];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
      for (int j = 0; j < TT; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  };
  // one step of 16 values of k, the small products first.  BONE: b holds bf16 values
  auto multiply = [&](const floatx8 (&x)[TT], const floatx8 (&y)[TT], auto bone) {
    constexpr bool BONE = decltype(bone)::value;
    if (g.fp32) {                        // uniform: the caller wants the float32 matrix cores
#pragma unroll
      for (int i = 0; i < TT; ++i)
#pragma unroll
        for (int j = 0; j < TT; ++j)
          if ((i == 0 || r_two) && (j == 0 || c_two)) acc[i][j] = fp32_products(x[i], y[j], acc[i][j]);
      return;
    }
    Bf16Terms a[TT], b[TT];
#pragma unroll
    for (int i = 0; i < TT; ++i) if (i == 0 || r_two) bf16_split<false>(x[i], a[i]);
#pragma unroll
    for (int j = 0; j < TT; ++j) if (j == 0 || c_two) bf16_split<BONE>(y[j], b[j]);
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
      for (int j = 0; j < TT; ++j)
        if ((i == 0 || r_two) && (j == 0 || c_two))
          acc[i][j] = bf16_mfma(a[i].h, b[j].h, bf16_small_products<false, BONE>(a[i], b[j], acc[i][j]));
  };
  // ---- T = c1 Lbar G: A(i, k) = Lbar[i][k] from memory, B(k, j) = G[k][j] from LDS
  const SbRange Li = sb_range(g.ws + sbk.off_Linv, (int64_t)m * m * 4), Ri = sb_range(g.ws + sbk.off_Rinv, (int64_t)n * n * 4);
  auto request_l = [&](int s, int k) {
#pragma unroll
    for (int i = 0; i < TT; ++i)
      if (k < m && (i == 0 || r_two)) ring[s][i] = sb_get8(Li, ((r0 + 32 * i + l32) * m + k + 8 * khalf) * 4);
  };
  auto request_r = [&](int s, int k) {
#pragma unroll
    for (int j = 0; j < TT; ++j)
      if (k < n && (j == 0 || c_two)) ring[s][j] = sb_get8(Ri, ((c0 + 32 * j + l32) * n + k + 8 * khalf) * 4);
  };
  if (active) {
    clear();
#pragma unroll
    for (int s = 0; s < RING; ++s) request_l(s, 16 * s);
    for (int k0 = 0; k0 < m; k0 += 16 * RING)
#pragma unroll
      for (int s = 0; s < RING; ++s) {
        const int k = k0 + 16 * s;
        if (k < m) {
          floatx8 x[TT], y[TT];
#pragma unroll
          for (int i = 0; i < TT; ++i) x[i] = ring[s][i];
          request_l(s, k + 16 * RING);
#pragma unroll
          for (int j = 0; j < TT; ++j) if (j == 0 || c_two) y[j] = lds_col8<LD>(Gs, k + 8 * khalf, c0 + 32 * j + l32);
          multiply(x, y, std::integral_constant<bool, BF && !FILT>());
        }
      }
#pragma unroll
    for (int s = 0; s < RING; ++s) request_r(s, 16 * s);
  }
  __syncthreads();        // every wavefront has finished reading G
  if (active) {
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
      for (int j = 0; j < TT; ++j)
        if ((i == 0 || r_two) && (j == 0 || c_two))
#pragma unroll
          for (int v = 0; v < 16; ++v)
            Gs[(r0 + 32 * i + 8 * (v >> 2) + 4 * khalf + (v & 3)) * LD + c0 + 32 * j + l32] = g.gd_scale * acc[i][j][v];
  }
  __syncthreads();        // T is in place
  // ---- P_sh = T Rbar: A(i, k) = T[i][k] from LDS, B(k, j) = Rbar[j][k] from memory
  float wv[TT][TT][16], mv[TT][TT][16];
  const int64_t span = ((int64_t)(m - 1) * ld + n) * 4;
  const SbRange wr = sb_range(wp, span), mr = sb_range(mp, mp ? span : 0), pr = sb_range(g.ws + sbk.off_P, (int64_t)m * n * 4);
  // element v of tile (x, y): row_of(x, v), column c0 + 32 y + l32; rows past the end lie past the ranges
  auto row_of = [&](int x, int v) { return r0 + 32 * x + 8 * (v >> 2) + 4 * khalf + (v & 3); };
  auto offset = [&](int x, int y, int v, int stride) {
    const int i = row_of(x, v), j = c0 + 32 * y + l32;
    return i < m && j < n ? (i * stride + j) * 4 : SB_NOWHERE;
  };
  auto request_w = [&]() {
#pragma unroll
    for (int x = 0; x < TT; ++x)
#pragma unroll
      for (int y = 0; y < TT; ++y)
        if ((x == 0 || r_two) && (y == 0 || c_two))
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int at = offset(x, y, v, ld);
            wv[x][y][v] = sb_get(wr, at);
            mv[x][y][v] = sb_get(mr, at);
          }
  };
  float sp = 0.f;
  const float inv_sf = 1.f / sf;
  if (active) {
    clear();
    if constexpr (TT == 1) request_w();
    for (int k0 = 0; k0 < n; k0 += 16 * RING)
#pragma unroll
      for (int s = 0; s < RING; ++s) {
        const int k = k0 + 16 * s;
        if (k < n) {
          floatx8 x[TT], y[TT];
#pragma unroll
          for (int j = 0; j < TT; ++j) y[j] = ring[s][j];
          request_r(s, k + 16 * RING);
#pragma unroll
          for (int i = 0; i < TT; ++i) if (i == 0 || r_two) x[i] = lds_row8<LD>(Gs, r0 + 32 * i + l32, k + 8 * khalf);
          multiply(x, y, std::integral_constant<bool, false>());
        }
      }
    if constexpr (TT > 1) request_w();
    // ---- norm, scale, momentum and parameter update straight from the accumulators
#pragma unroll
    for (int x = 0; x < TT; ++x)
#pragma unroll
      for (int y = 0; y < TT; ++y)
        if ((x == 0 || r_two) && (y == 0 || c_two))
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const float p = acc[x][y][v] * inv_sf;
            acc[x][y][v] = p;
            if (row_of(x, v) < m && c0 + 32 * y + l32 < n) sp += p * p;
          }
  }
  sp = sb_reduce(sp, red[3], tid);
  if (tid == 0) norms[1] = sp;
  if (!active) return;
  // zero (or non-finite) norms give a zero step for the block instead of NaN
  const bool ok = (ss > 0.f) && (sp > 0.f) && (ss <= 3.0e38f) && (sp <= 3.0e38f);
  const float sc = ok ? (float)(-sqrt((double)ss / (double)sp)) : 0.f;
#pragma unroll
  for (int x = 0; x < TT; ++x)
#pragma unroll
    for (int y = 0; y < TT; ++y)
      if ((x == 0 || r_two) && (y == 0 || c_two))
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float psh = acc[x][y][v], w = wv[x][y][v];
          const int at = offset(x, y, v, ld);
          sb_put(pr, offset(x, y, v, n), psh);
          float pv = sc * psh;
          if (g.wd_decoupled != 0.f) pv -= g.wd_decoupled * w;
          if (mp) {
            const float mnew = g.mu * mv[x][y][v] + pv;
            sb_put(mr, at, mnew);
            pv = g.nesterov ? g.mu * mnew + pv : mnew;
          }
          sb_put(wr, at, w + g.lr * pv);
        }
}

}  // namespace shampoo
