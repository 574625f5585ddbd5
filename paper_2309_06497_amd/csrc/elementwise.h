// Coalesced elementwise stages of the step (HBM-bandwidth bound):
//   prep_kernel       G1 = G + wd W (l2 weight decay), Gf <- beta1 Gf + (1-beta1) G1   (Sec. 3.1.1, 3.1.2)
//   graft_kernel      A <- A + G.^2 ; partial sums of ||Gf / (sqrt(A) + eps_g)||_F^2  (Sec. 2.4)
//   scale_kernel      per block: -||P_graft||_F / ||P_shampoo||_F from the partial sums
//   update_kernel     P = scale * P_shampoo (or -P_graft) ; M <- mu M + P ; W <- W + lr M (Sec. 3.1.3)
//   diag_kernel       1-D parameters: diagonal AdaGrad + momentum in one pass (Sec. 4.2.2)
// A block is addressed inside the caller's row-major tensors through its
// BlockDesc; rows of a block are contiguous runs, read as 4-element vectors
// when the block's origin and leading dimension allow it.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "gemm_mfma.h"
#include "group.h"

namespace shampoo {

constexpr int EW_THREADS = 256;

struct EwGeom {        // how 256 threads tile a block of m x n
  int32_t lanes_x_log2;   // threads along columns = 1 << lanes_x_log2 (each owns 4 columns per pass)
  int32_t rows_per_wg;
  int32_t chunks;         // workgroups per block = ceil(m / rows_per_wg)
};

struct EwArgs {
  const BlockDesc *desc;
  void *const *w_table;          // parameter pointers (float32)
  const void *const *g_table;    // gradients that feed the grafting state (G, or G + wd W)
  const void *const *gd_table;   // gradients that feed the directions (filtered gradient if beta1 > 0)
  float *a_state;                // grafting state, parameter layout, all parameters concatenated
  float *m_state;                // momentum state, same layout (nullptr when mu == 0)
  const float *p;                // [slot][m][n] Shampoo directions
  float *sg_partial;             // [slot][chunks]
  float *gmax_partial;           // graft_kernel: [slot][chunks] max |G| of the chunk, direction gradients (nullptr: not wanted)
  float *gmax;                   // [2][blocks]: largest element of state and direction gradients; zero between steps (graft_kernel: nullptr
                                 // where no product wants it)
  const float *scale;            // [slot]
  int32_t m, n, blocks;
  EwGeom geom;
  float graft_eps, mu, lr;
  float gd_scale;                // direction gradients are multiplied by this (bias correction, 1 = off)
  // grafting state A <- a_decay A + a_gain G.^2 and P_graft = Gf / (sqrt(a_bc A) + eps):
  // (1, 1, 1) AdaGrad; (beta_g, 1 - beta_g, 1) RMSprop; Adam adds a_bc = 1 / (1 - beta_g^(t+1))
  float a_decay, a_gain, a_bc;
  float wd_decoupled;            // update_kernel: P <- P - wd_decoupled * W (0 = off)
  int32_t nesterov;              // update_kernel: step with mu M + P instead of M
  int32_t sgd_graft;             // P_graft = G (no grafting state) instead of AdaGrad
  int32_t same_src;              // g_table and gd_table are the same tensors
  int32_t graft_only;            // update_kernel: use -P_graft instead of scale * P
  __device__ __forceinline__ void globals() { to_global(desc, w_table, g_table, gd_table, a_state, m_state, p, sg_partial, gmax_partial, gmax, scale); }
};

template <typename GT>
__device__ __forceinline__ void load_g4(const GT *g, bool vec, int valid, float v[4]) {
  if (vec) { Elem<GT>::load4(g, v); return; }
  if (valid == 4) { load_u4<GT>(g, *reinterpret_cast<float (*)[4]>(v)); return; }
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = e < valid ? Elem<GT>::load1(g + e) : 0.f;
}
// 16 bytes that this step touches once: marked as streaming, so that they do not displace what
// the next kernel wants to find in the caches
typedef float ew_floatx4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 nt_load4(const float *p) {
  const ew_floatx4 v = __builtin_nontemporal_load(reinterpret_cast<const ew_floatx4 *>(p));
  return make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void nt_store4(float *p, const float4 &v) {
  const ew_floatx4 x = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(x, reinterpret_cast<ew_floatx4 *>(p));
}
__device__ __forceinline__ void load_f4(const float *p, bool vec, int valid, float v[4]) {
  load_g4<float>(p, vec, valid, v);
}
__device__ __forceinline__ void store_f4(float *p, bool vec, int valid, const float v[4]) {
  if (vec) { *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]); return; }
  if (valid == 4) { store_u4(p, *reinterpret_cast<const float (*)[4]>(v)); return; }
#pragma unroll
  for (int e = 0; e < 4; ++e) if (e < valid) p[e] = v[e];
}

// The quads of four columns that a thread has, row by row, from (i, j) on: U of them at a time, so that their loads are in flight
// together whether they lie in one row or in several.
template <int V> struct BoolConst { static constexpr int value = V; };
template <int U> struct QuadWalk {
  int i[U], j[U];
  int row, col;
  __device__ __forceinline__ void next(int first_col, int n, int col_step, int row_step) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      i[u] = row; j[u] = col;
      col += col_step;
      if (col >= n) { col = first_col; row += row_step; }
    }
  }
};

// workgroups of a bucket: chunks * blocks, chunk index fastest.
// GS / GD: element types of the state-source and direction-source gradients.
template <typename GS, typename GD>
__global__ __launch_bounds__(EW_THREADS) void graft_kernel(const Group<EwArgs> grp) {
  __shared__ float red[2 * EW_THREADS / 64];
  int wg;
  const EwArgs g = group_pick(grp, wg);
  const int slot = wg / g.geom.chunks, chunk = wg - slot * g.geom.chunks, tid = threadIdx.x;
  if (slot >= g.blocks) return;
  const BlockDesc d = g.desc[slot];
  const GS *gp = global_ptr<const GS>(g.g_table[d.param]) + d.offset;
  const GD *dp = global_ptr<const GD>(g.gd_table[d.param]) + d.offset;
  float *ap = g.a_state + d.state_offset;
  const int ld = d.ld, n = g.n;
  const bool vec = ((ld & 3) == 0) && ((n & 3) == 0) && ((d.offset & 3) == 0) && ((d.state_offset & 3) == 0) &&
                   ((reinterpret_cast<uintptr_t>(g.g_table[d.param]) & 15) == 0) &&
                   ((reinterpret_cast<uintptr_t>(g.gd_table[d.param]) & 15) == 0);
  const int lx = g.geom.lanes_x_log2;
  const int tx = tid & ((1 << lx) - 1), ty = tid >> lx, ny = EW_THREADS >> lx;
  const int r0 = chunk * g.geom.rows_per_wg;
  const int r1 = min(r0 + g.geom.rows_per_wg, g.m);
  float ss = 0.f, gmax = 0.f, smax = 0.f;
  if (g.same_src && !g.sgd_graft) {
    // The common case, four quads at a time, every load requested before the first store.
    auto graft = [&](auto aligned) {
      constexpr bool VEC = decltype(aligned)::value != 0;
      constexpr int U = 4;
      QuadWalk<U> at;
      at.row = r0 + ty; at.col = tx * 4;
      while (at.row < r1 && at.col < n) {
        at.next(tx * 4, n, 4 << lx, ny);
        float gq[U][4], av[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {                 // rows past the end: the last one again, loads without a branch
          const int64_t e = (int64_t)min(at.i[u], r1 - 1) * ld + at.j[u];
          load_g4<GD>(dp + e, VEC, min(4, n - at.j[u]), gq[u]);
          if constexpr (VEC) { const float4 x = nt_load4(ap + e); av[u][0] = x.x; av[u][1] = x.y; av[u][2] = x.z; av[u][3] = x.w; }
          else load_f4(ap + e, false, min(4, n - at.j[u]), av[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (at.i[u] < r1) {
            const int valid = min(4, n - at.j[u]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float gv = gq[u][e];
              gmax = fmaxf(gmax, fabsf(gv));
              av[u][e] = g.a_decay * av[u][e] + g.a_gain * (gv * gv);
              const float pg = (gv * g.gd_scale) / (sqrtf(g.a_bc * av[u][e]) + g.graft_eps);
              if (VEC || e < valid) ss += pg * pg;
            }
            float *to = ap + (int64_t)at.i[u] * ld + at.j[u];
            if constexpr (VEC) nt_store4(to, make_float4(av[u][0], av[u][1], av[u][2], av[u][3]));
            else store_f4(to, false, valid, av[u]);
          }
      }
    };
    if (vec) graft(BoolConst<1>()); else graft(BoolConst<0>());
  } else
  for (int i = r0 + ty; i < r1; i += ny)
    for (int j = tx * 4; j < n; j += 4 << lx) {
      const int valid = min(4, n - j);
      float gv[4], dv[4], av[4];
      load_g4<GD>(dp + (int64_t)i * ld + j, vec, valid, dv);
      gmax = fmaxf(fmaxf(gmax, fmaxf(fabsf(dv[0]), fabsf(dv[1]))), fmaxf(fabsf(dv[2]), fabsf(dv[3])));
      if (g.same_src) {
#pragma unroll
        for (int e = 0; e < 4; ++e) gv[e] = dv[e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) dv[e] *= g.gd_scale;
      if (g.sgd_graft) {
#pragma unroll
        for (int e = 0; e < 4; ++e) if (e < valid) ss += dv[e] * dv[e];
        continue;
      }
      if (!g.same_src) {
        load_g4<GS>(gp + (int64_t)i * ld + j, vec, valid, gv);
        smax = fmaxf(fmaxf(smax, fmaxf(fabsf(gv[0]), fabsf(gv[1]))), fmaxf(fabsf(gv[2]), fabsf(gv[3])));
      }
      load_f4(ap + (int64_t)i * ld + j, vec, valid, av);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        av[e] = g.a_decay * av[e] + g.a_gain * (gv[e] * gv[e]);
        const float pg = dv[e] / (sqrtf(g.a_bc * av[e]) + g.graft_eps);
        if (e < valid) ss += pg * pg;
      }
      store_f4(ap + (int64_t)i * ld + j, vec, valid, av);
    }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  if (tid == 0) g.sg_partial[(int64_t)slot * g.geom.chunks + chunk] = (red[0] + red[1]) + (red[2] + red[3]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) { gmax = fmaxf(gmax, __shfl_xor(gmax, off, 64)); smax = fmaxf(smax, __shfl_xor(smax, off, 64)); }
  __syncthreads();
  if ((tid & 63) == 0) { red[tid >> 6] = gmax; red[EW_THREADS / 64 + (tid >> 6)] = smax; }
  __syncthreads();
  if (tid == 0) {
    gmax = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    smax = g.same_src ? gmax : fmaxf(fmaxf(red[4], red[5]), fmaxf(red[6], red[7]));
    if (g.gmax_partial) g.gmax_partial[(int64_t)slot * g.geom.chunks + chunk] = gmax;
    if (g.gmax) {
      // not negative, so that their bits order like integers and the result does not depend on the order
      atomicMax(reinterpret_cast<int *>(g.gmax + slot), __float_as_int(smax));
      atomicMax(reinterpret_cast<int *>(g.gmax + g.blocks + slot), __float_as_int(gmax));
    }
  }
}

struct ScaleArgs {
  const float *sg_partial; int32_t sg_count;   // per block
  const float *ssh_partial; int32_t ssh_count; // per block
  float *scale;    // [blocks]
  float *norms;    // [blocks][2]
  int32_t blocks;
  __device__ __forceinline__ void globals() { to_global(sg_partial, ssh_partial, scale, norms); }
};

// One wavefront per block; fixed summation order, so results are reproducible.
__global__ __launch_bounds__(64) void scale_kernel(const Group<ScaleArgs> grp) {
  int b;
  const ScaleArgs g = group_pick(grp, b);
  if (b >= g.blocks) return;
  const int lane = threadIdx.x;
  double sg = 0.0, ssh = 0.0;
  for (int i = lane; i < g.sg_count; i += 64) sg += (double)g.sg_partial[(int64_t)b * g.sg_count + i];
  for (int i = lane; i < g.ssh_count; i += 64) ssh += (double)g.ssh_partial[(int64_t)b * g.ssh_count + i];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    sg += __shfl_xor(sg, off, 64);
    ssh += __shfl_xor(ssh, off, 64);
  }
  if (lane == 0) {
    // zero (or non-finite) norms give a zero step for the block instead of NaN
    const bool ok = (sg > 0.0) && (ssh > 0.0) && (sg <= 1.0e300) && (ssh <= 1.0e300);
    g.scale[b] = ok ? (float)(-sqrt(sg / ssh)) : 0.f;
    g.norms[2 * b] = (float)sg;
    g.norms[2 * b + 1] = (float)ssh;
  }
}

// GD: element type of the direction-source gradients (read only in the grafting-only phase).
template <typename GD>
__global__ __launch_bounds__(EW_THREADS) void update_kernel(const Group<EwArgs> grp) {
  int wg;
  const EwArgs g = group_pick(grp, wg);
  const int slot = wg / g.geom.chunks, chunk = wg - slot * g.geom.chunks, tid = threadIdx.x;
  if (slot >= g.blocks) return;
  const BlockDesc d = g.desc[slot];
  float *wp = global_ptr<float>(g.w_table[d.param]) + d.offset;
  const GD *gp = global_ptr<const GD>(g.gd_table[d.param]) + d.offset;
  float *ap = g.a_state + d.state_offset;
  float *mp = g.m_state ? g.m_state + d.state_offset : nullptr;
  const int ld = d.ld, n = g.n;
  const float *pp = g.p + (int64_t)slot * g.m * n;
  const bool vec = ((ld & 3) == 0) && ((n & 3) == 0) && ((d.offset & 3) == 0) && ((d.state_offset & 3) == 0) &&
                   ((reinterpret_cast<uintptr_t>(g.w_table[d.param]) & 15) == 0) &&
                   ((reinterpret_cast<uintptr_t>(g.gd_table[d.param]) & 15) == 0);
  const int lx = g.geom.lanes_x_log2;
  const int tx = tid & ((1 << lx) - 1), ty = tid >> lx, ny = EW_THREADS >> lx;
  const int r0 = chunk * g.geom.rows_per_wg;
  const int r1 = min(r0 + g.geom.rows_per_wg, g.m);
  const float sc = g.graft_only ? 0.f : g.scale[slot];
  if (chunk == 0 && tid < 2) g.gmax[tid * g.blocks + slot] = 0.f;      // read by all products of the step by now
  if (!g.graft_only && mp) {
    // The common case, four quads at a time: all twelve 16-byte loads of a thread are
    // requested before the first store (a store between two loads would make the second one
    // wait: the compiler cannot tell that M, W and P do not overlap).
    auto update = [&](auto aligned) {
      constexpr bool VEC = decltype(aligned)::value != 0;
      constexpr int U = 4;
      QuadWalk<U> at;
      at.row = r0 + ty; at.col = tx * 4;
      while (at.row < r1 && at.col < n) {
        at.next(tx * 4, n, 4 << lx, ny);
        float pv[U][4], wv[U][4], mv[U][4];
        auto get = [&](const float *p, int u, float (&v)[4]) {
          if constexpr (VEC) { const float4 x = nt_load4(p); v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w; }
          else load_f4(p, false, min(4, n - at.j[u]), v);
        };
        auto put = [&](float *p, int u, const float (&v)[4]) {
          if constexpr (VEC) nt_store4(p, make_float4(v[0], v[1], v[2], v[3]));
          else store_f4(p, false, min(4, n - at.j[u]), v);
        };
#pragma unroll
        for (int u = 0; u < U; ++u) {                 // rows past the end: the last one again, loads without a branch
          const int i = min(at.i[u], r1 - 1);
          const int64_t e = (int64_t)i * ld + at.j[u];
          get(pp + (int64_t)i * n + at.j[u], u, pv[u]);
          get(wp + e, u, wv[u]);
          get(mp + e, u, mv[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (at.i[u] < r1) {
            const int64_t at_e = (int64_t)at.i[u] * ld + at.j[u];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              float p = pv[u][e] * sc;
              if (g.wd_decoupled != 0.f) p -= g.wd_decoupled * wv[u][e];
              mv[u][e] = g.mu * mv[u][e] + p;
              wv[u][e] += g.lr * (g.nesterov ? g.mu * mv[u][e] + p : mv[u][e]);
            }
            put(mp + at_e, u, mv[u]);
            put(wp + at_e, u, wv[u]);
          }
      }
    };
    if (vec) update(BoolConst<1>()); else update(BoolConst<0>());
    return;
  }
  for (int i = r0 + ty; i < r1; i += ny)
    for (int j = tx * 4; j < n; j += 4 << lx) {
      const int valid = min(4, n - j);
      float pv[4], wv[4], mv[4];
      if (g.graft_only) {
        float gv[4], av[4];
        load_g4<GD>(gp + (int64_t)i * ld + j, vec, valid, gv);
#pragma unroll
        for (int e = 0; e < 4; ++e) gv[e] *= g.gd_scale;
        if (g.sgd_graft) {
#pragma unroll
          for (int e = 0; e < 4; ++e) pv[e] = -gv[e];
        } else {
          load_f4(ap + (int64_t)i * ld + j, vec, valid, av);
#pragma unroll
          for (int e = 0; e < 4; ++e) pv[e] = -gv[e] / (sqrtf(g.a_bc * av[e]) + g.graft_eps);
        }
      } else {
        load_f4(pp + (int64_t)i * n + j, vec, valid, pv);
#pragma unroll
        for (int e = 0; e < 4; ++e) pv[e] *= sc;
      }
      load_f4(wp + (int64_t)i * ld + j, vec, valid, wv);
      if (g.wd_decoupled != 0.f) {
#pragma unroll
        for (int e = 0; e < 4; ++e) pv[e] -= g.wd_decoupled * wv[e];
      }
      if (mp) {
        load_f4(mp + (int64_t)i * ld + j, vec, valid, mv);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          mv[e] = g.mu * mv[e] + pv[e];
          wv[e] += g.lr * (g.nesterov ? g.mu * mv[e] + pv[e] : mv[e]);
        }
        store_f4(mp + (int64_t)i * ld + j, vec, valid, mv);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) wv[e] += g.lr * pv[e];
      }
      store_f4(wp + (int64_t)i * ld + j, vec, valid, wv);
    }
}

// 1-D parameters, cut into chunks of at most DIAG_CHUNK elements.
constexpr int DIAG_CHUNK = 4096;
struct DiagChunk {
  int32_t param;
  int32_t len;
  int64_t start;         // first element inside the parameter
  int64_t state_offset;  // offset of that element in the A / M state arrays
};
struct DiagArgs {
  const DiagChunk *chunks;
  void *const *w_table;
  const void *const *g_table;
  float *a_state, *m_state, *gf_state;   // gf_state: filtered gradient (nullptr when beta1 == 0)
  float graft_eps, mu, lr;
  float beta1, wd_l2, wd_decoupled;
  float gd_scale;        // bias correction of the filtered gradient (1 = off)
  float a_decay, a_gain, a_bc;   // as in EwArgs
  int32_t nesterov;
};

// One chunk, with the pointers of its parameter.  Four elements of a thread at a time, every load ahead of the stores.
template <typename GT>
__device__ __forceinline__ void diag_chunk(const DiagArgs &g, const DiagChunk &c, float *w, const GT *gp) {
  constexpr int U = 4;
  float *a = g.a_state + c.state_offset;
  float *m = g.m_state ? g.m_state + c.state_offset : nullptr;
  float *gf = g.gf_state ? g.gf_state + c.state_offset : nullptr;
  w += c.start;
  gp += c.start;
  for (int i0 = threadIdx.x; i0 < c.len; i0 += U * EW_THREADS) {
    float wv[U], gv[U], av[U], mv[U], fv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * EW_THREADS;
      if (i < c.len) {
        wv[u] = w[i]; gv[u] = Elem<GT>::load1(gp + i); av[u] = a[i];
        mv[u] = m ? m[i] : 0.f;
        fv[u] = gf ? gf[i] : 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * EW_THREADS;
      if (i >= c.len) break;
      if (g.wd_l2 != 0.f) gv[u] += g.wd_l2 * wv[u];
      const float an = g.a_decay * av[u] + g.a_gain * (gv[u] * gv[u]);
      a[i] = an;
      float dv = gv[u];
      if (gf) { dv = g.beta1 * fv[u] + (1.f - g.beta1) * gv[u]; gf[i] = dv; }
      float p = -(g.gd_scale * dv) / (sqrtf(g.a_bc * an) + g.graft_eps);
      if (g.wd_decoupled != 0.f) p -= g.wd_decoupled * wv[u];
      if (m) {
        const float mn = g.mu * mv[u] + p;
        m[i] = mn;
        p = g.nesterov ? g.mu * mn + p : mn;
      }
      w[i] = wv[u] + g.lr * p;
    }
  }
}
template <typename GT>
__global__ __launch_bounds__(EW_THREADS) void diag_kernel(const DiagArgs g) {
  const DiagChunk c = g.chunks[blockIdx.x];
  diag_chunk<GT>(g, c, global_ptr<float>(g.w_table[c.param]), global_ptr<const GT>(g.g_table[c.param]));
}

// 2-D parameters, flat chunks: G1 = G + wd W (if g1 != nullptr) and
// Gf <- beta1 Gf + (1 - beta1) G1 (if gf != nullptr); both in the A / M state layout.
struct PrepArgs {
  const DiagChunk *chunks;
  void *const *w_table;
  const void *const *g_table;
  float *g1, *gf;
  float wd_l2, beta1;
};

template <typename GT>
__global__ __launch_bounds__(EW_THREADS) void prep_kernel(const PrepArgs g) {
  const DiagChunk c = g.chunks[blockIdx.x];
  const float *w = global_ptr<const float>(g.w_table[c.param]) + c.start;
  const GT *gp = global_ptr<const GT>(g.g_table[c.param]) + c.start;
  for (int i = threadIdx.x; i < c.len; i += EW_THREADS) {
    float gv = Elem<GT>::load1(gp + i);
    if (g.g1) { gv += g.wd_l2 * w[i]; g.g1[c.state_offset + i] = gv; }
    if (g.gf) {
      const float f = g.beta1 * g.gf[c.state_offset + i] + (1.f - g.beta1) * gv;
      g.gf[c.state_offset + i] = f;
    }
  }
}

// Parameter and gradient pointers of one step, passed by value (the 4 KB of a kernel's arguments
// hold 240 pairs) and written to the tables that the other kernels read.
constexpr int POINTER_SET = 240;
struct PointerSet {
  void **w_table, **g_table;
  int32_t count;
  void *w[POINTER_SET], *g[POINTER_SET];
};
__global__ __launch_bounds__(256) void pointer_table_kernel(const PointerSet p) {
  const int i = threadIdx.x;
  if (i < p.count) { p.w_table[i] = p.w[i]; p.g_table[i] = p.g[i]; }
}

struct ClearArgs {
  float *p; int32_t n;
  __device__ __forceinline__ void globals() { to_global(p); }
};
__global__ __launch_bounds__(256) void clear_kernel(const Group<ClearArgs> grp) {
  int wg;
  const ClearArgs g = group_pick(grp, wg);
  const int i = wg * 256 + threadIdx.x;
  if (i < g.n) g.p[i] = 0.f;
}
__global__ __launch_bounds__(256) void fill_kernel(float *p, float v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = v;
}

// roots start as the identity: count matrices of n x n
__global__ __launch_bounds__(256) void eye_kernel(float *p, int32_t n, int64_t total) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int64_t e = i % ((int64_t)n * n);
  p[i] = (e / n == e % n) ? 1.f : 0.f;
}

}  // namespace shampoo
