// Host side of libshampoo: configuration checks, block planner, workspace
// layout, kernel launches and the extern "C" boundary declared in shampoo.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <tuple>
#include <new>
#include <optional>
#include <utility>
#include <vector>

#include "../../include/shampoo.h"
#include "bf16_planes.h"
#include "block_step_small.h"
#include "congruence_f64.h"
#include "diag_shampoo.h"
#include "eigh_jacobi.h"
#include "elementwise.h"
#include "gemm_f16x2.h"
#include "gemm_mfma.h"
#include "gram_split.h"
#include "group.h"
#include "newton_root.h"
#include "root_band.h"
#include "root_tridiag.h"
#include "syrk_bf16.h"
#include "tensor_blocks.h"

using namespace shampoo;

// Scratch of shampoo_root_inverse_static: the block solver's working arrays (float64 copy of
// the matrices, accumulated rotations, pivot blocks, flags) for as many matrices at a time as
// fit.  One copy per GPU the library runs on, held until the process ends.  In host code the
// name is only a handle for hipGetSymbolAddress: kernels are given the address obtained there.
static __device__ __align__(256) unsigned char scratch[SHAMPOO_STATIC_SCRATCH_BYTES];

namespace {

constexpr int64_t MAX_BLOCK_SIZE = 8192;
constexpr size_t ALIGN = 256;
constexpr size_t EIG_CHUNK_BYTES = (size_t)3 << 30;   // W + Qt of one chunk of the block solver

inline size_t align_up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }

#define HIP_TRY(expr)                          \
  do {                                         \
    hipError_t e_ = (expr);                    \
    if (e_ != hipSuccess) return SHAMPOO_ERR_HIP; \
  } while (0)

// ---------------------------------------------------------------------------
// Planner (Sec. 4.2.1 blocking)
// ---------------------------------------------------------------------------
struct Block {
  int32_t param;
  int64_t row0, col0;
  int32_t m, n;
  int32_t bucket, slot;
  // tensor blocks (Sec. 2.3): start and size along the third and fourth dimension, and where
  // the block sits in the block-contiguous copy of the parameter that the kernels work on
  int64_t s3 = 0, s4 = 0;
  int32_t d3 = 1, d4 = 1;
  int64_t voff = 0;
  bool tensor = false;
};
// How a parameter is worked on after merging of small dimensions (Sec. 4.2.1).
enum { P_VECTOR = 0, P_MATRIX = 1, P_TENSOR = 2 };
struct PShape {
  int kind = P_VECTOR;
  int64_t rows = 1, cols = 1;   // P_MATRIX: the (merged) shape; P_VECTOR: rows = length
  int64_t d[4] = {1, 1, 1, 1};  // P_TENSOR: the merged dimensions
  int modes = 0;                // P_TENSOR: 3 or 4, or 1 when everything merged into one dimension
  int64_t elems() const { return kind == P_TENSOR ? d[0] * d[1] * d[2] * d[3] : rows * cols; }
};
struct Bucket {
  int32_t m, n, count;
  // byte offsets into the workspace
  size_t off_L, off_R, off_Linv, off_Rinv, off_P, off_desc, off_sgp, off_sshp, off_scale, off_norms;
  // bf16_mfma buckets: both roots as two scaled fp16 planes, or three bf16 ones, what the scales
  // are made from (matrix_stats_kernel of both roots, max |G| per piece of a block) and the
  // scales themselves
  size_t off_Linvp = 0, off_Rinvp = 0, off_stat_l = 0, off_stat_r = 0, off_gmaxp = 0, off_s_g = 0, off_t_scale = 0, off_inv_ts = 0;
  size_t off_QtL = 0, off_QtR = 0;   // warm start: eigenvectors of the previous refresh, [count][np][np] float32
  size_t off_Gt = 0;     // 16-bit transpose of the bucket's gradient blocks (bf16, or scaled fp16 where the fp16 products follow), made by the factor update and
                         // read again by the first preconditioning product of the same step
  bool planes = false;
  // three: float32 directions, from three bf16 planes of every operand; split_factor: of float32 gradients that feed the
  // factors too, which then take the planes of the block both ways round.  Planes of a block live in T, of
  // plane_chunk blocks at a time: cols, the transpose, and behind it rows, the block as it lies, or T = Lbar G
  bool three = false, split_factor = false, cols_wait = false;   // cols_wait: the factor update's cols serve the products too
  int32_t plane_chunk = 0;
  size_t off_gmax = 0;            // [2][count]: largest |element| of a block's gradients (factors, directions), zero between steps
  size_t off_t = 0, off_t2 = 0;   // this bucket's part of the scratch arrays T and T2
  int32_t set = 0;                // buckets of a set are worked on together (their parts do not overlap)
  EwGeom geom;
  int32_t tiles_m, tiles_n;
  bool bf16_mfma;   // shapes, offsets and leading dimensions allow the bf16 matrix-core factor update
  // diagonal Shampoo (Sec. 4.2.3): the factor of that side is a vector (its diagonal); such a
  // bucket holds whole parameters, one per slot
  bool diagL = false, diagR = false;
  int32_t col_segs = 1, rows_per_seg = 0;   // row segments of the column-sum reduction
  // tensor blocks d1 x d2 x d3 (x d4): the elementwise kernels see them as m x n = d1 x (d2 d3 d4)
  // matrices inside a block-contiguous copy of the parameter; L belongs to the first
  // dimension, R to the last, mid[0] (and mid[1] for order 4) to the ones between
  bool t3 = false;
  int32_t td[4] = {1, 1, 1, 1}, modes = 0;
  size_t off_mid[2] = {0, 0}, off_midinv[2] = {0, 0}, off_desc3 = 0;
  int32_t split3 = 1;   // row ranges of the (N / d_last) x d_last unfolding whose Gram matrices are formed separately
  bool whole() const { return diagL || diagR; }
  bool wide = false;   // of a parameter so wide that the bytes of a block's rows span more than 2^31
  bool small() const { return m <= SB && n <= SB && !whole() && !t3 && !wide; }   // one workgroup per block (block_step_small.h)
  int32_t dlast() const { return modes > 1 ? td[modes - 1] : 1; }
  int32_t rdim() const { return t3 ? dlast() : n; }
  size_t l_elems() const { return diagL ? (size_t)m : (size_t)m * m; }
  size_t r_elems() const { return diagR ? (size_t)n : (size_t)rdim() * rdim(); }
};
struct Plan {
  std::vector<Block> blocks;
  std::vector<Bucket> buckets;
  std::vector<std::vector<int32_t>> param_blocks;  // per parameter: indices into blocks (row-major)
  std::vector<int64_t> param_state_offset;         // element offset of each parameter in A / M
  std::vector<DiagChunk> diag_chunks;   // 1-D parameters
  std::vector<DiagChunk> prep_chunks;   // 2-D parameters, flat (used by the l2 / filtering pre-pass); the first n_prep_rest
  int64_t n_prep_rest = 0;              // of them of parameters that are not made of small blocks only
  std::vector<PShape> pshape;           // per parameter
  int64_t total_elems = 0;
  int n_sets = 0;                       // of buckets (layout)
};

// Merging of small dimensions (Sec. 4.2.1) and the resulting kind of parameter.  Returns
// SHAMPOO_OK, or the error for a shape that is out of range.
int param_shape(const shampoo_config *c, int i, PShape &ps) {
  const int nd = c->ndim[i];
  if (nd < 1 || nd > SHAMPOO_MAX_NDIM) return SHAMPOO_ERR_SHAPE;
  const int64_t *sh = c->shape + (size_t)SHAMPOO_MAX_NDIM * i;
  for (int k = 0; k < nd; ++k) {
    if (sh[k] < 1) return SHAMPOO_ERR_SHAPE;
    if (sh[k] > (int64_t)1 << 30) return SHAMPOO_ERR_UNSUPPORTED;
  }
  ps = PShape();
  if (nd == 1) { ps.kind = P_VECTOR; ps.rows = sh[0]; return SHAMPOO_OK; }
  if (nd == 2) { ps.kind = P_MATRIX; ps.rows = sh[0]; ps.cols = sh[1]; return SHAMPOO_OK; }
  int64_t merged[SHAMPOO_MAX_NDIM];
  int cnt = 0;
  int64_t cur = sh[0];
  for (int k = 1; k < nd; ++k) {
    // a dimension of size 1 changes no product and always merges
    if (cur * sh[k] <= c->block_size || sh[k] == 1 || cur == 1) cur *= sh[k];
    else { merged[cnt++] = cur; cur = sh[k]; }
  }
  merged[cnt++] = cur;
  if (cnt == 2) { ps.kind = P_MATRIX; ps.rows = merged[0]; ps.cols = merged[1]; return SHAMPOO_OK; }
  ps.kind = P_TENSOR;
  ps.modes = cnt;
  for (int k = 0; k < cnt; ++k) ps.d[k] = merged[k];
  if ((double)ps.d[0] * (double)ps.d[1] * (double)ps.d[2] * (double)ps.d[3] > (double)((int64_t)1 << 40)) return SHAMPOO_ERR_UNSUPPORTED;
  // one block is indexed with 32-bit products of its sizes
  double block_elems = 1.0;
  for (int k = 0; k < cnt; ++k) block_elems *= (double)std::min<int64_t>(ps.d[k], c->block_size);
  if (block_elems > (double)(1 << 30)) return SHAMPOO_ERR_UNSUPPORTED;
  return SHAMPOO_OK;
}

// p = 1 / r when that is 1, 2, 4 or 8 (the powers the coupled Newton iteration forms by
// repeated squaring), else 0
int newton_p_of(float r) {
  for (int p : {1, 2, 4, 8})
    if (std::fabs(1.0 / (double)r - (double)p) <= 1e-4 * p) return p;
  return 0;
}

int check_config(const shampoo_config *c) {
  if (!c || !c->ndim || !c->shape) return SHAMPOO_ERR_NULL;
  if (c->n_params < 1) return SHAMPOO_ERR_SHAPE;
  if (c->block_size < 1) return SHAMPOO_ERR_SHAPE;
  if (c->block_size > MAX_BLOCK_SIZE) return SHAMPOO_ERR_UNSUPPORTED;
  for (int i = 0; i < c->n_params; ++i) {
    PShape ps;
    const int rc = param_shape(c, i, ps);
    if (rc) return rc;
  }
  if (!(c->beta2 > 0.f && c->beta2 <= 1.f)) return SHAMPOO_ERR_HYPER;
  if (!(c->epsilon > 0.f) || !std::isfinite(c->epsilon)) return SHAMPOO_ERR_HYPER;
  if (!(c->root_exponent > 0.f) || !std::isfinite(c->root_exponent)) return SHAMPOO_ERR_HYPER;
  if (c->precondition_frequency < 1 || c->start_preconditioning_step < 0) return SHAMPOO_ERR_HYPER;
  if (!(c->graft_epsilon >= 0.f) || !std::isfinite(c->graft_epsilon)) return SHAMPOO_ERR_HYPER;
  if (!(c->momentum >= 0.f && c->momentum < 1.f)) return SHAMPOO_ERR_HYPER;
  if (c->grad_dtype != SHAMPOO_GRAD_F32 && c->grad_dtype != SHAMPOO_GRAD_BF16) return SHAMPOO_ERR_HYPER;
  if (!(c->beta1 >= 0.f && c->beta1 < 1.f)) return SHAMPOO_ERR_HYPER;
  if (!(c->weight_decay >= 0.f) || !std::isfinite(c->weight_decay)) return SHAMPOO_ERR_HYPER;
  if (c->grafting_type < SHAMPOO_GRAFT_ADAGRAD || c->grafting_type > SHAMPOO_GRAFT_ADAM) return SHAMPOO_ERR_HYPER;
  if ((c->grafting_type == SHAMPOO_GRAFT_RMSPROP || c->grafting_type == SHAMPOO_GRAFT_ADAM) &&
      !(c->grafting_beta2 > 0.f && c->grafting_beta2 <= 1.f))
    return SHAMPOO_ERR_HYPER;
  if (c->large_dim_method < SHAMPOO_LARGE_DIM_BLOCKING || c->large_dim_method > SHAMPOO_LARGE_DIM_DIAGONAL)
    return SHAMPOO_ERR_HYPER;
  if (c->large_dim_method == SHAMPOO_LARGE_DIM_DIAGONAL)
    for (int i = 0; i < c->n_params; ++i) {
      PShape ps;
      param_shape(c, i, ps);
      if (ps.kind == P_MATRIX && (ps.rows > INT32_MAX / 2 || ps.cols > INT32_MAX / 2)) return SHAMPOO_ERR_UNSUPPORTED;
    }
  if (c->root_method != SHAMPOO_ROOT_EIGH && c->root_method != SHAMPOO_ROOT_NEWTON) return SHAMPOO_ERR_HYPER;
  if (c->precond_matrix_cores != SHAMPOO_MATRIX_CORES_AUTO && c->precond_matrix_cores != SHAMPOO_MATRIX_CORES_FP32)
    return SHAMPOO_ERR_HYPER;
  if (c->root_method == SHAMPOO_ROOT_NEWTON) {
    if (c->newton_tolerance < 0.f || !std::isfinite(c->newton_tolerance)) return SHAMPOO_ERR_HYPER;
    if (c->newton_max_iterations < 0 || c->newton_max_iterations > 1000) return SHAMPOO_ERR_HYPER;
    if (newton_p_of(c->root_exponent) == 0) return SHAMPOO_ERR_UNSUPPORTED;
    for (int i = 0; i < c->n_params; ++i) {
      PShape ps;
      param_shape(c, i, ps);
      if (ps.kind == P_TENSOR && newton_p_of(2.f * c->root_exponent / (float)ps.modes) == 0) return SHAMPOO_ERR_UNSUPPORTED;
    }
  }
  return SHAMPOO_OK;
}

EwGeom make_geom(int m, int n) {
  EwGeom g;
  const int vecs = (n + 3) / 4;
  int lx = 0;
  while ((1 << lx) < vecs && lx < 6) ++lx;
  g.lanes_x_log2 = lx;
  const int ny = EW_THREADS >> lx;
  const int cols_per_pass = 4 << lx;
  const int passes = (n + cols_per_pass - 1) / cols_per_pass;
  // about 8192 elements per workgroup, a whole number of thread rows
  int rows = std::max(1, 8192 / (cols_per_pass * passes));
  rows = (rows + ny - 1) / ny * ny;
  g.rows_per_wg = rows;
  g.chunks = (m + rows - 1) / rows;
  return g;
}

void make_plan(const shampoo_config *c, Plan &p) {
  const int64_t b = c->block_size;
  // (m, n, diagonal sides | tensor, d2, d3, d4, order of the tensor) -> bucket; the order gives the root's exponent, also
  // where a block has a single index along the last dimension
  std::map<std::tuple<int, int, int, int, int, int, int>, int> bucket_of;
  p.param_blocks.assign(c->n_params, {});
  p.param_state_offset.assign(c->n_params, 0);
  p.pshape.assign(c->n_params, PShape());
  int64_t off = 0;
  auto bucket_for = [&](int m, int n, int flags, int d2, int d3, int d4, int modes) {
    auto key = std::make_tuple(m, n, flags, d2, d3, d4, modes);
    auto it = bucket_of.find(key);
    if (it == bucket_of.end()) {
      Bucket bk{};
      bk.m = m; bk.n = n; bk.count = 0;
      bk.diagL = (flags & 1) != 0; bk.diagR = (flags & 2) != 0;
      bk.t3 = (flags & 4) != 0; bk.td[0] = m; bk.td[1] = d2; bk.td[2] = d3; bk.td[3] = d4; bk.modes = modes;
      bucket_of[key] = (int)p.buckets.size();
      p.buckets.push_back(bk);
      it = bucket_of.find(key);
    }
    return it->second;
  };
  for (int i = 0; i < c->n_params; ++i) {
    p.param_state_offset[i] = off;
    PShape &ps = p.pshape[i];
    param_shape(c, i, ps);
    const int64_t rows = ps.rows, cols = ps.cols;
    const bool large = ps.kind == P_MATRIX && (rows > b || cols > b);
    // 1-D parameters, and under the "adagrad" large-dimension method (Sec. 4.2.2) every
    // matrix with a dimension above the block size, take the diagonal path on their entries
    if (ps.kind == P_VECTOR || (large && c->large_dim_method == SHAMPOO_LARGE_DIM_ADAGRAD)) {
      const int64_t len = rows * cols;
      for (int64_t s = 0; s < len; s += DIAG_CHUNK) {
        DiagChunk dc;
        dc.param = i;
        dc.len = (int32_t)std::min<int64_t>(DIAG_CHUNK, len - s);
        dc.start = s;
        dc.state_offset = off + s;
        p.diag_chunks.push_back(dc);
      }
      off += (len + 3) / 4 * 4;
      continue;
    }
    const int64_t elems = ps.elems();
    for (int64_t st = 0; st < elems; st += DIAG_CHUNK) {
      DiagChunk dc;
      dc.param = i;
      dc.len = (int32_t)std::min<int64_t>(DIAG_CHUNK, elems - st);
      dc.start = st;
      dc.state_offset = off + st;
      p.prep_chunks.push_back(dc);
    }
    if (ps.kind == P_TENSOR) {
      // every dimension cut into pieces of at most b; blocks in row-major order of their
      // indices.  All pieces before the last one of a dimension are full, which gives the
      // offset of a block inside the block-contiguous copy in closed form.
      const int64_t D1 = ps.d[0], D2 = ps.d[1], D3 = ps.d[2], D4 = ps.d[3];
      const int64_t k1n = (D1 + b - 1) / b, k2n = (D2 + b - 1) / b, k3n = (D3 + b - 1) / b, k4n = (D4 + b - 1) / b;
      for (int64_t k1 = 0; k1 < k1n; ++k1)
        for (int64_t k2 = 0; k2 < k2n; ++k2)
          for (int64_t k3 = 0; k3 < k3n; ++k3)
            for (int64_t k4 = 0; k4 < k4n; ++k4) {
              Block blk;
              blk.param = i; blk.tensor = true;
              blk.row0 = k1 * b; blk.col0 = k2 * b; blk.s3 = k3 * b; blk.s4 = k4 * b;
              blk.m = (int32_t)std::min<int64_t>(b, D1 - blk.row0);
              blk.n = (int32_t)std::min<int64_t>(b, D2 - blk.col0);
              blk.d3 = (int32_t)std::min<int64_t>(b, D3 - blk.s3);
              blk.d4 = (int32_t)std::min<int64_t>(b, D4 - blk.s4);
              blk.voff = blk.row0 * D2 * D3 * D4 + (int64_t)blk.m * (blk.col0 * D3 * D4) +
                         (int64_t)blk.m * blk.n * (blk.s3 * D4) + (int64_t)blk.m * blk.n * blk.d3 * blk.s4;
              blk.bucket = bucket_for(blk.m, blk.n * blk.d3 * blk.d4, 4, blk.n, blk.d3, blk.d4, ps.modes);
              blk.slot = p.buckets[blk.bucket].count++;
              p.param_blocks[i].push_back((int32_t)p.blocks.size());
              p.blocks.push_back(blk);
            }
      off += (elems + 3) / 4 * 4;
      continue;
    }
    // diagonal Shampoo (Sec. 4.2.3): the parameter stays whole, one "block"
    const bool whole = large && c->large_dim_method == SHAMPOO_LARGE_DIM_DIAGONAL;
    const int64_t bb = whole ? std::max(rows, cols) : b;
    const int flags = whole ? ((rows > b ? 1 : 0) | (cols > b ? 2 : 0)) : 0;
    const int64_t km = (rows + bb - 1) / bb, kn = (cols + bb - 1) / bb;
    for (int64_t bi = 0; bi < km; ++bi)
      for (int64_t bj = 0; bj < kn; ++bj) {
        Block blk;
        blk.param = i;
        blk.row0 = bi * bb;
        blk.col0 = bj * bb;
        blk.m = (int32_t)std::min<int64_t>(bb, rows - blk.row0);
        blk.n = (int32_t)std::min<int64_t>(bb, cols - blk.col0);
        blk.bucket = bucket_for(blk.m, blk.n, flags, 1, 1, 1, 0);
        blk.slot = p.buckets[blk.bucket].count++;
        p.param_blocks[i].push_back((int32_t)p.blocks.size());
        p.blocks.push_back(blk);
      }
    off += (rows * cols + 3) / 4 * 4;
  }
  p.total_elems = off;
  for (auto &bk : p.buckets)
    bk.bf16_mfma = (bk.m % 8 == 0) && (bk.n % 8 == 0) && bk.count <= 65535 && !bk.whole() && !bk.t3;
  for (const Block &blk : p.blocks) {
    if (blk.tensor) continue;
    const int64_t ld = p.pshape[blk.param].cols;
    if (ld % 8 != 0 || (blk.row0 * ld + blk.col0) % 8 != 0) p.buckets[blk.bucket].bf16_mfma = false;
    if (ld > (int64_t)1 << 22) p.buckets[blk.bucket].wide = true;
  }
  auto only_small = [&](int32_t param) {
    for (int32_t k : p.param_blocks[param]) if (!p.buckets[p.blocks[k].bucket].small()) return false;
    return true;
  };
  std::vector<char> is_small(c->n_params);
  for (int i = 0; i < c->n_params; ++i) is_small[i] = only_small(i);
  p.n_prep_rest = std::stable_partition(p.prep_chunks.begin(), p.prep_chunks.end(), [&](const DiagChunk &d) { return !is_small[d.param]; }) -
                  p.prep_chunks.begin();
  for (auto &bk : p.buckets) {
    if (bk.t3 && bk.modes >= 3) {
      // the factor of the last dimension sums over N / d_last rows into one small tile per
      // block: split the rows (whole slices of the first index) so that the launch fills the GPU
      const int64_t inner = (int64_t)bk.n / bk.dlast();   // rows of the unfolding per slice of the first index
      for (int sdiv = 1; sdiv <= std::min(bk.m, 64); ++sdiv)
        if (bk.m % sdiv == 0 && (int64_t)(bk.m / sdiv) * inner >= 64 && (int64_t)sdiv * bk.dlast() <= (int64_t)bk.m * inner &&
            (int64_t)bk.count * sdiv <= 1 << 20)
          bk.split3 = sdiv;
    }
    bk.geom = make_geom(bk.m, bk.n);
    bk.tiles_m = (bk.m + BM - 1) / BM;
    bk.tiles_n = (bk.n + BN - 1) / BN;
    bk.col_segs = std::max(1, std::min(64, bk.m / 256));
    bk.rows_per_seg = (bk.m + bk.col_segs - 1) / bk.col_segs;
  }
}

// Whole-parameter and tensor buckets are launched with the block index as grid.y / grid.z.
int check_plan(const Plan &p) {
  for (const auto &b : p.buckets)
    if ((b.whole() || b.t3) && b.count > 65535) return SHAMPOO_ERR_UNSUPPORTED;
  return SHAMPOO_OK;
}

// ---------------------------------------------------------------------------
// Root-inverse workspace (shared by the optimizer and the stand-alone call)
// ---------------------------------------------------------------------------
constexpr int CONGRUENCE_PANEL = 256;   // columns of T = A Qt^T formed at a time (warm start)

// Whether roots of n x n matrices with exponent r can do without eigenvectors (root_band.h), where no caller asks for
// them or for eigenvalues.  Exponents above 0.4 up to n = 224 stay with Jacobi, which is the more accurate one there
// (r = 1/2, factors of one gradient, n = 129 ... 224: 3.4e-7 ... 4.4e-7 against 4.0e-7 ... 4.6e-7; the other way round from
// 256 on).
bool band_serves(int n, float r) {
  RatTable table;
  return n > JAC_SMALL_MAX && n <= BAND_MAX_N && !(r > 0.4f && n <= 224) && rat_table(r, table);
}

// Workspace of the band reduction: 33 MB for a matrix of 1024, of which 20 are the eliminations of all poles.  Chunks of one size take up to
// BAND_CHUNK_BYTES (128 of 1024), the pass over all sizes of a refresh up to band_pass_bytes().
constexpr size_t BAND_CHUNK_BYTES = (size_t)4 << 30;
struct BandLayout {
  int32_t np = 0, nb = 0, chunk = 0;
  size_t off_w = 0, off_vall = 0, off_vp = 0, off_z = 0, off_y = 0, off_t = 0, off_part = 0, off_tall = 0, off_dblk = 0, off_cblk = 0,
         off_kf = 0, off_gf = 0, off_v1 = 0, off_ok = 0, off_dec = 0, off_skip = 0, off_meta = 0;
  size_t bytes = 0;
};
// of `cnt` matrices
BandLayout band_layout_of(int n, int cnt) {
  BandLayout e;
  if (n > BAND_MAX_N) return e;
  e.np = (n + BAND - 1) / BAND * BAND; e.nb = e.np / BAND;
  const size_t np = e.np, blk = (size_t)e.nb * BAND * BAND, parts = (np + BAND_ZROWS - 1) / BAND_ZROWS;
  size_t off = 0;
  auto take = [&](size_t per) { const size_t at = off; off += align_up(per * (size_t)cnt); return at; };
  e.off_w = take(np * np * 8); e.off_vall = take(np * np * 4);
  e.off_vp = take(np * BAND * 8); e.off_z = take(np * BAND * 8); e.off_y = take(np * BAND * 8);
  e.off_t = take(BAND * BAND * 8); e.off_part = take(parts * BAND * BAND * 8); e.off_tall = take(blk * 4);
  e.off_dblk = take(blk * 8); e.off_cblk = take(blk * 8);
  e.off_kf = take(blk * 8 * BAND_SLOTS); e.off_gf = take(blk * 8 * BAND_SLOTS);
  e.off_v1 = take(np * 8); e.off_ok = take(2 * BAND_SHIFTS * 4); e.off_dec = take(np * 4); e.off_skip = take(4); e.off_meta = take(sizeof(BandMeta));
  e.chunk = cnt;
  e.bytes = off;
  return e;
}
// A panel is one workgroup per matrix, and its chain of columns does not take longer for more matrices while there is a CU for each of
// them: a matrix of 1024 for every CU, 8 GiB, which is 3 % of the GPU's memory.  Refreshes in passes of 4, 8 and 16 GiB: 128
// matrices of 1024 23.4, 20.7, 20.7 ms; 256 of them 43.9, 38.4, 38.5; 800 132, 122, 117; 48 of 2048 56.2, 46.2, 47.1; 96 102, 94.0, 85.6; 512 of
// 512 18.4 in all; 250 of 1024 and 250 of 700 65.3, 60.9, 58.6.
size_t band_pass_bytes() { return band_layout_of(1024, 256).bytes; }
// of a chunk of the `batch`
BandLayout band_layout(int n, int batch) {
  const BandLayout one = band_layout_of(n, 1);
  if (!one.bytes) return one;
  return band_layout_of(n, (int)std::max<size_t>(1, std::min<size_t>({(size_t)batch, (size_t)32768, BAND_CHUNK_BYTES / one.bytes})));
}

struct EigLayout {
  BandLayout band;         // bytes = 0: not available
  int32_t np = 0, chunk = 0;
  bool warm = false;       // block solver: room for the float64 panel of the congruence W = Qt A Qt^T
  size_t off_w = 0, off_qt = 0, off_j = 0, off_ident = 0, off_j16 = 0, off_rot = 0, off_dmax = 0, off_failed = 0, off_f = 0, off_t = 0;
  size_t bytes = 0;
};

// Offsets for chunks of `chunk` matrices of the block solver (np already set).
void eig_offsets(EigLayout &e) {
  const size_t mat = (size_t)e.np * e.np * sizeof(float);
  size_t off = 0;
  e.off_w = off; off += align_up(2 * mat * e.chunk);
  e.off_qt = off; off += align_up(mat * e.chunk);
  const int hp = e.np / JAC_PIV;
  // rotation blocks and flags of two rounds (the Q^T update of a meeting of two super-columns
  // reads both): [2][chunk][hp]
  e.off_j = off; off += align_up(2 * (size_t)e.chunk * hp * JAC_PIV * JAC_PIV * sizeof(float));
  e.off_ident = off; off += align_up(2 * (size_t)e.chunk * hp * sizeof(int32_t));
  e.off_j16 = off; off += align_up(2 * (size_t)e.chunk * hp * 2 * JAC_PIV * JAC_PIV * sizeof(uint16_t));   // the same blocks, transposed, as two fp16 planes
  e.off_rot = off; off += align_up((size_t)e.chunk * JAC_OUTER_SWEEPS * sizeof(int32_t));
  e.off_dmax = off; off += align_up(2 * (size_t)e.chunk * sizeof(float));   // largest |diagonal entry|, largest absolute row sum
  e.off_failed = off; off += align_up(3 * (size_t)e.chunk * sizeof(int32_t));   // failed, done, skip (failed | done)
  e.off_f = off; off += align_up(2 * (size_t)e.chunk * e.np * sizeof(float));   // weights of the reconstruction; float32 eigenvalues of matrices that skip the float64 phase
  if (e.warm) { e.off_t = off; off += align_up((size_t)e.chunk * e.np * std::min(e.np, CONGRUENCE_PANEL) * sizeof(double)); }
  e.bytes = off;
}

// budget: bytes that the W and Qt arrays of one chunk may take (the other arrays are small);
// hard_cap != 0: the whole layout must fit into that many bytes (bytes = 0 in the result if
// not even one matrix does).
// band: with room for the band reduction (callers that can take it: band_serves, no eigenvectors wanted).
EigLayout eig_layout(int n, int batch, bool band, size_t budget = EIG_CHUNK_BYTES, size_t hard_cap = 0) {
  EigLayout e;
  e.warm = n > JAC_SMALL_MAX;   // the float64 panel serves the warm start and the mixed-precision cold solve alike
  if (n <= JAC_SMALL_MAX) {     // LDS solver: no scratch in device memory
    e.chunk = batch;
    e.off_failed = 0;
    e.bytes = align_up((size_t)std::max(batch, 1) * sizeof(int32_t));
    return e;
  }
  e.np = (n + JAC_PIV - 1) / JAC_PIV * JAC_PIV;
  const size_t mat = (size_t)e.np * e.np * sizeof(float);
  // W is float64, Qt float32: 3 float-sized matrices per solve
  e.chunk = (int)std::max<size_t>(1, std::min<size_t>(std::min<size_t>((size_t)batch, 32768), budget / (3 * mat)));
  eig_offsets(e);
  if (hard_cap) {
    while (e.bytes > hard_cap && e.chunk > 1) { --e.chunk; eig_offsets(e); }
    if (e.bytes > hard_cap) e.bytes = 0;
  } else if (band) {
    e.band = band_layout(n, batch);
    e.bytes = std::max(e.bytes, e.band.bytes);
  }
  return e;
}

// One launch of a kernel for the buckets added to it (group.h), or several where they are more than an argument table
// holds.  Nothing is launched before flush: what the kernel reads may be written by a launch that is still to come.
// Extra: further arguments, of RESERVE bytes.
template <typename Args, int RESERVE = 0, typename... Extra> struct Batch {
  using Kernel = void (*)(const Group<Args, RESERVE>, Extra...);
  struct Entry { Args args; int64_t workgroups; };
  Kernel kernel; int threads; hipStream_t s;
  std::vector<Entry> entries;
  Batch(Kernel k, int threads_, hipStream_t s_) : kernel(k), threads(threads_), s(s_) {}
  int add(const Args &a, int64_t workgroups) {
    if (workgroups > ((int64_t)1 << 30) - NUM_XCD) return SHAMPOO_ERR_UNSUPPORTED;
    if (workgroups > 0) entries.push_back(Entry{a, (workgroups + NUM_XCD - 1) / NUM_XCD * NUM_XCD});
    return SHAMPOO_OK;
  }
  int flush(const Extra &...extra) {
    Group<Args, RESERVE> g;
    for (size_t at = 0; at < entries.size();) {
      int64_t total = 0;
      g.count = 0;
      while (at < entries.size() && g.count < group_max<Args, RESERVE>() && total + entries[at].workgroups <= (int64_t)1 << 30) {
        g.a[g.count] = entries[at].args;
        g.first[g.count++] = (int32_t)total;
        total += entries[at++].workgroups;
      }
      hipLaunchKernelGGL(kernel, dim3((unsigned)total), dim3(threads), 0, s, g, extra...);
      HIP_TRY(hipGetLastError());
    }
    entries.clear();
    return SHAMPOO_OK;
  }
};

// Products of several buckets with gemm_mfma_kernel, in tiles of 128 x 128 or of 64 x 64.  Sets the counts of tiles, and those of
// the partial sums of squares that the caller wants to know.
// The smaller tile reads and splits its operands twice as often, but has four workgroups on a CU instead of two and four times as
// many: it is taken where the larger would leave half of the GPU's 512 places empty or fill them but once or twice, and where
// k is so short that a tile is little but its latency.  Step, large and small tiles: one layer of 331 in blocks of 1024 (float32) 418 and
// 223 us, of 526 in blocks of 512 301 and 215, one matrix of 191 144 and 82; two layers of 900, where the
// products have 576 tiles, 1225 and 1100, with those of 2048 in small tiles too 1190; ResNet-50 with convolution tensors, products
// over 128 of 6200 tiles, 893 and 843.
constexpr int64_t GEMM_FEW_TILES = 1024;
constexpr int GEMM_SHORT_K = 128;

constexpr int64_t OVERLAP_STAGED = 4 << 20;

struct GemmKernels { Batch<GemmArgs>::Kernel large, small; };
template <int AO, int BO, typename TA, typename TB, int EPI, bool ACC64 = false, bool FP32 = false> constexpr GemmKernels gemm_kernels() {
  return {gemm_mfma_kernel<AO, BO, TA, TB, EPI, false, ACC64, FP32>, gemm_mfma_kernel<AO, BO, TA, TB, EPI, false, ACC64, FP32, GEMM_SMALL>};
}
template <int EPI> struct GemmBatch {
  struct Entry { GemmArgs g; int *parts; int first_row; };
  GemmKernels kernels; hipStream_t s;
  std::vector<Entry> entries;
  GemmBatch(GemmKernels k, hipStream_t s_) : kernels(k), s(s_) {}
  // first_row (EPI_SYRK): the rows in front of it may stay as they are
  void add(const GemmArgs &g, int *parts = nullptr, int first_row = 0) { entries.push_back(Entry{g, parts, first_row}); }
  static void tile(Entry &e, int size) {
    GemmArgs &g = e.g;
    const int skipped = e.first_row / size;
    g.tiles_m = (g.M + size - 1) / size; g.tiles_n = (g.N + size - 1) / size;
    g.tile0 = skipped * (skipped + 1) / 2;
    g.tiles = EPI == EPI_SYRK ? g.tiles_m * (g.tiles_m + 1) / 2 - g.tile0 : g.tiles_m * g.tiles_n;
  }
  int flush() {
    int64_t total = 0;
    int k = 0;
    for (Entry &e : entries) { tile(e, BM); total += (int64_t)e.g.tiles * e.g.batch; k = std::max(k, e.g.K); }
    const bool small = total <= GEMM_FEW_TILES || k <= GEMM_SHORT_K;
    Batch<GemmArgs> x(small ? kernels.small : kernels.large, GEMM_THREADS, s);
    for (Entry &e : entries) {
      if (small) tile(e, GEMM_SMALL);
      if (e.parts) *e.parts = e.g.tiles;
      if (const int rc = x.add(e.g, (int64_t)e.g.tiles * e.g.batch)) return rc;
    }
    entries.clear();
    return x.flush();
  }
};

template <int AO, int BO, typename TA, typename TB, int EPI, bool KS, bool ACC64 = false>
int launch_gemm(const GemmArgs &g, hipStream_t s) {
  Batch<GemmArgs> one(gemm_mfma_kernel<AO, BO, TA, TB, EPI, KS, ACC64>, GEMM_THREADS, s);
  if (const int rc = one.add(g, (int64_t)g.tiles * g.batch)) return rc;
  return one.flush();
}

int launch_fill(float *p, float v, int64_t n, hipStream_t s) {
  if (n <= 0) return SHAMPOO_OK;
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, v, n);
  HIP_TRY(hipGetLastError());
  return SHAMPOO_OK;
}

constexpr int JAC_STREAMS = 4;   // sub-chunks of the block solver that run concurrently

// Helper streams (default priority) and fork / join events of root refreshes and of steps of small and larger blocks.
struct AuxStreams {
  hipStream_t stream[JAC_STREAMS - 1] = {};
  hipEvent_t fork = nullptr, join[JAC_STREAMS - 1] = {};
  int state = 0;   // 0 = not tried, 1 = ready, -1 = unavailable (everything then runs on the caller's stream)
  bool ready() {
    if (state == 0) {
      state = 1;
      if (hipEventCreateWithFlags(&fork, hipEventDisableTiming) != hipSuccess) { fork = nullptr; state = -1; }
      for (int i = 0; i < JAC_STREAMS - 1 && state == 1; ++i) {
        if (hipStreamCreateWithFlags(&stream[i], hipStreamNonBlocking) != hipSuccess) { stream[i] = nullptr; state = -1; }
        else if (hipEventCreateWithFlags(&join[i], hipEventDisableTiming) != hipSuccess) { join[i] = nullptr; state = -1; }
      }
      if (state == -1) { release(); (void)hipGetLastError(); }
    }
    return state == 1;
  }
  // Waits for the helper streams' work, then frees streams and events.
  void release() {
    for (int i = 0; i < JAC_STREAMS - 1; ++i) {
      if (stream[i]) { (void)hipStreamSynchronize(stream[i]); (void)hipStreamDestroy(stream[i]); stream[i] = nullptr; }
      if (join[i]) { (void)hipEventDestroy(join[i]); join[i] = nullptr; }
    }
    if (fork) { (void)hipEventDestroy(fork); fork = nullptr; }
  }
};

// What the stand-alone entry points keep per GPU until the process ends.
constexpr int MAX_DEVICES = 64;
struct PerDevice {
  std::mutex mutex;
  AuxStreams aux;                      // helper streams of shampoo_root_inverse
  unsigned char *scratch = nullptr;    // device address of `scratch` on this GPU
};
PerDevice per_device[MAX_DEVICES];

// Block-Jacobi root inverse of `cnt` matrices, using workspace slots [slot0, slot0 + cnt).
// Warm start (WarmStart::qt != nullptr): the rows of Qt are kept between solves in the caller's
// array; with `start` set the solve begins at W = Qt A Qt^T instead of W = A, Qt = I.
struct WarmStart {
  float *qt = nullptr;          // [batch][np][np]: eigenvectors, read (start) and written
  bool start = false;
  int32_t *sweeps = nullptr;    // optional [batch]: sweeps in which anything rotated
  bool young = false;           // the factors have seen few gradient columns (young_factor): badly conditioned, they
                                // take three more sweeps than well-conditioned ones, and a cold solve then runs two
                                // more of them in float32, where a sweep costs half of what it does in float64
                                // (256 factors of a single gradient, n = 1024: 345 -> 322 ms; well-conditioned
                                // factors would pay for the two sweeps and gain nothing: 268 -> 293 ms)
};

// One sub-chunk of a block-Jacobi solve: `cnt` matrices in workspace slots [slot0, slot0 + cnt),
// all of its work on one stream.  The solve is enqueued phase by phase (begin, then sweep after
// sweep, then finish) so that the caller can interleave the sub-chunks of a chunk: the host
// needs a few microseconds per launch and a solve is thousands of launches, so a sub-chunk
// that were enqueued whole before the next one would run alone for most of its time.
struct BlockSolve {
  const float *a; int n, cnt; float eps, r, scale; float *x, *lambda; int32_t *failed_user;
  unsigned long long *fail_count; unsigned char *ws; const EigLayout *e; int slot0; hipStream_t s;
  const int32_t *only; WarmStart warm_in;
  // derived
  int np = 0, nblk = 0, hp = 0, sw = 0;
  bool warm = false;
  double *w = nullptr; float *w32 = nullptr, *qt = nullptr, *fv = nullptr, *d32 = nullptr;
  int32_t *rot = nullptr, *failed = nullptr, *done = nullptr, *skipc = nullptr;
  float *jslot[2] = {nullptr, nullptr}; int32_t *islot[2] = {nullptr, nullptr}; uint16_t *hslot[2] = {nullptr, nullptr};
  BlockJacArgs ja{};

  int begin() {
    np = e->np; nblk = np / JAC_NB; hp = nblk / 2;
    w = reinterpret_cast<double *>(ws + e->off_w) + (int64_t)slot0 * np * np;
    qt = warm_in.qt ? warm_in.qt : reinterpret_cast<float *>(ws + e->off_qt) + (int64_t)slot0 * np * np;
    warm = warm_in.qt && warm_in.start && e->warm;
    for (int k = 0; k < 2; ++k) {
      jslot[k] = reinterpret_cast<float *>(ws + e->off_j) + ((int64_t)k * e->chunk + slot0) * hp * JAC_PIV * JAC_PIV;
      islot[k] = reinterpret_cast<int32_t *>(ws + e->off_ident) + ((int64_t)k * e->chunk + slot0) * hp;
      hslot[k] = reinterpret_cast<uint16_t *>(ws + e->off_j16) + ((int64_t)k * e->chunk + slot0) * hp * 2 * JAC_PIV * JAC_PIV;
    }
    rot = reinterpret_cast<int32_t *>(ws + e->off_rot) + (int64_t)slot0 * JAC_OUTER_SWEEPS;
    float *dmax = reinterpret_cast<float *>(ws + e->off_dmax) + slot0;
    failed = reinterpret_cast<int32_t *>(ws + e->off_failed) + slot0;
    done = failed + e->chunk; skipc = failed + 2 * e->chunk;
    fv = reinterpret_cast<float *>(ws + e->off_f) + (int64_t)slot0 * np;
    d32 = reinterpret_cast<float *>(ws + e->off_f) + ((int64_t)e->chunk + slot0) * np;
    float *wbound = reinterpret_cast<float *>(ws + e->off_dmax) + e->chunk + slot0;
    int rc = launch_fill(dmax, 0.f, cnt, s);
    if (rc) return rc;
    rc = launch_fill(wbound, 0.f, cnt, s);
    if (rc) return rc;
    rc = launch_fill(reinterpret_cast<float *>(failed), 0.f, cnt, s);
    if (rc) return rc;
    rc = launch_fill(reinterpret_cast<float *>(done), 0.f, cnt, s);
    if (rc) return rc;
    BlockInitArgs ia;
    ia.a = a; ia.a_stride = (int64_t)n * n; ia.n = n;
    ia.qt = qt; ia.np = np; ia.dmax = dmax; ia.wbound = wbound; ia.failed = failed; ia.rot = rot; ia.only = only;
    // A solve runs its first sweeps on a float32 copy of W (twice the matrix-core and vector
    // rates, half the bytes): W = A, Qt = I for a cold solve, W = Qt A Qt^T rounded to float32
    // for a warm one.  Then W = Qt A Qt^T is formed in float64 from the rotations accumulated so
    // far, and float64 sweeps finish the job.  What the float32 sweeps cannot resolve
    // (eigenvalues below 1e-7 of the largest) is left to them.
    w32 = reinterpret_cast<float *>(w);      // shares the memory of W: it is dead when W is formed
    ia.warm = warm ? 1 : 0;
    ia.w = w32;
    hipLaunchKernelGGL(blockjac_init_kernel, dim3(nblk, cnt), dim3(256), 0, s, ia);
    HIP_TRY(hipGetLastError());
    if (warm) congruence(failed, true);
    ja.w = w; ja.w32 = w32; ja.qt = qt; ja.jbuf = jslot[0]; ja.ident = islot[0]; ja.rot = rot; ja.dmax = dmax; ja.wbound = wbound; ja.failed = failed; ja.done = done;
    ja.ident2 = islot[1]; ja.jt16 = hslot[0]; ja.jt16_2 = hslot[1];
    ja.np = np;
    ja.group = (nblk % 4 == 0) ? 2 : 1;
    ja.inner_sweeps = JAC_INNER_SWEEPS;
    sw = 0;
    return SHAMPOO_OK;
  }
  int f32_sweeps() const {
    if (warm) return JAC_F32_SWEEPS_WARM;
    return warm_in.young ? JAC_F32_SWEEPS_YOUNG : JAC_F32_SWEEPS;
  }
  // The next sweep: float32 while sw < f32_sweeps(), then (once) the congruence, then float64.
  int sweep() {
    const int appw_seg = appw_segments(hp);
    const int q_blocks = hp * ((np / JAC_PIV + APPQ_TILES - 1) / APPQ_TILES);
    const bool f32 = sw < f32_sweeps();
    if (f32) {
      ja.phase_start = 0; ja.tol_rel = JAC_F32_TOL_REL; ja.tol_abs_rel = JAC_F32_TOL_ABS;
    } else {
      if (sw == f32_sweeps()) {
        // matrices that float32 has served well enough leave here
        BlockVerdictArgs va{d32, w32, np, n, failed, done, skipc};
        hipLaunchKernelGGL(blockjac_f32_verdict_kernel, dim3(cnt), dim3(256), 0, s, va);
        congruence(skipc, false);
      }
      ja.phase_start = f32_sweeps(); ja.tol_rel = JAC_BLOCK_TOL_REL; ja.tol_abs_rel = JAC_SMALL_TOL_ABS;
    }
    for (int rd = 0; rd < nblk - 1; ++rd) {
      // group == 2: rounds 1 + 2 R and 2 + 2 R are the two rounds of one meeting of super-columns;
      // the second keeps its rotation blocks apart, and Q^T takes both after it
      const int sub = (ja.group == 2 && rd > 0) ? (rd - 1) & 1 : 0;
      ja.round = rd; ja.sweep = sw;
      ja.jbuf = jslot[sub]; ja.ident = islot[sub]; ja.jt16 = hslot[sub];
      // group == 2: the pairs inside a block column are rotated by the pivots of round 0 only (once
      // per sweep, like every other pair); the pivots of the other rounds keep to the pairs across
      // their two block columns, which halves their rounds
      ja.cross_only = (ja.group == 2 && rd > 0) ? 1 : 0;
      if (f32) {
        if (ja.cross_only) hipLaunchKernelGGL((blockjac_pivot_kernel<float, true>), dim3(hp, cnt), dim3(JAC_PIV_THREADS), 0, s, ja);
        else hipLaunchKernelGGL((blockjac_pivot_kernel<float, false>), dim3(hp, cnt), dim3(JAC_PIV_THREADS), 0, s, ja);
        hipLaunchKernelGGL(blockjac_apply_w32_kernel, dim3(appw_segments(hp, W16_SEG), cnt), dim3(JAC_THREADS), 0, s, ja);
      } else {
        if (ja.cross_only) hipLaunchKernelGGL((blockjac_pivot_kernel<double, true>), dim3(hp, cnt), dim3(JAC_PIV_THREADS), 0, s, ja);
        else hipLaunchKernelGGL((blockjac_pivot_kernel<double, false>), dim3(hp, cnt), dim3(JAC_PIV_THREADS), 0, s, ja);
        hipLaunchKernelGGL(blockjac_apply_w_kernel, dim3(appw_seg, cnt), dim3(JAC_THREADS), 0, s, ja);
      }
      if (ja.group == 1 || rd == 0) {
        hipLaunchKernelGGL(blockjac_apply_q_kernel, dim3(q_blocks, cnt), dim3(JAC_THREADS), 0, s, ja);
      } else if (sub == 1) {
        ja.round = rd - 1; ja.jbuf = jslot[0]; ja.ident = islot[0]; ja.jt16 = hslot[0];
        hipLaunchKernelGGL(blockjac_apply_q2_kernel, dim3(q_blocks / 2, cnt), dim3(APPQ2_THREADS), 0, s, ja);
      }
    }
    HIP_TRY(hipGetLastError());
    ++sw;
    return SHAMPOO_OK;
  }
  void congruence(const int32_t *skip, bool out32) {
    // W = Qt A Qt^T, a panel of columns at a time: T = A Qt^T[:, panel], W[:, panel] = Qt T
    // (out32: rounded to float32, into the float32 copy of W)
    const int pw_max = std::min(np, CONGRUENCE_PANEL);
    double *tp = reinterpret_cast<double *>(ws + e->off_t) + (int64_t)slot0 * np * pw_max;
    for (int col0 = 0; col0 < np; col0 += pw_max) {
      const int pw = std::min(pw_max, np - col0);
      CongruenceArgs c1{};
      c1.a = a; c1.a_batch = (int64_t)n * n; c1.lda = n;
      c1.b = qt + (int64_t)col0 * np; c1.b_batch = (int64_t)np * np; c1.ldb = np;
      c1.c = tp; c1.c_batch = (int64_t)np * pw_max; c1.ldc = pw_max;
      c1.M = n; c1.N = pw; c1.K = n; c1.col0 = 0; c1.skip = skip;
      hipLaunchKernelGGL((congruence_gemm_kernel<false, false>), dim3((pw + CG_TILE - 1) / CG_TILE, (n + CG_TILE - 1) / CG_TILE, cnt),
                         dim3(CG_THREADS), 0, s, c1);
      CongruenceArgs c2{};
      c2.a = qt; c2.a_batch = (int64_t)np * np; c2.lda = np;
      c2.b = tp; c2.b_batch = (int64_t)np * pw_max; c2.ldb = pw_max;
      c2.c = w; c2.c_batch = (int64_t)np * np; c2.ldc = np;
      c2.M = np; c2.N = pw; c2.K = n; c2.col0 = col0; c2.skip = skip;
      const dim3 grid2((pw + CG_TILE - 1) / CG_TILE, (np + CG_TILE - 1) / CG_TILE, cnt);
      if (out32) hipLaunchKernelGGL((congruence_gemm_kernel<true, true, true>), grid2, dim3(CG_THREADS), 0, s, c2);
      else hipLaunchKernelGGL((congruence_gemm_kernel<true, true, false>), grid2, dim3(CG_THREADS), 0, s, c2);
    }
  }
  int finish() {
    BlockFinalArgs fa;
    fa.w = w; fa.qt = qt; fa.np = np; fa.n = n; fa.epsilon = eps; fa.r = r; fa.scale = scale; fa.fvals = fv;
    fa.lambda = lambda;
    fa.failed = failed; fa.failed_out = failed_user; fa.fail_count = fail_count;
    fa.rot = rot; fa.sweeps_out = warm_in.sweeps; fa.done = done; fa.d32 = d32;
    BlockRowNormArgs rn{qt, fv, failed, np, n};
    hipLaunchKernelGGL(blockjac_rownorm_kernel, dim3((n + 3) / 4, cnt), dim3(256), 0, s, rn);
    hipLaunchKernelGGL(blockjac_final_kernel, dim3(cnt), dim3(256), 0, s, fa);
    HIP_TRY(hipGetLastError());
    GemmArgs g{};
    g.a.base = qt; g.a.batch_stride = (int64_t)np * np; g.a.ld = np; g.a.from_table = 0;
    g.b = g.a;
    g.c = x; g.c_batch_stride = (int64_t)n * n; g.ldc = n;
    g.M = n; g.N = n; g.K = np; g.alpha = 1.f; g.beta = 0.f;
    g.kscale = fv; g.kscale_stride = np; g.skip = failed;
    g.tiles_m = g.tiles_n = (n + BM - 1) / BM;
    g.tiles = g.tiles_m * (g.tiles_m + 1) / 2;
    g.batch = cnt;
    return launch_gemm<ROW_CONTIG, ROW_CONTIG, float, float, EPI_SYRK, true>(g, s);
  }
};

// Band reductions on one stream: matrices of one size or of several, each launch for all of them (the panels, groups and
// rounds that a size does not have are left out).  Enqueued panel by panel, so
// that the caller can interleave two of them: while one is in a QR
// factorisation, which uses one CU per matrix, the other's products fill the chip.
struct BandSolve {
  std::vector<BandJob> jobs;
  hipStream_t s;
  const RatTable *table;
  using Kernel = void (*)(const BandJobs);
  // wgs: workgroups of a job, 0 where it takes no part; may set its k
  template <typename F> int each(Kernel kernel, int threads, F wgs) {
    Batch<BandJob> x(kernel, threads, s);
    for (BandJob &j : jobs)
      if (const int64_t n = wgs(j))
        if (const int rc = x.add(j, n)) return rc;
    return x.flush();
  }
  int most(int (*f)(const BandArgs &)) const { int m = 0; for (const BandJob &j : jobs) m = std::max(m, f(j.g)); return m; }
  int panels() const { return most([](const BandArgs &g) { return (int)g.nb; }); }
  int groups() const { return most([](const BandArgs &g) { return band_groups(g); }); }
  int begin() {
    int rc;
    if ((rc = each(band_clear_kernel, 256, [](BandJob &j) { return (j.cnt + 255) / 256; }))) return rc;
    if ((rc = each(band_init_kernel, 256, [](BandJob &j) { return (int64_t)j.g.nb * j.cnt; }))) return rc;
    return each(band_alone_kernel, 256, [](BandJob &j) { return j.cnt; });
  }
  int forward(int p) {
    int rc, m = 0;
    for (BandJob &j : jobs) { j.k = p; if (p < j.g.nb) m = std::max(m, band_left(j.g, p)); }
    const Kernel qr = m <= 256 ? band_qr_kernel<8> : m <= 512 ? band_qr_kernel<16> : m <= 1024 ? band_qr_kernel<32> : band_qr_kernel<64>;
    if ((rc = each(qr, BAND_QR_THREADS, [&](BandJob &j) { return p < j.g.nb ? j.cnt : 0; }))) return rc;
    auto rows = [&](BandJob &j) { return p + 1 < j.g.nb ? (int64_t)band_row_wgs(j.g, p) * j.cnt : 0; };
    if ((rc = each(band_z_kernel, 512, [&](BandJob &j) { return p + 1 < j.g.nb ? (int64_t)band_z_wgs(j.g, p) * j.cnt : 0; }))) return rc;
    if ((rc = each(band_y_kernel, 256, rows))) return rc;
    return each(band_update_kernel, 256, [&](BandJob &j) { return rows(j) * (p + 1 < j.g.nb ? band_col_wgs(j.g, p) : 0); });
  }
  int function() {
    int rc;
    auto one = [](BandJob &j) { return j.cnt; };
    auto per_block = [](BandJob &j) { return (int64_t)j.g.nb * j.cnt; };
    if ((rc = each(band_bounds_kernel, 256, one))) return rc;
    for (int round = 0; round < BAND_ROUNDS; ++round)
      if ((rc = each(band_probe_kernel, 64, [&](BandJob &j) { j.k = round; return (int64_t)BAND_SHIFTS * j.cnt; }))) return rc;
    if ((rc = each(band_plan_kernel, 64, [](BandJob &j) { return (j.cnt + 63) / 64; }))) return rc;
    Batch<BandJob, BAND_TABLE_RESERVE, const RatTable> factor(band_factor_kernel, 64, s);
    for (const BandJob &j : jobs) if ((rc = factor.add(j, (int64_t)BAND_SLOTS * j.cnt))) return rc;
    if ((rc = factor.flush(*table))) return rc;
    for (const Kernel rows : {band_rows_kernel<2>, band_rows_kernel<3>, band_rows_kernel<4>, band_rows_kernel<5>})
      if ((rc = each(rows, 512, per_block))) return rc;
    if ((rc = each(band_fv_kernel, 256, per_block)) || (rc = each(band_deflate_kernel, 256, per_block))) return rc;
    return each(band_group_t_kernel, 1024, [](BandJob &j) { return (int64_t)band_groups(j.g) * j.cnt; });
  }
  // the u-th group of panels from the end
  int back(int u) {
    // The sums are what these products lose accuracy by: those of 32 values of k go into float64.  Error of
    // the root of a factor of one gradient at n = 160, 256, 1024: 1.4e-6, 1.4e-6, 1.9e-6 with float32 sums but in Z, 4.8e-7,
    // 4.8e-7, 6.2e-7 so; block Jacobi 8.8e-7, 1.0e-6, 3.0e-6.  The update of F moves the root by a tenth of that:
    // float64 where the margin to Jacobi is small.
    int rc;
    auto takes_part = [&](BandJob &j) { j.k = band_groups(j.g) - 1 - u; return j.k >= 0; };
    GemmBatch<EPI_STORE> zs(gemm_kernels<K_CONTIG, ROW_CONTIG, float, float, EPI_STORE, true>(), s);
    Batch<GemmArgs> ys(gemm_mfma_kernel<K_CONTIG, ROW_CONTIG, float, float, EPI_STORE, false, true>, GEMM_THREADS, s);
    GemmBatch<EPI_SYRK> us64(gemm_kernels<K_CONTIG, K_CONTIG, float, float, EPI_SYRK, true>(), s), us(gemm_kernels<K_CONTIG, K_CONTIG, float, float, EPI_SYRK>(), s);
    for (BandJob &j : jobs) {
      if (!takes_part(j)) continue;
      const BandArgs &g = j.g;
      const int np = g.np, r0 = (BAND_GROUP * j.k + 1) * BAND, tiles = (np + BM - 1) / BM;
      float *p = band_p(g);
      const int64_t pstride = band_p_stride(g);
      GemmArgs z{};                        // Z = F V
      z.a.base = g.f + r0; z.a.batch_stride = (int64_t)np * np * 2; z.a.ld = np;
      z.b.base = p + (int64_t)r0 * BAND_PLD + BAND_GW; z.b.batch_stride = pstride; z.b.ld = BAND_PLD;
      z.c = p; z.c_batch_stride = pstride; z.ldc = BAND_PLD;
      z.M = np; z.N = BAND_GW; z.K = np - r0; z.alpha_d = 1.0; z.skip = g.skip;
      z.tiles_m = z.tiles = tiles; z.tiles_n = 1; z.batch = j.cnt;
      zs.add(z);
      // Y = [Z V] [T^T; -T M T^T / 2], over Z: a workgroup stores only rows that no other reads, after it has read them (tiles as
      // wide as Z)
      GemmArgs y = z;
      y.a = Operand{p, pstride, BAND_PLD, 0};
      y.b = Operand{band_ts(g), pstride, BAND_GW, 0};
      y.K = 2 * BAND_GW;
      if ((rc = ys.add(y, (int64_t)y.tiles * y.batch))) return rc;
      GemmArgs f = z;                      // F <- F - [Y V] [V Y]^T; V has no rows in front of r0
      f.a = y.a;
      f.b = Operand{p + BAND_GW, pstride, BAND_PLD, 0};
      f.c = g.f; f.c_batch_stride = (int64_t)np * np * 2; f.ldc = np;
      f.N = np; f.K = 2 * BAND_GW; f.alpha = -1.f; f.beta = 1.f; f.alpha_d = -1.0; f.beta_d = 1.0;
      (np <= 512 ? us64 : us).add(f, nullptr, r0);
    }
    auto stage = [&](BandJob &j) { return takes_part(j) ? (int64_t)(j.g.np / 8) * j.cnt : 0; };
    if ((rc = each(band_stage_kernel<false>, 256, stage)) || (rc = zs.flush())) return rc;
    auto four = [&](BandJob &j) { return takes_part(j) ? (int64_t)4 * j.cnt : 0; };
    if ((rc = each(band_m_kernel, 1024, four)) || (rc = each(band_s_kernel, 256, four)) || (rc = ys.flush())) return rc;
    if ((rc = each(band_stage_kernel<true>, 256, stage)) || (rc = us64.flush())) return rc;
    return us.flush();
  }
  int finish() {
    return each(band_out_kernel, 256, [](BandJob &j) { return (int64_t)(j.g.nb * (j.g.nb + 1) / 2) * j.cnt; });
  }
};

// Parts on streams of their own: while one is in the chain of a panel's columns or of the pivots, the
// others have products to do.  On two and on three streams: 64 matrices of 1024 12.8 and 12.4 ms, refresh of two layers of 1300
// 20.7 and 20.2, of two transformer layers (192 matrices of 1024) 30.7 and 30.0; 16 of 2048 26.9 and 27.1, 8 of 172 0.80 and 0.87.
constexpr int BAND_STREAMS = 3;
constexpr int64_t BAND_MANY = 32;        // matrices from which on there are three
static_assert(BAND_STREAMS < JAC_STREAMS, "helper streams, and one more");

// Helper streams forked off s, and joined to it again on every way out, also where a call fails or host memory runs out: whatever a
// call returns, s waits for all that the call has enqueued.
struct Fork {
  AuxStreams *aux = nullptr; int first = 0, last = 0; hipStream_t s = nullptr;      // streams first ... last - 1 are forked
  Fork() = default;
  Fork(const Fork &) = delete;
  Fork &operator=(const Fork &) = delete;
  int begin(AuxStreams *a, int from, int to, hipStream_t stream) {
    aux = a; first = last = from; s = stream;
    if (from >= to) return SHAMPOO_OK;
    HIP_TRY(hipEventRecord(aux->fork, s));
    for (; last < to; ++last) HIP_TRY(hipStreamWaitEvent(aux->stream[last], aux->fork, 0));
    return SHAMPOO_OK;
  }
  int join() {
    int rc = SHAMPOO_OK;
    for (; first < last; ++first)
      if (hipEventRecord(aux->join[first], aux->stream[first]) != hipSuccess || hipStreamWaitEvent(s, aux->join[first], 0) != hipSuccess) rc = SHAMPOO_ERR_HIP;
    return rc;
  }
  ~Fork() { (void)join(); }
};

// Roots of a batch of dense n x n matrices that the band reduction or the tridiagonal one serves.
struct RootJob {
  const float *a; int n, batch; float r, scale; float *x; int32_t *failed_user; const int32_t *only;
};

// Jobs of one exponent, of any sizes: as many of their matrices at a time as fit into `room` bytes of ws, those
// in equal parts on two or three streams.  The launches of few matrices leave most of the GPU idle, and every panel of every size is a
// launch: the two sides of a dozen buckets take one pass here, not one each.  Refresh of three layers of 700 in blocks of 512:
// 31 ms one size at a time, 5.4 so; two layers of 1300 in blocks of 1024: 100 and 24; one layer of 896 in blocks of 256, where
// nothing is ragged: 1.9 and 1.5.
int band_roots(const std::vector<RootJob> &todo, float eps, unsigned long long *fail_count, unsigned char *ws, size_t room, hipStream_t s,
               AuxStreams *aux, const RatTable &table) {
  int rc;
  size_t i = 0;
  int done = 0;                            // matrices of todo[i]
  int64_t left_over = 0;
  for (const RootJob &j : todo) left_over += j.batch;
  while (i < todo.size()) {
    BandSolve solve[BAND_STREAMS];
    size_t at = 0;
    int turn = 0;
    const int subs = !aux ? 1 : left_over >= BAND_MANY ? BAND_STREAMS : 2;
    // passes of equal size: a small one at the end takes as long as a large one (192 matrices of 1024 in 180 and 12: 36 ms, in 96 and 96 33)
    size_t bytes_left = 0;
    for (size_t k = i; k < todo.size(); ++k) bytes_left += band_layout_of(todo[k].n, todo[k].batch - (k == i ? done : 0)).bytes;
    const size_t fair = bytes_left / ((bytes_left + room - 1) / room);
    while (i < todo.size()) {
      const RootJob &j = todo[i];
      const int left = std::min(j.batch - done, 32768);
      int cnt = (int)std::min<size_t>(left, (room - at) / band_layout_of(j.n, 1).bytes);
      while (cnt < left && at + band_layout_of(j.n, cnt + 1).bytes <= room) ++cnt;   // the arrays of a single matrix are padded
      if (bytes_left > room) cnt = std::min<int64_t>(cnt, at < fair ? (int64_t)((fair - at) / band_layout_of(j.n, 1).bytes) + 1 : 0);
      if (cnt == 0) break;
      const BandLayout e = band_layout_of(j.n, cnt);
      BandArgs base{};
      unsigned char *w = ws + at;
      base.a = j.a + (int64_t)done * j.n * j.n; base.n = j.n; base.np = e.np; base.nb = e.nb;
      base.eps = eps; base.r = j.r; base.scale = j.scale; base.x = j.x + (int64_t)done * j.n * j.n; base.fail_count = fail_count;
      base.meta = reinterpret_cast<BandMeta *>(w + e.off_meta);
      base.w = reinterpret_cast<double *>(w + e.off_w); base.f = reinterpret_cast<float *>(w + e.off_w);
      base.vp = reinterpret_cast<double *>(w + e.off_vp); base.t = reinterpret_cast<double *>(w + e.off_t);
      base.z = reinterpret_cast<double *>(w + e.off_z); base.y = reinterpret_cast<double *>(w + e.off_y);
      base.part = reinterpret_cast<double *>(w + e.off_part); base.skip = reinterpret_cast<int32_t *>(w + e.off_skip);
      base.vall = reinterpret_cast<float *>(w + e.off_vall); base.tall = reinterpret_cast<float *>(w + e.off_tall);
      base.dblk = reinterpret_cast<double *>(w + e.off_dblk); base.cblk = reinterpret_cast<double *>(w + e.off_cblk);
      base.kf = reinterpret_cast<double *>(w + e.off_kf); base.gf = reinterpret_cast<double *>(w + e.off_gf);
      base.v1 = reinterpret_cast<double *>(w + e.off_v1);
      base.ok = reinterpret_cast<int32_t *>(w + e.off_ok); base.dec = reinterpret_cast<int32_t *>(w + e.off_dec);
      // in equal parts; odd ones out go to the streams in turn
      int first = 0;
      for (int k = 0; k < subs; ++k) {
        const int part = cnt / subs + ((k + turn) % subs < cnt % subs ? 1 : 0);
        if (part == 0) continue;
        BandJob job{base, 0, part};
        band_select(job.g, first);
        job.g.failed_user = j.failed_user ? j.failed_user + done + first : nullptr;
        job.g.only = j.only ? j.only + done + first : nullptr;
        solve[k].jobs.push_back(job);
        first += part;
      }
      turn += subs - cnt % subs;
      left_over -= cnt;
      at += e.bytes;
      done += cnt;
      if (done < j.batch) break;           // no room for the rest
      ++i; done = 0;
    }
    if (at == 0) return SHAMPOO_ERR_WORKSPACE;
    int n_solve = 0;                       // the parts that have matrices, in front
    for (int k = 0; k < subs; ++k)
      if (!solve[k].jobs.empty()) {
        if (k != n_solve) solve[n_solve].jobs.swap(solve[k].jobs);
        solve[n_solve].table = &table;
        solve[n_solve].s = n_solve == 0 ? s : aux->stream[n_solve - 1];
        ++n_solve;
      }
    BandSolve *v = solve;
    Fork fork;
    if ((rc = fork.begin(aux, 0, n_solve - 1, s))) return rc;
    int panels = 0, groups = 0;
    for (int k = 0; k < n_solve; ++k) { panels = std::max(panels, v[k].panels()); groups = std::max(groups, v[k].groups()); }
    for (int k = 0; k < n_solve; ++k) if ((rc = v[k].begin())) return rc;
    for (int q = 0; q < panels; ++q)
      for (int k = 0; k < n_solve; ++k) if (q < v[k].panels() && (rc = v[k].forward(q))) return rc;
    for (int k = 0; k < n_solve; ++k) if ((rc = v[k].function())) return rc;
    for (int u = 0; u < groups; ++u)
      for (int k = 0; k < n_solve; ++k) if (u < v[k].groups() && (rc = v[k].back(u))) return rc;
    for (int k = 0; k < n_solve; ++k) if ((rc = v[k].finish())) return rc;
    if ((rc = fork.join())) return rc;
  }
  return SHAMPOO_OK;
}

// Roots of up to 128 x 128: one launch for all jobs of a kernel (of one exponent), the largest matrices first.
int tridiag_roots(std::vector<RootJob> todo, float eps, unsigned long long *fail_count, hipStream_t s, const RatTable &table) {
  std::stable_sort(todo.begin(), todo.end(), [](const RootJob &x, const RootJob &y) { return x.n > y.n; });
  using Roots = Batch<SmallRootArgs, TRI_TABLE_RESERVE, const RatTable>;
  Roots large(rootinv_tridiag_kernel<128, 256>, 256, s), middle(rootinv_tridiag_kernel<64, 128>, 128, s), small(rootinv_tridiag_kernel<32, 64>, 64, s);
  for (const RootJob &j : todo) {
    SmallRootArgs g{};
    g.a = j.a; g.a_stride = (int64_t)j.n * j.n; g.x = j.x; g.x_stride = (int64_t)j.n * j.n;
    g.failed = j.failed_user; g.fail_count = fail_count; g.n = j.n; g.epsilon = eps; g.r = j.r; g.scale = j.scale; g.only = j.only;
    g.batch = j.batch;
    if (const int rc = (j.n > 64 ? large : j.n > 32 ? middle : small).add(g, j.batch)) return rc;
  }
  for (Roots *x : {&large, &middle, &small})
    if (const int rc = x->flush(table)) return rc;
  return SHAMPOO_OK;
}

// X_i = rootinv(scale * A_i) for a batch of dense n x n matrices.  ws: eig_layout(n, >= chunk) region.
// aux: helper streams for the sub-chunks of the block solver (the caller owns them and
// serialises their use), or nullptr.
// only: optional device array [batch]; matrices whose entry is 0 are skipped (x left as it is).
int root_inverse_batched(const float *a, int n, int batch, float eps, float r, float scale, float *x, float *lambda,
                         int32_t *failed_user, unsigned long long *fail_count, unsigned char *ws,
                         const EigLayout &e, hipStream_t s, AuxStreams *aux, const int32_t *only = nullptr,
                         const WarmStart &warm = WarmStart()) {
  if (batch <= 0) return SHAMPOO_OK;
  if (n <= JAC_SMALL_MAX) {
    SmallRootArgs g{};
    g.a = a; g.a_stride = (int64_t)n * n;
    g.x = x; g.x_stride = (int64_t)n * n;
    g.lambda = lambda; g.failed = failed_user; g.fail_count = fail_count;
    g.n = n; g.epsilon = eps; g.r = r; g.scale = scale; g.only = only;
    // without eigenvectors where nobody asks for eigenvalues and the exponent has a rational fit
    RatTable table;
    if (!lambda && rat_table(r, table)) return tridiag_roots({RootJob{a, n, batch, r, scale, x, failed_user, only}}, eps, fail_count, s, table);
    const size_t lds = rootinv_small_lds_bytes(n);
    if (n <= 64) {
      HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(rootinv_small_kernel<256>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
      hipLaunchKernelGGL(rootinv_small_kernel<256>, dim3(batch), dim3(256), lds, s, g);
    } else {
      HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(rootinv_small_kernel<1024>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
      hipLaunchKernelGGL(rootinv_small_kernel<1024>, dim3(batch), dim3(1024), lds, s, g);
    }
    HIP_TRY(hipGetLastError());
    return SHAMPOO_OK;
  }
  // Large matrices: block Jacobi.  A chunk of matrices is cut into a few sub-chunks
  // that run on separate streams: the pivot kernel is bound by LDS, the W update by
  // the float64 matrix cores and the Q update by HBM, so sub-chunks that are in
  // different phases overlap on the same CUs.
  // aux == nullptr: everything on the caller's stream.
  if (aux && !aux->ready()) aux = nullptr;
  RatTable table;
  if (!lambda && !warm.qt && e.band.bytes && band_serves(n, r) && rat_table(r, table))
    return band_roots({RootJob{a, n, batch, r, scale, x, failed_user, only}}, eps, fail_count, ws, e.band.bytes, s, aux, table);
  const int n_sub = aux ? JAC_STREAMS : 1;
  for (int b0 = 0; b0 < batch; b0 += e.chunk) {
    const int cb = std::min(e.chunk, batch - b0);
    const int subs = std::min(n_sub, cb);
    Fork fork;
    if (const int rc = fork.begin(aux, 0, subs - 1, s)) return rc;
    BlockSolve solve[JAC_STREAMS];
    int first = 0;
    for (int k = 0; k < subs; ++k) {
      const int cnt = cb / subs + (k < cb % subs ? 1 : 0);
      WarmStart wk = warm;
      if (wk.qt) wk.qt += (int64_t)(b0 + first) * e.np * e.np;
      if (wk.sweeps) wk.sweeps += b0 + first;
      solve[k] = BlockSolve{a + (int64_t)(b0 + first) * n * n, n, cnt, eps, r, scale,
                            x + (int64_t)(b0 + first) * n * n,
                            lambda ? lambda + (int64_t)(b0 + first) * n : nullptr,
                            failed_user ? failed_user + b0 + first : nullptr, fail_count, ws, &e, first,
                            k == 0 ? s : aux->stream[k - 1], only ? only + b0 + first : nullptr, wk};
      first += cnt;
    }
    // sweep by sweep across the sub-chunks, so that all of them are under way from the start
    for (int k = 0; k < subs; ++k)
      if (const int rc = solve[k].begin()) return rc;
    for (int sw = 0; sw < JAC_OUTER_SWEEPS; ++sw)
      for (int k = 0; k < subs; ++k)
        if (const int rc = solve[k].sweep()) return rc;
    for (int k = 0; k < subs; ++k)
      if (const int rc = solve[k].finish()) return rc;
    if (const int rc = fork.join()) return rc;
  }
  return SHAMPOO_OK;
}

// ---------------------------------------------------------------------------
// Coupled inverse Newton iteration (Sec. 3.2.1, item 2): workspace and driver
// ---------------------------------------------------------------------------
struct NewtonLayout {
  int32_t chunk = 0;
  size_t mat = 0;          // bytes of one n x n float32 matrix (aligned)
  size_t off_mats = 0, off_rowpart = 0, off_err = 0, off_prev = 0, off_done = 0, off_failed = 0, off_iters = 0, off_arrived = 0, off_xdone = 0;
  size_t bytes = 0;
};
constexpr int NEWTON_MATS = 7;   // M, M', X, X', T and two buffers for the powers of T

NewtonLayout newton_layout(int n, int batch) {
  NewtonLayout e;
  if (n <= NEWTON_SMALL) { e.bytes = ALIGN; return e; }      // newton_small_kernel keeps everything in registers and LDS
  e.mat = align_up((size_t)n * n * sizeof(float));
  // the kernels take the matrix index as grid.y
  e.chunk = (int)std::max<size_t>(1, std::min<size_t>(std::min<size_t>((size_t)std::max(batch, 1), 32768), EIG_CHUNK_BYTES / (NEWTON_MATS * e.mat)));
  size_t off = 0;
  e.off_mats = off; off += (size_t)NEWTON_MATS * e.chunk * e.mat;
  e.off_rowpart = off; off += align_up((size_t)e.chunk * ((n + NEWTON_TILE - 1) / NEWTON_TILE) * sizeof(double));
  e.off_err = off; off += align_up((size_t)e.chunk * sizeof(float));
  e.off_prev = off; off += align_up((size_t)e.chunk * sizeof(float));
  e.off_done = off; off += align_up((size_t)e.chunk * sizeof(int32_t));
  e.off_failed = off; off += align_up((size_t)e.chunk * sizeof(int32_t));
  e.off_iters = off; off += align_up((size_t)e.chunk * sizeof(int32_t));
  e.off_arrived = off; off += align_up((size_t)e.chunk * sizeof(int32_t));
  e.off_xdone = off; off += align_up((size_t)e.chunk * sizeof(int32_t));
  e.bytes = off;
  return e;
}

// p must be 1, 2, 4 or 8: T^p is formed by repeated squaring
inline bool newton_p_supported(int p) { return p == 1 || p == 2 || p == 4 || p == 8; }

// C = A B on the lower tiles, mirrored (A, B symmetric and commuting), for the matrices not yet done; launched by flush.
void newton_product(GemmBatch<EPI_SYRK> &to, const float *A, const float *B, float *C, int n, int cnt, const int32_t *done) {
  GemmArgs g{};
  g.a.base = A; g.a.batch_stride = (int64_t)n * n; g.a.ld = n; g.a.from_table = 0;
  g.b.base = B; g.b.batch_stride = (int64_t)n * n; g.b.ld = n; g.b.from_table = 0;
  g.c = C; g.c_batch_stride = (int64_t)n * n; g.ldc = n;
  g.M = n; g.N = n; g.K = n; g.alpha = 1.f; g.beta = 0.f;
  g.skip = done;
  g.batch = cnt;
  to.add(g);
}

// X_i = (scale * A_i + eps I)^(-1/p) for a batch of dense n x n matrices.
int newton_root_batched(const float *a, int n, int batch, float eps, int p, float scale, float tol, int max_iter,
                        float *x, int32_t *iters_user, int32_t *failed_user, unsigned long long *fail_count,
                        unsigned char *ws, const NewtonLayout &e, hipStream_t s) {
  if (batch <= 0) return SHAMPOO_OK;
  if (n <= NEWTON_SMALL) {
    NewtonSmallArgs g{a, x, iters_user, failed_user, fail_count, n, p, max_iter, eps, scale, tol};
    launch_newton_small(g, batch, s);
    HIP_TRY(hipGetLastError());
    return SHAMPOO_OK;
  }
  const size_t mat_elems = e.mat / sizeof(float);
  for (int b0 = 0; b0 < batch; b0 += e.chunk) {
    const int cb = std::min(e.chunk, batch - b0);
    float *buf[NEWTON_MATS];
    for (int i = 0; i < NEWTON_MATS; ++i) buf[i] = reinterpret_cast<float *>(ws + e.off_mats) + (size_t)i * e.chunk * mat_elems;
    // matrices of a chunk are stored back to back with stride n * n inside each buffer
    float *M = buf[0], *M2 = buf[1], *X = buf[2], *X2 = buf[3], *T = buf[4], *Pa = buf[5], *Pb = buf[6];
    NewtonArgs g{};
    g.a = a + (int64_t)b0 * n * n; g.a_stride = (int64_t)n * n;
    g.rowpart = reinterpret_cast<double *>(ws + e.off_rowpart);
    g.err = reinterpret_cast<float *>(ws + e.off_err); g.prev = reinterpret_cast<float *>(ws + e.off_prev);
    g.done = reinterpret_cast<int32_t *>(ws + e.off_done); g.failed = reinterpret_cast<int32_t *>(ws + e.off_failed);
    g.iters = reinterpret_cast<int32_t *>(ws + e.off_iters); g.arrived = reinterpret_cast<int32_t *>(ws + e.off_arrived);
    g.xdone = reinterpret_cast<int32_t *>(ws + e.off_xdone);
    g.n = n; g.p = p; g.max_iter = max_iter; g.epsilon = eps; g.scale = scale; g.tol = tol;
    int rc = launch_fill(reinterpret_cast<float *>(g.failed), 0.f, cb, s);
    if (rc) return rc;
    g.M = M; g.X = X; g.T = T;
    NewtonFinishArgs fa{};
    fa.X[0] = X; fa.X[1] = X2;
    const dim3 blocks((n + NEWTON_TILE - 1) / NEWTON_TILE, cb), rows((n + NEWTON_ROWS - 1) / NEWTON_ROWS, cb);
    hipLaunchKernelGGL(newton_norm_kernel, blocks, dim3(256), 0, s, g);
    hipLaunchKernelGGL(newton_init_kernel, blocks, dim3(256), 0, s, g);
    HIP_TRY(hipGetLastError());
    for (int k = 0; k <= max_iter; ++k) {
      // the X / M buffers swap roles from one k to the next, and a matrix whose iteration has ended is not written by the products
      g.k = k; g.M = M; g.X = X; g.X1 = k == 0 ? X2 : nullptr; g.T = T;
      hipLaunchKernelGGL(newton_prep_kernel, rows, dim3(256), 0, s, g);
      HIP_TRY(hipGetLastError());
      if (k == max_iter) break;
      // T^p by repeated squaring, X' = X T, M' = T^p M.  X T goes along with the first of the others (X_1 comes from newton_prep_kernel): of a
      // few matrices a launch is what an iteration costs (one of 129 x 129: 1.65 ms, 100 iterations of four launches).
      GemmBatch<EPI_SYRK> products(gemm_kernels<K_CONTIG, K_CONTIG, float, float, EPI_SYRK>(), s);     // symmetric: read along k
      if (k > 0) newton_product(products, X, T, X2, n, cb, g.xdone);
      const float *Tp = T;
      float *sq[2] = {Pa, Pb};
      int w = 0;
      for (int q = 1; q < p; q *= 2) {
        newton_product(products, Tp, Tp, sq[w], n, cb, g.done);
        if ((rc = products.flush())) return rc;
        Tp = sq[w]; w ^= 1;
      }
      newton_product(products, Tp, M, M2, n, cb, g.done);
      if ((rc = products.flush())) return rc;
      std::swap(M, M2); std::swap(X, X2);
    }
    fa.x = x + (int64_t)b0 * n * n; fa.x_stride = (int64_t)n * n;
    fa.failed = g.failed; fa.failed_out = failed_user ? failed_user + b0 : nullptr;
    fa.fail_count = fail_count;
    fa.iters = g.iters; fa.iters_out = iters_user ? iters_user + b0 : nullptr; fa.n = n;
    hipLaunchKernelGGL(newton_finish_kernel, rows, dim3(256), 0, s, fa);
    HIP_TRY(hipGetLastError());
  }
  return SHAMPOO_OK;
}

}  // namespace

// ---------------------------------------------------------------------------
// The optimizer object
// ---------------------------------------------------------------------------
struct shampoo_opt {
  shampoo_config cfg;
  std::vector<int32_t> ndim;
  std::vector<int64_t> shape;   // [SHAMPOO_MAX_NDIM * n_params], as given
  Plan plan;
  unsigned char *ws = nullptr;
  size_t ws_bytes = 0;
  // workspace offsets
  size_t off_G1 = 0, off_Gf = 0, off_g1tab = 0, off_gftab = 0, off_prep = 0, off_small = 0;
  int64_t n_small = 0;     // blocks of at most 128 x 128 (single-workgroup step kernel)
  bool small_half = false; // all of them at most 64 x 64
  int64_t n_prep_rest = 0; // of plan.prep_chunks, the first ones: parameters with other blocks too
  bool use_l2 = false, use_b1 = false;
  size_t off_A = 0, off_M = 0, off_T = 0, off_wtab = 0, off_gtab = 0, off_diag = 0, off_count = 0, off_eig = 0;
  size_t eig_bytes = 0;
  std::vector<EigLayout> eig_L, eig_R, eig_mid[2];   // per bucket (eig_mid: the middle dimensions of tensor blocks)
  // tensor parameters: block-contiguous copies of the gradient and the parameter (byte offsets
  // into the workspace, 0 for other parameters), and a second scratch array the size of T
  std::vector<size_t> off_Gb, off_Wb;
  size_t off_T2 = 0;
  bool has_tensor = false;
  size_t off_nfail = 0;   // coupled Newton: per-matrix failure flags of one batch (int32)
  std::vector<void *> last_w, last_g;    // [n_params] the caller's pointers of the last step; null before the first
  AuxStreams aux;                        // helper streams, made by shampoo_create where steps or refreshes can use them
  bool overlap = false;                  // the stages of the larger blocks are worth a stream of their own for the small ones
  bool tables_stale = true;              // last_w and last_g may not be what the device's tables hold
  bool tables_recorded = false;          // a graph holds a launch that writes them
  bool ptrs_aligned16 = false;           // every gradient pointer is 16-byte aligned
  // per bucket: a factor update has left out the tiles above the diagonal of tiles, a step in one workgroup per block all above the
  // diagonal.  Either may do so again in the replay of a graph, of which the host learns nothing: never reset
  std::vector<char> upper_stale, half_stale;
  int64_t last_step = -1;
  int64_t n_refresh = 0;
  bool timing = false;
  struct Interval { hipEvent_t a, b; };
  std::vector<Interval> intervals[SHAMPOO_STAGE_COUNT];
};

namespace {

// Planes of float32 gradients live only as long as the products that read them: those of 170 blocks of 1024 x 1024
// at a time (both ways round, or the transpose and T, 12 bytes per element), which is 24 tiles per CU of a factor update.
constexpr size_t PLANE_BYTES = (size_t)2 << 30;
// Scratch of the buckets that are worked on together: as much as the planes of one of them may take, so that the workspace
// of a set of any size grows by no more than this.
constexpr size_t SET_BYTES = (size_t)2 << 30;

size_t layout(const shampoo_config *c, Plan &p, shampoo_opt *o) {
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t r = off; off += align_up(bytes); return r; };
  const size_t offA = take((size_t)p.total_elems * 4);
  const size_t offM = c->momentum > 0.f ? take((size_t)p.total_elems * 4) : 0;
  const bool use_l2 = c->weight_decay > 0.f && !c->use_decoupled_weight_decay;
  const bool use_b1 = c->beta1 > 0.f;
  const size_t offG1 = use_l2 ? take((size_t)p.total_elems * 4) : 0;
  const size_t offGf = use_b1 ? take((size_t)p.total_elems * 4) : 0;
  const size_t offG1tab = take((size_t)c->n_params * sizeof(void *));
  const size_t offGftab = take((size_t)c->n_params * sizeof(void *));
  const size_t offPrep = (use_l2 || use_b1) ? take(std::max<size_t>(1, p.prep_chunks.size()) * sizeof(DiagChunk)) : 0;
  size_t eig_bytes = 0, max_count = 1, band_all = 0;
  std::vector<size_t> t_need;
  std::vector<EigLayout> eL, eR, eM[2];
  for (auto &b : p.buckets) {
    const size_t B = b.count, m = b.m, n = b.n;
    b.off_L = take(B * b.l_elems() * 4);
    b.off_R = take(B * b.r_elems() * 4);
    b.off_Linv = take(B * b.l_elems() * 4);
    b.off_Rinv = take(B * b.r_elems() * 4);
    if (b.t3) {
      for (int k = 0; k + 2 < b.modes; ++k) {
        b.off_mid[k] = take(B * (size_t)b.td[k + 1] * b.td[k + 1] * 4);
        b.off_midinv[k] = take(B * (size_t)b.td[k + 1] * b.td[k + 1] * 4);
      }
      b.off_desc3 = take(B * (size_t)b.split3 * sizeof(BlockDesc));
    }
    b.off_P = take(B * m * n * 4);
    // the preconditioning products run on the fp16 matrix cores from operands kept split in two
    // scaled fp16 planes, float32 directions on the bf16 ones from three planes.  These also have to be split in every
    // step, and blocks of one 128-wide tile leave half of the 256-wide one idle: their terms are made on the way into LDS.
    // Factors and both products of 2^25 float32 elements in blocks of 1024, 512, 256 and 192: 1.61, 1.01, 0.74 and 0.99 ms with the terms made
    // there, 1.42, 0.87, 0.69 and 0.87 on planes.  Just above a multiple of the tile the planes lose by their padding (144: 1.18 and
    // 1.38, 264: 1.16 and 1.56, 392: 1.19 and 1.44), which the line does not take into account.
    const bool dir32 = c->grad_dtype != SHAMPOO_GRAD_BF16 || use_l2 || use_b1;
    b.planes = b.bf16_mfma && c->precond_matrix_cores != SHAMPOO_MATRIX_CORES_FP32 && (!dir32 || (b.m > BM && b.n > BN));
    b.three = b.planes && dir32;
    if (b.planes) {
      b.off_Linvp = take(B * m * m * (b.three ? 6 : 4));
      b.off_Rinvp = take(B * n * n * (b.three ? 6 : 4));
      b.off_stat_l = take(B * 8);
      b.off_stat_r = take(B * 8);
      b.off_gmaxp = take(B * b.geom.chunks * 4);
      b.off_s_g = take(B * 4);
      b.off_t_scale = take(B * 4);
      b.off_inv_ts = take(B * 4);
    }
    b.off_desc = take(B * sizeof(BlockDesc));
    b.off_sgp = take(B * b.geom.chunks * 4);
    // partial sums of ||P_shampoo||^2: one per tile of the last product (tensor blocks: the
    // (d2 d1) x d3 product of the third dimension) or per chunk of an elementwise pass
    auto parts = [](size_t rows, size_t cols) { return ((rows + GEMM_SMALL - 1) / GEMM_SMALL) * ((cols + GEMM_SMALL - 1) / GEMM_SMALL); };
    size_t ssh_parts = std::max(parts(m, n), (size_t)b.geom.chunks);
    if (b.t3) ssh_parts = std::max(ssh_parts, parts(m * n / b.dlast(), b.dlast()));
    if (b.t3 && b.modes >= 3) ssh_parts = std::max(ssh_parts, (size_t)narrow_tiles(m * n / b.dlast() / b.td[b.modes - 2], b.td[b.modes - 2]));
    b.off_sshp = take(B * ssh_parts * 4);
    b.off_scale = take(B * 4);
    b.off_norms = take(B * 8);
    b.off_gmax = take(B * 8);
    b.split_factor = b.three && !use_b1;   // the directions' gradient feeds the factors too
    // float32 or two fp16 planes; tensor blocks: float64 sums of the ranges of k of two dimensions (split_gram), and float32
    // ones of the last
    size_t need = B * m * n * 4;
    if (b.t3) need = B * m * n * 16 + (b.modes >= 3 ? B * b.split3 * b.dlast() * b.dlast() * 4 : 0);
    if (b.three) need = std::max(need, std::min(B, std::max<size_t>(1, PLANE_BYTES / (12 * m * n))) * 12 * m * n);
    if (b.three) {                       // even shares
      const int64_t most = std::min<int64_t>(b.count, (int64_t)(need / (12 * m * n))), passes = (b.count + most - 1) / most;
      b.plane_chunk = (int32_t)((b.count + passes - 1) / passes);
    }
    t_need.push_back(align_up(need));
    if (c->grad_dtype == SHAMPOO_GRAD_BF16 && b.bf16_mfma && !use_l2) b.off_Gt = take(B * m * n * 2);
    // a diagonalised side needs no eigensolver workspace (stand-in layout of a 1 x 1 problem)
    const int em = b.diagL ? 1 : b.m, en = b.diagR ? 1 : b.rdim();
    const bool warm = c->warm_start_roots != 0 && c->root_method == SHAMPOO_ROOT_EIGH && !b.t3;   // tensor blocks start cold
    const float r_exp = b.t3 ? 2.f * c->root_exponent / (float)b.modes : c->root_exponent;
    auto eig = [&](int n_) {
      const EigLayout e = eig_layout(n_, b.count, !warm && band_serves(n_, r_exp));
      if (e.band.bytes) band_all += band_layout_of(n_, b.count).bytes;
      return e;
    };
    eL.push_back(eig(em));
    eR.push_back(eig(en));
    if (warm && eL.back().np > 0) b.off_QtL = take(B * (size_t)eL.back().np * eL.back().np * 4);
    if (warm && eR.back().np > 0) b.off_QtR = take(B * (size_t)eR.back().np * eR.back().np * 4);
    for (int k = 0; k < 2; ++k) eM[k].push_back(eig(b.td[k + 1]));
    // under coupled Newton the eigensolver is the fallback of the guard (Sec. 3.2.3): room for both
    if (c->root_method == SHAMPOO_ROOT_NEWTON)
      eig_bytes = std::max(eig_bytes, std::max(std::max(newton_layout(em, b.count).bytes, newton_layout(en, b.count).bytes),
                                               std::max(newton_layout(b.td[1], b.count).bytes, newton_layout(b.td[2], b.count).bytes)));
    eig_bytes = std::max(eig_bytes, std::max(std::max(eL.back().bytes, eR.back().bytes),
                                             std::max(eM[0].back().bytes, eM[1].back().bytes)));
    max_count = std::max(max_count, (size_t)b.count);
  }
  // roots of all sizes at once (band_roots)
  eig_bytes = std::max(eig_bytes, std::min(band_all, band_pass_bytes()));
  // Sets of buckets whose scratch fits side by side into what the largest bucket needs, or SET_BYTES
  size_t t_bytes = 0, t2_bytes = 0;
  {
    const size_t room = std::max(SET_BYTES, t_need.empty() ? 0 : *std::max_element(t_need.begin(), t_need.end()));
    size_t at = 0, at2 = 0;
    int set = 0;
    for (size_t i = 0; i < p.buckets.size(); ++i) {
      Bucket &b = p.buckets[i];
      if (at + t_need[i] > room) { ++set; at = 0; at2 = 0; }
      b.set = set; b.off_t = at; b.off_t2 = at2;
      at += t_need[i];
      if (b.t3) at2 += align_up((size_t)b.count * b.m * b.n * 4);
      t_bytes = std::max(t_bytes, at); t2_bytes = std::max(t2_bytes, at2);
    }
    p.n_sets = p.buckets.empty() ? 0 : set + 1;
  }
  // Planes of the transposes wait in T for the products; otherwise nothing does while the roots are taken, whose scratch
  // is then the same memory
  bool t_waits = false;
  for (auto &b : p.buckets) {
    b.cols_wait = p.n_sets == 1 && b.three && b.split_factor && b.plane_chunk == b.count;
    t_waits = t_waits || b.cols_wait;
  }
  const size_t offT = take(t_waits ? t_bytes : std::max(t_bytes, eig_bytes));
  const size_t offT2 = t2_bytes ? take(t2_bytes) : 0;
  std::vector<size_t> offGb(c->n_params, 0), offWb(c->n_params, 0);
  bool has_tensor = false;
  for (int i = 0; i < c->n_params; ++i) {
    if (p.pshape[i].kind != P_TENSOR) continue;
    has_tensor = true;
    const size_t el = (size_t)p.pshape[i].elems();
    offGb[i] = take(el * (c->grad_dtype == SHAMPOO_GRAD_BF16 ? 2 : 4));
    offWb[i] = take(el * 4);
  }
  const size_t offW = take((size_t)c->n_params * sizeof(void *));
  const size_t offG = take((size_t)c->n_params * sizeof(void *));
  const size_t offD = take(std::max<size_t>(1, p.diag_chunks.size()) * sizeof(DiagChunk));
  int64_t n_small = 0;
  bool small_half = true;
  for (auto &b : p.buckets)
    if (b.small()) { n_small += b.count; small_half = small_half && b.m <= SB_HALF && b.n <= SB_HALF; }
  const size_t offSmall = take(std::max<size_t>(1, (size_t)n_small) * sizeof(SmallBlock));
  const size_t offC = take(64);
  const size_t offNf = take(max_count * 4);
  const size_t offE = t_waits ? take(eig_bytes) : offT;
  if (o) {
    o->off_A = offA; o->off_M = offM; o->off_T = offT;
    o->off_G1 = offG1; o->off_Gf = offGf; o->off_g1tab = offG1tab; o->off_gftab = offGftab; o->off_prep = offPrep;
    o->use_l2 = use_l2; o->use_b1 = use_b1; o->off_wtab = offW; o->off_gtab = offG;
    o->off_diag = offD; o->off_count = offC; o->off_eig = offE; o->eig_bytes = eig_bytes;
    o->off_small = offSmall; o->n_small = n_small; o->small_half = small_half; o->n_prep_rest = p.n_prep_rest;
    o->eig_L = eL; o->eig_R = eR; o->eig_mid[0] = eM[0]; o->eig_mid[1] = eM[1];
    o->upper_stale.assign(o->plan.buckets.size(), 0);
    o->half_stale.assign(o->plan.buckets.size(), 0);
    o->off_nfail = offNf;
    o->off_T2 = offT2; o->off_Gb = offGb; o->off_Wb = offWb; o->has_tensor = has_tensor;
  }
  return off;
}

struct StageTimer {
  shampoo_opt *o; int stage; hipStream_t s; bool on; hipEvent_t a{};
  StageTimer(const StageTimer &) = delete;
  StageTimer(shampoo_opt *o_, int st, hipStream_t s_) : o(o_), stage(st), s(s_), on(o_->timing) {
    // room for the interval now: nothing may throw on the way out
    if (on && o->intervals[st].size() == o->intervals[st].capacity()) o->intervals[st].reserve(std::max<size_t>(16, 2 * o->intervals[st].size()));
    if (on) { if (hipEventCreate(&a) != hipSuccess) { on = false; return; } (void)hipEventRecord(a, s); }
  }
  ~StageTimer() {
    if (!on) return;
    hipEvent_t b;
    if (hipEventCreate(&b) != hipSuccess) { (void)hipEventDestroy(a); return; }
    (void)hipEventRecord(b, s);
    o->intervals[stage].push_back({a, b});
  }
};

// Re-splits the roots of every bucket that keeps them as planes (after create and after
// every refresh).
int split_roots(shampoo_opt *o, hipStream_t s) {
  int rc;
  Batch<ClearArgs> clears(clear_kernel, 256, s);
  Batch<MatrixStatsArgs> stats(matrix_stats_kernel, 256, s);
  Batch<SplitRootsArgs> two(split_roots_kernel<false>, 256, s), three(split_roots_kernel<true>, 256, s);
  for (auto &b : o->plan.buckets) {
    if (!b.planes) continue;
    for (int side = 0; side < 2; ++side) {
      const int n = side == 0 ? b.m : b.n;
      const float *x = reinterpret_cast<const float *>(o->ws + (side == 0 ? b.off_Linv : b.off_Rinv));
      float *stat = reinterpret_cast<float *>(o->ws + (side == 0 ? b.off_stat_l : b.off_stat_r));
      const int64_t per = (int64_t)n * n;
      const MatrixStatsArgs ms{x, stat, n, std::max(1, std::min(32, n / 32)), b.count};
      const SplitRootsArgs sr{x, stat, reinterpret_cast<uint16_t *>(o->ws + (side == 0 ? b.off_Linvp : b.off_Rinvp)), per,
                              (int32_t)((per + 1023) / 1024), b.count};
      if ((rc = clears.add(ClearArgs{stat, 2 * b.count}, (2 * (int64_t)b.count + 255) / 256)) ||
          (rc = stats.add(ms, (int64_t)ms.parts * b.count)) || (rc = (b.three ? three : two).add(sr, (int64_t)sr.pieces * b.count)))
        return rc;
    }
  }
  if ((rc = clears.flush()) || (rc = stats.flush()) || (rc = two.flush())) return rc;
  return three.flush();
}

// Coupled Newton with the guard of Sec. 3.2.3.  The paper retries a failed root computation in
// higher precision and keeps the previous root only if that fails too; here the float32
// iteration is the first attempt, and a matrix whose iterates do not stay finite (a condition
// number beyond float32) is handed to the eigendecomposition, which works on a float64 copy.
// Whether any matrix failed is read back, so a refresh under root_method = NEWTON waits for
// the stream once per factor batch; failures of the fallback are what gets counted.
int newton_root_guarded(shampoo_opt *o, const float *F, int dim, int count, float r_exp, float c2, float *Fi,
                        const EigLayout &lay, hipStream_t s) {
  const shampoo_config &c = o->cfg;
  unsigned char *ws = o->ws;
  unsigned long long *counters = reinterpret_cast<unsigned long long *>(ws + o->off_count);
  unsigned long long *newton_failed = counters + 1;
  int32_t *flags = reinterpret_cast<int32_t *>(ws + o->off_nfail);
  const float tol = c.newton_tolerance > 0.f ? c.newton_tolerance : 1e-6f;
  const int cap = c.newton_max_iterations > 0 ? c.newton_max_iterations : 100;
  int rc = launch_fill(reinterpret_cast<float *>(newton_failed), 0.f, 2, s);
  if (rc) return rc;
  rc = newton_root_batched(F, dim, count, c.epsilon, newton_p_of(r_exp), c2, tol, cap, Fi, nullptr, flags, newton_failed,
                           ws + o->off_eig, newton_layout(dim, count), s);
  if (rc) return rc;
  unsigned long long n_failed = 0;
  HIP_TRY(hipMemcpyAsync(&n_failed, newton_failed, sizeof(n_failed), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  if (n_failed == 0) return SHAMPOO_OK;
  return root_inverse_batched(F, dim, count, c.epsilon, r_exp, c2, Fi, nullptr, nullptr, counters, ws + o->off_eig, lay, s,
                              &o->aux, flags);
}

// The bf16 factor update writes only the tiles on and below the diagonal of tiles, the step of a small block in one
// workgroup only the lower triangle; whoever needs the whole symmetric factor (the refresh, the state query) completes
// it first.  half: all above the diagonal.  One side (0: L, 1: R) of `count` blocks of a bucket from slot `first` on.
int complete_factor(shampoo_opt *o, size_t bucket, int side, int first, int count, bool half, Batch<MirrorArgs> &mirrors) {
  if (!half && !o->upper_stale[bucket]) return SHAMPOO_OK;
  const Bucket &b = o->plan.buckets[bucket];
  const int n = side == 0 ? b.m : b.n, pieces = (n + 31) / 32;
  if (n <= (half ? 1 : BM)) return SHAMPOO_OK;        // a single tile: nothing above the diagonal of tiles
  float *c = reinterpret_cast<float *>(o->ws + (side == 0 ? b.off_L : b.off_R)) + (int64_t)first * n * n;
  return mirrors.add(MirrorArgs{c, n, half ? 1 : 0, pieces, count}, (int64_t)pieces * pieces * count);
}
int complete_factors(shampoo_opt *o, size_t bucket, bool half, Batch<MirrorArgs> &mirrors) {
  for (int side = 0; side < 2; ++side)
    if (const int rc = complete_factor(o, bucket, side, 0, o->plan.buckets[bucket].count, half, mirrors)) return rc;
  return SHAMPOO_OK;
}

// A factor of dimension `dim` that has so far summed (step + 1) gradients of `cols` columns
// each is a near-singular Gram matrix until it holds a few times more columns than it has
// rows (a Gaussian dim x N matrix has the condition number ((sqrt N + sqrt dim) / (sqrt N -
// sqrt dim))^2 squared into its Gram matrix: 1e7 and more at N = dim, 34 at N = 2 dim, 9 at
// N = 4 dim).  While it is, a root taken from it weights its smallest eigenvalues most, and
// the bf16 factor update sums in float64 (syrk_bf16.h).
constexpr int64_t WARM_RESTART_PERIOD = 16;

inline bool young_factor(int64_t step, int cols, int dim) { return (step + 1) * (int64_t)cols < 4 * (int64_t)dim; }

// Whether what is enqueued on s goes into a graph.  A query that fails (another capture may forbid it) counts as one that does.
bool recording(hipStream_t s) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

// The device's tables of parameter and gradient pointers.  The pointers travel as kernel
// arguments: nothing on the host has to outlive the call, so the stream is not waited for, and
// a training loop whose gradients come in other buffers every step pays one or two launches of
// a few microseconds (two copies from pageable memory behind a drained stream before: a step of
// 512 blocks of 128 x 128 took 482 us, now 168).
// A launch recorded into a graph writes in every replay and not now, and the host learns of no replay: a recorded step always
// brings its pointers, and from then on every eager one does.
int send_pointer_tables(shampoo_opt *o, hipStream_t s) {
  const bool record = recording(s);
  if (!o->tables_stale && !record) return SHAMPOO_OK;
  const int np = o->cfg.n_params;
  for (int at = 0; at < np; at += POINTER_SET) {
    PointerSet ps;
    ps.w_table = reinterpret_cast<void **>(o->ws + o->off_wtab) + at;
    ps.g_table = reinterpret_cast<void **>(o->ws + o->off_gtab) + at;
    ps.count = std::min(POINTER_SET, np - at);
    for (int k = 0; k < ps.count; ++k) {
      // tensor parameters are worked on in block-contiguous copies inside the workspace
      const int i = at + k;
      const bool t = o->plan.pshape[i].kind == P_TENSOR;
      ps.w[k] = t ? o->ws + o->off_Wb[i] : o->last_w[i];
      ps.g[k] = t ? o->ws + o->off_Gb[i] : o->last_g[i];
    }
    hipLaunchKernelGGL(pointer_table_kernel, dim3(1), dim3(256), 0, s, ps);
    HIP_TRY(hipGetLastError());
  }
  o->tables_recorded = o->tables_recorded || record;
  o->tables_stale = o->tables_recorded;
  return SHAMPOO_OK;
}

// GT: element type of the caller's gradients.  GS: of the gradients that feed the factors and
// the grafting state (GT, or float when l2 weight decay materialises G + wd W).  GD: of the
// gradients that feed the directions (float when filtered or shifted, else GT).
template <typename GT, typename GS, typename GD>
int step_impl(shampoo_opt *o, float lr, int64_t step, hipStream_t s) {
  const shampoo_config &c = o->cfg;
  Plan &p = o->plan;
  unsigned char *ws = o->ws;
  float *A = reinterpret_cast<float *>(ws + o->off_A);
  float *M = c.momentum > 0.f ? reinterpret_cast<float *>(ws + o->off_M) : nullptr;
  float *G1 = o->use_l2 ? reinterpret_cast<float *>(ws + o->off_G1) : nullptr;
  float *Gf = o->use_b1 ? reinterpret_cast<float *>(ws + o->off_Gf) : nullptr;
  void *const *wtab = reinterpret_cast<void *const *>(ws + o->off_wtab);
  const void *const *gtab = reinterpret_cast<const void *const *>(ws + o->off_gtab);
  // gradients feeding factors + grafting state / feeding the directions
  const void *const *gs_tab = o->use_l2 ? reinterpret_cast<const void *const *>(ws + o->off_g1tab) : gtab;
  const void *const *gd_tab = o->use_b1 ? reinterpret_cast<const void *const *>(ws + o->off_gftab) : gs_tab;
  unsigned long long *fail_count = reinterpret_cast<unsigned long long *>(ws + o->off_count);
  const bool use_shampoo = step >= c.start_preconditioning_step;
  const bool refresh = use_shampoo && (step % c.precondition_frequency == 0);
  // EMA weights from the float32 beta2 the caller gave, evaluated in float64
  const double alpha = c.beta2 < 1.f ? 1.0 - (double)c.beta2 : 1.0;
  const double beta = c.beta2 < 1.f ? (double)c.beta2 : 1.0;
  const float wd_l2 = o->use_l2 ? c.weight_decay : 0.f;
  const float wd_dec = (c.weight_decay > 0.f && c.use_decoupled_weight_decay) ? c.weight_decay : 0.f;
  const int sgd = c.grafting_type == SHAMPOO_GRAFT_SGD ? 1 : 0;
  // bias correction (Sec. 3.1.1): directions use Gf / (1 - beta1^(t+1)), roots are taken of
  // L / (1 - beta2^(t+1)); the stored state stays uncorrected
  const bool bc = c.use_bias_correction != 0;
  const float c1 = (bc && c.beta1 > 0.f) ? (float)(1.0 / (1.0 - std::pow((double)c.beta1, (double)(step + 1)))) : 1.f;
  const float c2 = (bc && c.beta2 < 1.f) ? (float)(1.0 / (1.0 - std::pow((double)c.beta2, (double)(step + 1)))) : 1.f;
  // grafting second moment: sum (AdaGrad) or EMA (RMSprop, Adam; Adam bias-corrected on request)
  const bool ema = c.grafting_type == SHAMPOO_GRAFT_RMSPROP || c.grafting_type == SHAMPOO_GRAFT_ADAM;
  const float a_decay = ema ? c.grafting_beta2 : 1.f;
  const float a_gain = (ema && c.grafting_beta2 < 1.f) ? (float)(1.0 - (double)c.grafting_beta2) : 1.f;
  const float a_bc = (c.grafting_type == SHAMPOO_GRAFT_ADAM && bc && c.grafting_beta2 < 1.f)
                         ? (float)(1.0 / (1.0 - std::pow((double)c.grafting_beta2, (double)(step + 1)))) : 1.f;
  int rc;

  // Blocks of at most 128 x 128 take the whole step in one workgroup (gradient block
  // resident in LDS) whenever no refresh separates the factor update from the
  // preconditioning (l2 weight decay and SGD grafting go stage by stage).
  const bool small_ok = use_shampoo && !refresh && !o->use_l2 && !sgd && o->n_small > 0;
  auto fused = [&](const Bucket &b) { return small_ok && b.small(); };
  // A step of nothing but such blocks and 1-D parameters, of which few enough, brings its pointers along
  const bool by_value = small_ok && o->n_small == (int64_t)p.blocks.size() && c.n_params <= SB_POINTERS;
  if (!by_value && (rc = send_pointer_tables(o, s))) return rc;
  DiagArgs d;
  d.chunks = reinterpret_cast<const DiagChunk *>(ws + o->off_diag);
  d.w_table = wtab; d.g_table = gtab; d.a_state = A; d.m_state = M; d.gf_state = Gf;
  d.graft_eps = c.graft_epsilon; d.mu = c.momentum; d.lr = lr;
  d.beta1 = c.beta1; d.wd_l2 = wd_l2; d.wd_decoupled = wd_dec; d.nesterov = c.use_nesterov ? 1 : 0;
  d.gd_scale = c1; d.a_decay = a_decay; d.a_gain = a_gain; d.a_bc = a_bc;

  // Tensor parameters (Sec. 2.3): the step works on block-contiguous copies of their gradient
  // and of the parameter itself; the pointer tables on the device name those copies.
  TensorCopySet copies{};
  int copy_wgs = 0;
  auto send_copies = [&](bool scatter) {
    if (copies.count == 0) return;
    if (scatter) hipLaunchKernelGGL(tensor_block_copy_kernel<true>, dim3((unsigned)copy_wgs), dim3(256), 0, s, copies);
    else hipLaunchKernelGGL(tensor_block_copy_kernel<false>, dim3((unsigned)copy_wgs), dim3(256), 0, s, copies);
    copies.count = 0; copy_wgs = 0;
  };
  auto add_copy = [&](int i, void *tensor, void *copy, int bytes, bool scatter) {
    const PShape &ps = p.pshape[i];
    TensorCopyArgs ta{};
    ta.tensor = tensor; ta.copy = copy; ta.bytes = bytes;
    ta.D1 = ps.d[0]; ta.D2 = ps.d[1]; ta.D3 = ps.d[2]; ta.D4 = ps.d[3]; ta.b = c.block_size;
    ta.k2n = (int32_t)((ps.d[1] + c.block_size - 1) / c.block_size);
    ta.k3n = (int32_t)((ps.d[2] + c.block_size - 1) / c.block_size);
    ta.k4n = (int32_t)((ps.d[3] + c.block_size - 1) / c.block_size);
    const int64_t per = std::min<int64_t>(c.block_size, ps.d[0]) * std::min<int64_t>(c.block_size, ps.d[1]) *
                        std::min<int64_t>(c.block_size, ps.d[2]) * std::min<int64_t>(c.block_size, ps.d[3]);
    ta.chunks = (int32_t)std::max<int64_t>(1, std::min<int64_t>(64, (per + 2047) / 2048));
    const int64_t wgs = (int64_t)ta.chunks * (int64_t)p.param_blocks[i].size();
    if (copies.count == TENSOR_COPY_SET || copy_wgs + wgs > ((int64_t)1 << 30)) send_copies(scatter);
    ta.first = copy_wgs;
    copy_wgs += (int)wgs;
    copies.t[copies.count++] = ta;
  };
  if (o->has_tensor) {
    StageTimer t(o, SHAMPOO_STAGE_GRAFT, s);
    for (int i = 0; i < c.n_params; ++i) {
      if (p.pshape[i].kind != P_TENSOR) continue;
      add_copy(i, const_cast<void *>(o->last_g[i]), ws + o->off_Gb[i], (int)sizeof(GT), false);
      add_copy(i, o->last_w[i], ws + o->off_Wb[i], 4, false);
    }
    send_copies(false);
    HIP_TRY(hipGetLastError());
  }

  const int64_t n_prep = small_ok ? o->n_prep_rest : (int64_t)p.prep_chunks.size();
  if ((o->use_l2 || o->use_b1) && n_prep > 0) {
    StageTimer t(o, SHAMPOO_STAGE_GRAFT, s);
    PrepArgs pa;
    pa.chunks = reinterpret_cast<const DiagChunk *>(ws + o->off_prep);
    pa.w_table = wtab; pa.g_table = gtab; pa.g1 = G1; pa.gf = Gf; pa.wd_l2 = wd_l2; pa.beta1 = c.beta1;
    hipLaunchKernelGGL(prep_kernel<GT>, dim3((unsigned)n_prep), dim3(EW_THREADS), 0, s, pa);
    HIP_TRY(hipGetLastError());
  }
  // The small blocks' kernel beside the stages of the others.  The fork and the join cost the host some 15 us, which shows
  // where the launches of the stages take as long as their kernels: not below 4e6 elements in the stages.  Step one after the other and so:
  // ResNet-50 in blocks of 256, 101 parameters, 283 and 241 us; one layer of 640 in blocks of 512 183 and 144; ResNet-50 with
  // convolution tensors, 101 and 161 parameters, 234 and 205, 695 and 682; its first 14 (0.2e6 elements) 104 and 130.
  const bool beside = small_ok && o->overlap && !o->timing && o->aux.state == 1;
  Fork helper;
  if (beside && (rc = helper.begin(&o->aux, 0, 1, s))) return rc;
  if (small_ok) {
    StageTimer t(o, SHAMPOO_STAGE_FUSED, s);
    const hipStream_t own = beside ? o->aux.stream[0] : s;
    SmallStepArgs f;
    f.blocks = reinterpret_cast<const SmallBlock *>(ws + o->off_small); f.ws = ws;
    f.w_table = wtab; f.g_table = gtab; f.a_state = A; f.m_state = M; f.gf_state = Gf;
    f.alpha_d = alpha; f.beta_d = beta;
    f.graft_eps = c.graft_epsilon; f.mu = c.momentum; f.lr = lr; f.wd_decoupled = wd_dec;
    f.nesterov = c.use_nesterov ? 1 : 0;
    f.a_decay = a_decay; f.a_gain = a_gain; f.a_bc = a_bc; f.beta1 = c.beta1; f.gd_scale = c1;
    f.fp32 = c.precond_matrix_cores == SHAMPOO_MATRIX_CORES_FP32 ? 1 : 0;
    f.n_blocks = (int32_t)o->n_small; f.diag = d;
    f.by_value = by_value ? 1 : 0;
    if (by_value)
      for (int i = 0; i < c.n_params; ++i) { f.w_ptr[i] = o->last_w[i]; f.g_ptr[i] = o->last_g[i]; }
    const dim3 grid((unsigned)(o->n_small + (int64_t)p.diag_chunks.size())), block(SB_THREADS);
    constexpr bool FILT_ONLY = sizeof(GT) == 2 && sizeof(GD) == 4;   // bf16 gradients with float directions are filtered
    if (FILT_ONLY || Gf) {
      if (o->small_half) hipLaunchKernelGGL((block_step_small_kernel<GT, SB_HALF, true>), grid, block, 0, own, f);
      else hipLaunchKernelGGL((block_step_small_kernel<GT, SB, true>), grid, block, 0, own, f);
    } else {
      if (o->small_half) hipLaunchKernelGGL((block_step_small_kernel<GT, SB_HALF, false>), grid, block, 0, own, f);
      else hipLaunchKernelGGL((block_step_small_kernel<GT, SB, false>), grid, block, 0, own, f);
    }
    HIP_TRY(hipGetLastError());
    for (size_t i = 0; i < p.buckets.size(); ++i) if (p.buckets[i].small()) o->half_stale[i] = 1;
  }
  // ---- stage by stage.  Buckets are independent of one another, so that each stage is one launch for all of them
  // (group.h); those of a set have their own parts of the scratch T, and sets follow one another.
  auto bucket_t = [&](const Bucket &b) { return reinterpret_cast<float *>(ws + o->off_T + b.off_t); };
  // Tensor blocks: the Gram matrix of an unfolding in ranges of k (gram_split.h), whose sums go through `sums` in float64, as
  // the one sum is held: it has room for m n of them per block of the bucket.
  // products with a block's gradients: the powers of two that keep their small terms from underflowing
  auto scale_factor = [&](const Bucket &b, GemmArgs &g, int per) {
    g.gmax = reinterpret_cast<const float *>(ws + b.off_gmax); g.gmax_per = per; g.scale_a = g.scale_b = 1; g.unscale = 2;
  };
  auto scale_direction = [&](const Bucket &b, GemmArgs &g, bool gradient, bool result) {
    g.gmax = reinterpret_cast<const float *>(ws + b.off_gmax) + b.count; g.gmax_per = 1;
    g.scale_b = gradient ? 1 : 0; g.unscale = result ? 1 : 0;
  };
  auto split_gram = [&](const Bucket &b, GemmArgs &g, double *sums) {
    const GramSplit sp = gram_split(g.K, (int64_t)b.m * b.n / ((int64_t)g.M * g.M), (int64_t)g.tiles * g.batch, BK);
    if (sp.ranges <= 1) return 1;
    g.ksplit = sp.ranges; g.krange = sp.range;
    g.c64 = sums; g.batch *= g.ksplit;
    return (int)g.ksplit;
  };
  auto reduce_gram = [&](Batch<GramReduceArgs> &to, const void *partial, size_t off_factor, int d, int splits, int count) {
    GramReduceArgs gr;
    gr.partial = partial; gr.factor = reinterpret_cast<float *>(ws + off_factor); gr.d = d; gr.splits = splits; gr.blocks = count;
    gr.alpha = alpha; gr.beta = beta;
    return to.add(gr, (((int64_t)d * d + 255) / 256) * count);
  };
  // scales of the fp16 operands of a bucket's preconditioning products (and of R's update)
  auto add_x2_scales = [&](Batch<X2ScaleArgs> &to, const Bucket &b) {
    X2ScaleArgs xs;
    xs.gmax_partial = reinterpret_cast<const float *>(ws + b.off_gmaxp); xs.parts = b.geom.chunks;
    xs.stat_l = reinterpret_cast<const float *>(ws + b.off_stat_l); xs.stat_r = reinterpret_cast<const float *>(ws + b.off_stat_r);
    xs.c1 = c1; xs.blocks = b.count;
    xs.s_g = reinterpret_cast<float *>(ws + b.off_s_g);
    xs.t_scale = reinterpret_cast<float *>(ws + b.off_t_scale); xs.inv_ts = reinterpret_cast<float *>(ws + b.off_inv_ts);
    return to.add(xs, b.count);
  };
  // the planes of blocks [b0, b0 + cnt) of a bucket's float32 gradients, after add_x2_scales
  auto planes_of = [&](const Bucket &b, int b0, int cnt, bool rows) {
    BlockPlanesArgs bp;
    bp.desc = reinterpret_cast<const BlockDesc *>(ws + b.off_desc) + b0; bp.g_table = gd_tab;
    bp.scale = reinterpret_cast<const float *>(ws + b.off_s_g) + b0; bp.m = b.m; bp.n = b.n; bp.blocks = cnt;
    bp.plane_stride = (int64_t)cnt * b.m * b.n;
    bp.cols = reinterpret_cast<uint16_t *>(bucket_t(b)); bp.rows = rows ? bp.cols + 3 * bp.plane_stride : nullptr;
    return bp;
  };
  auto planes_wgs = [](const Bucket &b, int cnt) { return (int64_t)((b.n + 63) / 64) * ((b.m + 63) / 64) * cnt; };
  auto syrk_wgs = [](const SyrkBf16Args &g) { return (int64_t)g.tiles * g.batch; };
  auto tensor_chunks = [](const Bucket &b) { return (int32_t)std::max<int64_t>(1, std::min<int64_t>(64, ((int64_t)b.m * b.n + 2047) / 2048)); };
  // how a bucket's factors are updated: fp16 / bf16 matrix cores, three bf16 planes, three bf16 terms made on the way into LDS
  enum { F_BF16, F_SPLIT, F_F32 };
  auto factor_path = [&](const Bucket &b) {
    if (sizeof(GS) == 2 && b.bf16_mfma && o->ptrs_aligned16) return F_BF16;
    if (sizeof(GS) == 4 && b.split_factor && use_shampoo && o->ptrs_aligned16) return F_SPLIT;
    return F_F32;
  };
  auto on_planes = [&](const Bucket &b) { return !b.t3 && !b.whole() && b.planes && o->ptrs_aligned16; };
  // products that split their operands on the way into LDS: they scale by the largest element of a block, which grafting finds.  Not for
  // others: its maxima over a block's workgroups, two atomics each on the same words, took 15 of 39 us (12 blocks of 1024), 24 of 58
  // (two bf16 parameters of 3000 x 3000, both factors diagonal: no product at all)
  auto scaled_inside = [&](const Bucket &b) { return !(b.diagL && b.diagR) && (factor_path(b) == F_F32 || (use_shampoo && !on_planes(b))); };
  auto fill_ew = [&](EwArgs &e, const Bucket &b) {
    e.desc = reinterpret_cast<const BlockDesc *>(ws + b.off_desc); e.w_table = wtab; e.g_table = gs_tab; e.gd_table = gd_tab; e.a_state = A; e.m_state = M;
    e.m = b.m; e.n = b.n; e.blocks = b.count; e.geom = b.geom; e.graft_eps = c.graft_epsilon; e.mu = c.momentum; e.lr = lr;
    e.gmax = reinterpret_cast<float *>(ws + b.off_gmax);
    e.sgd_graft = sgd; e.gd_scale = c1; e.a_decay = a_decay; e.a_gain = a_gain; e.a_bc = a_bc;
  };
  // the buckets of a set that go stage by stage
  auto members = [&](int set) {
    std::vector<Bucket *> v;
    for (auto &b : p.buckets) if (b.set == set && !fused(b)) v.push_back(&b);
    return v;
  };
  for (int set = 0; set < p.n_sets; ++set) {
    const std::vector<Bucket *> todo = members(set);
    if (todo.empty()) continue;
    // grafting state and norm first: the same pass finds max |G| of every block, which scales
    // the fp16 planes of this step's first product
    {
      StageTimer t(o, SHAMPOO_STAGE_GRAFT, s);
      Batch<EwArgs> graft(graft_kernel<GS, GD>, EW_THREADS, s);
      for (Bucket *b : todo) {
        EwArgs e{};
        fill_ew(e, *b);
        e.sg_partial = reinterpret_cast<float *>(ws + b->off_sgp);
        e.same_src = (gs_tab == gd_tab) ? 1 : 0;
        if (b->planes) e.gmax_partial = reinterpret_cast<float *>(ws + b->off_gmaxp);
        if (!scaled_inside(*b)) e.gmax = nullptr;
        if ((rc = graft.add(e, (int64_t)b->geom.chunks * b->count))) return rc;
      }
      if ((rc = graft.flush())) return rc;
    }
    StageTimer t(o, SHAMPOO_STAGE_FACTOR, s);
    // scales, then transposes and planes
    {
      Batch<X2ScaleArgs> scales(x2_scales_kernel, 64, s);
      Batch<TransposeArgs> transposes(transpose_bf16_kernel, 256, s);
      Batch<BlockPlanesArgs> planes(block_planes_kernel, 256, s);
      for (Bucket *b : todo) {
        const int path = factor_path(*b);
        if ((path == F_BF16 && sizeof(GD) == 2 && b->planes) || path == F_SPLIT) if ((rc = add_x2_scales(scales, *b))) return rc;
      }
      if ((rc = scales.flush())) return rc;
      for (Bucket *b : todo) {
        const int path = factor_path(*b);
        if (path == F_BF16) {
          TransposeArgs ta;
          ta.desc = reinterpret_cast<const BlockDesc *>(ws + b->off_desc); ta.g_table = gs_tab; ta.out = reinterpret_cast<uint16_t *>(ws + b->off_Gt);
          ta.m = b->m; ta.n = b->n; ta.blocks = b->count;
          ta.scale = sizeof(GD) == 2 && b->planes ? reinterpret_cast<const float *>(ws + b->off_s_g) : nullptr;
          if ((rc = transposes.add(ta, planes_wgs(*b, b->count)))) return rc;
        } else if (path == F_SPLIT && b->plane_chunk == b->count) {
          if ((rc = planes.add(planes_of(*b, 0, b->count, true), planes_wgs(*b, b->count)))) return rc;
        }
      }
      if ((rc = transposes.flush()) || (rc = planes.flush())) return rc;
    }
    // both factors of matrix blocks
    {
      Batch<MirrorArgs> mirrors(mirror_upper_tiles_kernel, 256, s);
      Batch<SyrkBf16Args> plain(syrk_bf16_kernel<false, false>, GEMM_THREADS, s), plain64(syrk_bf16_kernel<false, true>, GEMM_THREADS, s),
          half(syrk_bf16_kernel<true, false>, GEMM_THREADS, s), half64(syrk_bf16_kernel<true, true>, GEMM_THREADS, s),
          split(syrk_bf16_kernel<false, true, true>, GEMM_THREADS, s);
      GemmBatch<EPI_SYRK> left(gemm_kernels<K_CONTIG, K_CONTIG, GS, GS, EPI_SYRK, true>(), s),
          right(gemm_kernels<ROW_CONTIG, ROW_CONTIG, GS, GS, EPI_SYRK, true>(), s);
      for (Bucket *bp : todo) {
        Bucket &b = *bp;
        const size_t index = &b - p.buckets.data();
        const BlockDesc *desc = reinterpret_cast<const BlockDesc *>(ws + b.off_desc);
        const int path = factor_path(b);
        if (path == F_BF16) {
          // the kernel reads and writes the tiles on and below the diagonal, those on it whole (refresh: this step may be the
          // one that a graph repeats between others)
          if (b.small() && !o->use_l2 && !sgd && (refresh || o->half_stale[index]) && (rc = complete_factors(o, index, true, mirrors))) return rc;
          o->upper_stale[index] = 1;
          const bool x2 = sizeof(GD) == 2 && b.planes;
          SyrkBf16Args sa{};
          sa.desc = desc; sa.ptr_table = gs_tab; sa.alpha = alpha; sa.beta = beta; sa.batch = b.count;
          // L <- beta L + alpha G G^T
          sa.a.from_table = 1;
          sa.c = reinterpret_cast<float *>(ws + b.off_L); sa.c_batch_stride = (int64_t)b.m * b.m; sa.ldc = b.m;
          sa.M = b.m; sa.K = b.n; sa.tiles = b.tiles_m * (b.tiles_m + 1) / 2;
          if ((rc = (young_factor(step, b.n, b.m) ? plain64 : plain).add(sa, syrk_wgs(sa)))) return rc;
          // R <- beta R + alpha (G^T)(G^T)^T
          sa.a.from_table = 0; sa.a.base = ws + b.off_Gt; sa.a.batch_stride = (int64_t)b.m * b.n; sa.a.ld = b.m;
          sa.c = reinterpret_cast<float *>(ws + b.off_R); sa.c_batch_stride = (int64_t)b.n * b.n; sa.ldc = b.n;
          sa.M = b.n; sa.K = b.m; sa.tiles = b.tiles_n * (b.tiles_n + 1) / 2;
          const bool young = young_factor(step, b.m, b.n);
          if (x2) sa.x_scale = reinterpret_cast<const float *>(ws + b.off_s_g);
          if ((rc = (x2 ? (young ? half64 : half) : (young ? plain64 : plain)).add(sa, syrk_wgs(sa)))) return rc;
        } else if (path == F_SPLIT) {
          // float32 gradients: both factors from three bf16 planes, of as many blocks at a time as T has room for
          o->upper_stale[index] = 1;
          for (int b0 = 0; b0 < b.count; b0 += b.plane_chunk) {
            const int cnt = std::min(b.plane_chunk, b.count - b0);
            const BlockPlanesArgs bp = planes_of(b, b0, cnt, true);
            if (b.plane_chunk < b.count) {
              Batch<BlockPlanesArgs> planes(block_planes_kernel, 256, s);
              if ((rc = planes.add(bp, planes_wgs(b, cnt))) || (rc = planes.flush())) return rc;
            }
            SyrkBf16Args sa{};
            sa.alpha = alpha; sa.beta = beta; sa.batch = cnt;
            sa.plane = bp.plane_stride; sa.x_scale = bp.scale;
            for (int side = 0; side < 2; ++side) {
              const int dim = side == 0 ? b.m : b.n, tiles = side == 0 ? b.tiles_m : b.tiles_n;
              sa.a.base = side == 0 ? bp.rows : bp.cols; sa.a.batch_stride = (int64_t)b.m * b.n;
              sa.a.ld = sa.K = side == 0 ? b.n : b.m;
              sa.c_batch_stride = (int64_t)dim * dim; sa.ldc = sa.M = dim;
              sa.c = reinterpret_cast<float *>(ws + (side == 0 ? b.off_L : b.off_R)) + b0 * sa.c_batch_stride;
              sa.tiles = tiles * (tiles + 1) / 2;
              if ((rc = split.add(sa, syrk_wgs(sa)))) return rc;
            }
            if (b.plane_chunk < b.count && (rc = split.flush())) return rc;
          }
        } else if (!b.t3) {
          GemmArgs g{};                // these kernels read the lower triangle and write both
          g.a.from_table = 1; g.b.from_table = 1;
          g.desc = desc; g.ptr_table = gs_tab;
          g.alpha = (float)alpha; g.beta = (float)beta; g.alpha_d = alpha; g.beta_d = beta; g.batch = b.count;
          scale_factor(b, g, 1);
          DiagFactorArgs df{};
          df.desc = desc; df.g_table = gs_tab; df.a = beta; df.b = alpha; df.m = b.m; df.n = b.n;
          if (b.diagL) {
            // l_i <- beta l_i + alpha sum_j G_ij^2 (Sec. 4.2.3)
            df.vec = reinterpret_cast<float *>(ws + b.off_L);
            hipLaunchKernelGGL(diag_row_kernel<GS>, dim3((b.m + 3) / 4, b.count), dim3(256), 0, s, df);
            HIP_TRY(hipGetLastError());
          } else {
            // L <- beta L + alpha G G^T
            g.c = reinterpret_cast<float *>(ws + b.off_L); g.c_batch_stride = (int64_t)b.m * b.m; g.ldc = b.m;
            g.M = b.m; g.N = b.m; g.K = b.n;
            g.tiles_m = g.tiles_n = b.tiles_m; g.tiles = b.tiles_m * (b.tiles_m + 1) / 2;
            left.add(g);
          }
          if (b.diagR) {
            // r_j <- beta r_j + alpha sum_i G_ij^2, rows cut into segments whose partial sums go through T
            df.vec = reinterpret_cast<float *>(ws + b.off_R);
            df.partial = bucket_t(b); df.segs = b.col_segs; df.rows_per_seg = b.rows_per_seg;
            hipLaunchKernelGGL(diag_col_partial_kernel<GS>, dim3((b.n + 255) / 256, b.col_segs, b.count), dim3(256), 0, s, df);
            hipLaunchKernelGGL(diag_col_reduce_kernel, dim3((b.n + 255) / 256, b.count), dim3(256), 0, s, df);
            HIP_TRY(hipGetLastError());
          } else {
            // R <- beta R + alpha G^T G
            g.c = reinterpret_cast<float *>(ws + b.off_R); g.c_batch_stride = (int64_t)b.n * b.n; g.ldc = b.n;
            g.M = b.n; g.N = b.n; g.K = b.m;
            g.tiles_m = g.tiles_n = b.tiles_n; g.tiles = b.tiles_n * (b.tiles_n + 1) / 2;
            right.add(g);
          }
        }
      }
      if ((rc = mirrors.flush())) return rc;
      for (Batch<SyrkBf16Args> *x : {&plain, &plain64, &half, &half64, &split}) if ((rc = x->flush())) return rc;
      if ((rc = left.flush()) || (rc = right.flush())) return rc;
    }
    // Factors of tensor blocks.  First dimension: L_1 <- beta L_1 + alpha G_(1) G_(1)^T, the block being d1 x (d2 d3 d4).
    // Last dimension: the block as (N / d_last) x d_last, read "rows along k"; its rows are cut into split3 ranges, each a
    // batch entry that leaves its Gram matrix in scratch.  Middle dimensions k: the block as pre x d_k x post with its first
    // two indices swapped, d_k x (pre post).  gram_reduce_kernel adds the ranges up in float64 and applies the moving average.
    for (int mid = 0; mid < 2; ++mid) {
      Batch<PermuteArgs> swaps(permute_12_kernel<GS>, 256, s);
      GemmBatch<EPI_SYRK> first(gemm_kernels<K_CONTIG, K_CONTIG, GS, GS, EPI_SYRK, true>(), s),
          middle(gemm_kernels<K_CONTIG, K_CONTIG, float, float, EPI_SYRK, true>(), s),
          last(gemm_kernels<ROW_CONTIG, ROW_CONTIG, GS, GS, EPI_SYRK, true>(), s);
      Batch<GramNarrowArgs> narrow(gram_narrow_kernel<GS>, 256, s);
      Batch<GramReduceArgs> reduce64(gram_reduce_kernel<double>, 256, s), reduce32(gram_reduce_kernel<float>, 256, s);
      for (Bucket *bp : todo) {
        Bucket &b = *bp;
        if (!b.t3) continue;
        const BlockDesc *desc = reinterpret_cast<const BlockDesc *>(ws + b.off_desc);
        const int64_t mn = (int64_t)b.m * b.n;
        // parts of the bucket's scratch: sums of the first dimension, of a middle one, of the last one
        double *sums_l = reinterpret_cast<double *>(bucket_t(b)), *sums_m = sums_l + mn * b.count;
        float *sums_r = reinterpret_cast<float *>(sums_m + mn * b.count), *swapped = reinterpret_cast<float *>(ws + o->off_T2 + b.off_t2);
        GemmArgs g{};
        g.alpha = (float)alpha; g.beta = (float)beta; g.alpha_d = alpha; g.beta_d = beta; g.batch = b.count;
        scale_factor(b, g, 1);
        if (mid == 0) {
          g.a.from_table = 1; g.b.from_table = 1; g.desc = desc; g.ptr_table = gs_tab;
          g.c = reinterpret_cast<float *>(ws + b.off_L); g.c_batch_stride = (int64_t)b.m * b.m; g.ldc = b.m;
          g.M = b.m; g.N = b.m; g.K = b.n;
          g.tiles_m = g.tiles_n = b.tiles_m; g.tiles = b.tiles_m * (b.tiles_m + 1) / 2;
          const int sp = split_gram(b, g, sums_l);
          first.add(g);
          if (sp > 1 && (rc = reduce_gram(reduce64, sums_l, b.off_L, b.m, sp, b.count))) return rc;
          if (b.modes >= 3) {
            const int dl = b.dlast(), inner = b.n / dl;
            if (dl <= 16) {
              GramNarrowArgs gn;
              gn.desc = reinterpret_cast<const BlockDesc *>(ws + b.off_desc3); gn.table = gs_tab; gn.partial = sums_r;
              gn.d = dl; gn.rows = (b.m / b.split3) * inner; gn.entries = b.count * b.split3;
              if ((rc = narrow.add(gn, (gn.entries + 3) / 4))) return rc;
            } else {
              GemmArgs r = g;
              r.desc = reinterpret_cast<const BlockDesc *>(ws + b.off_desc3); r.ksplit = 0; r.c64 = nullptr;
              scale_factor(b, r, b.split3);
              r.c = sums_r; r.c_batch_stride = (int64_t)dl * dl; r.ldc = dl;
              r.M = dl; r.N = dl; r.K = (b.m / b.split3) * inner;
              r.alpha = 1.f; r.beta = 0.f; r.alpha_d = 1.0; r.beta_d = 0.0; r.batch = b.count * b.split3;
              r.tiles_m = r.tiles_n = (dl + BM - 1) / BM; r.tiles = r.tiles_m * (r.tiles_m + 1) / 2;
              last.add(r);
            }
            if ((rc = reduce_gram(reduce32, sums_r, b.off_R, dl, b.split3, b.count))) return rc;
          }
        }
        if (mid + 2 < b.modes) {
          const int pre = mid == 0 ? b.m : b.m * b.td[1], dk = b.td[mid + 1], post = (int)(mn / ((int64_t)pre * dk));
          PermuteArgs pm{};
          pm.desc = desc; pm.table = gs_tab; pm.dst = swapped; pm.d1 = pre; pm.d2 = dk; pm.d3 = post; pm.blocks = b.count;
          permute_shape(pm, tensor_chunks(b));
          if ((rc = swaps.add(pm, (int64_t)pm.chunks * b.count))) return rc;
          GemmArgs h{};
          h.a.base = swapped; h.a.batch_stride = mn; h.a.ld = pre * post;
          h.b = h.a;
          h.alpha = (float)alpha; h.beta = (float)beta; h.alpha_d = alpha; h.beta_d = beta; h.batch = b.count;
          h.c = reinterpret_cast<float *>(ws + b.off_mid[mid]); h.c_batch_stride = (int64_t)dk * dk; h.ldc = dk;
          h.M = dk; h.N = dk; h.K = pre * post;
          scale_factor(b, h, 1);
          h.tiles_m = h.tiles_n = (dk + BM - 1) / BM; h.tiles = h.tiles_m * (h.tiles_m + 1) / 2;
          const int sp = split_gram(b, h, sums_m);
          middle.add(h);
          if (sp > 1 && (rc = reduce_gram(reduce64, sums_m, b.off_mid[mid], dk, sp, b.count))) return rc;
        }
      }
      if ((rc = swaps.flush()) || (rc = first.flush()) || (rc = middle.flush()) || (rc = narrow.flush()) || (rc = last.flush()) ||
          (rc = reduce64.flush()) || (rc = reduce32.flush()))
        return rc;
    }
  }
  if (refresh) {
    StageTimer t(o, SHAMPOO_STAGE_ROOT, s);
    // Warm start: from the eigenvectors of the previous refresh, except at the first refresh and
    // at every WARM_RESTART_PERIOD-th one (the accumulated float32 eigenvectors drift away from
    // orthogonality by about 1e-6 per solve; a cold solve resets that).
    const bool warm_now = o->n_refresh > 0 && o->n_refresh % WARM_RESTART_PERIOD != 0;
    auto warm_of = [&](const EigLayout &lay, size_t off_qt, int cols, int dim) {
      WarmStart w;
      if (lay.warm && off_qt) { w.qt = reinterpret_cast<float *>(ws + off_qt); w.start = warm_now; }
      w.young = young_factor(step, cols, dim);
      return w;
    };
    // Roots that need no eigenvectors wait until all of them are known, and are then taken together, by exponent; the others
    // one batch after the other.
    std::vector<RootJob> waiting;
    auto take_root = [&](size_t off_factor, size_t off_root, int dim, int count, float r, const EigLayout &lay, const WarmStart &w) {
      const float *F = reinterpret_cast<const float *>(ws + off_factor);
      float *Fi = reinterpret_cast<float *>(ws + off_root);
      RatTable table;
      if (!w.qt && rat_table(r, table) && (dim <= JAC_SMALL_MAX || (lay.band.bytes && band_serves(dim, r)))) {
        waiting.push_back(RootJob{F, dim, count, r, c2, Fi, nullptr, nullptr});
        return (int)SHAMPOO_OK;
      }
      return root_inverse_batched(F, dim, count, c.epsilon, r, c2, Fi, nullptr, nullptr, fail_count, ws + o->off_eig, lay, s, &o->aux, nullptr, w);
    };
    Batch<MirrorArgs> mirrors(mirror_upper_tiles_kernel, 256, s);
    for (size_t i = 0; i < p.buckets.size(); ++i) if ((rc = complete_factors(o, i, false, mirrors))) return rc;
    if ((rc = mirrors.flush())) return rc;
    for (size_t i = 0; i < p.buckets.size(); ++i) {
      auto &b = p.buckets[i];
      const bool newton = c.root_method == SHAMPOO_ROOT_NEWTON;
      if (b.t3) {
        // one root per dimension, exponent 2 r / w (Sec. 2.3: "root 2w")
        const float rw = 2.f * c.root_exponent / (float)b.modes;
        for (int k = 0; k < b.modes; ++k) {
          const bool first = k == 0, last = !first && k == b.modes - 1;
          const size_t fac = first ? b.off_L : last ? b.off_R : b.off_mid[k - 1], inv = first ? b.off_Linv : last ? b.off_Rinv : b.off_midinv[k - 1];
          const EigLayout &lay = first ? o->eig_L[i] : last ? o->eig_R[i] : o->eig_mid[k - 1][i];
          if (newton) rc = newton_root_guarded(o, reinterpret_cast<float *>(ws + fac), b.td[k], b.count, rw, c2, reinterpret_cast<float *>(ws + inv), lay, s);
          else rc = take_root(fac, inv, b.td[k], b.count, rw, lay, WarmStart());
          if (rc) return rc;
        }
        continue;
      }
      for (int side = 0; side < 2; ++side) {
        const size_t fac = side == 0 ? b.off_L : b.off_R, inv = side == 0 ? b.off_Linv : b.off_Rinv;
        const int dim = side == 0 ? b.m : b.n, cols = side == 0 ? b.n : b.m;
        const EigLayout &lay = side == 0 ? o->eig_L[i] : o->eig_R[i];
        if (side == 0 ? b.diagL : b.diagR) {
          // diagonal sides: elementwise root
          DiagRootArgs da;
          da.vec = reinterpret_cast<float *>(ws + fac); da.out = reinterpret_cast<float *>(ws + inv); da.dim = dim; da.epsilon = c.epsilon;
          da.r = c.root_exponent; da.scale = c2; da.fail_count = fail_count;
          hipLaunchKernelGGL(diag_root_kernel, dim3(b.count), dim3(256), 0, s, da);
          HIP_TRY(hipGetLastError());
          continue;
        }
        if (newton && !b.whole())
          rc = newton_root_guarded(o, reinterpret_cast<float *>(ws + fac), dim, b.count, c.root_exponent, c2, reinterpret_cast<float *>(ws + inv), lay, s);
        else rc = take_root(fac, inv, dim, b.count, c.root_exponent, lay, warm_of(lay, side == 0 ? b.off_QtL : b.off_QtR, cols, dim));
        if (rc) return rc;
      }
    }
    while (!waiting.empty()) {
      const float r = waiting[0].r;
      std::vector<RootJob> small, band, rest;
      for (const RootJob &j : waiting) (j.r != r ? rest : j.n <= JAC_SMALL_MAX ? small : band).push_back(j);
      RatTable table;
      if (!rat_table(r, table)) return SHAMPOO_ERR_HYPER;
      // small matrices beside the large ones, on a stream that those do not use
      AuxStreams *aux = !band.empty() && o->aux.ready() ? &o->aux : nullptr;
      const bool apart = aux && !small.empty();
      Fork fork;
      if (apart && (rc = fork.begin(aux, BAND_STREAMS - 1, BAND_STREAMS, s))) return rc;
      if (!small.empty() && (rc = tridiag_roots(small, c.epsilon, fail_count, apart ? aux->stream[BAND_STREAMS - 1] : s, table))) return rc;
      if (!band.empty() && (rc = band_roots(band, c.epsilon, fail_count, ws + o->off_eig, o->eig_bytes, s, aux, table))) return rc;
      if ((rc = fork.join())) return rc;
      waiting.swap(rest);
    }
    o->n_refresh++;
    if ((rc = split_roots(o, s))) return rc;
  }
  for (int set = 0; set < p.n_sets; ++set) {
    const std::vector<Bucket *> todo = members(set);
    if (todo.empty()) continue;
    std::vector<int> ssh_count(todo.size());
    if (use_shampoo) {
      constexpr bool THREE = sizeof(GD) == 4;
      std::optional<StageTimer> timer(std::in_place, o, SHAMPOO_STAGE_PRECOND, s);      // one interval, of all up to the second product
      {
        // on a refresh the roots, and with them their scales, have just changed; filtered gradients have not been scaled yet
        Batch<X2ScaleArgs> scales(x2_scales_kernel, 64, s);
        Batch<BlockPlanesArgs> planes(block_planes_kernel, 256, s);
        for (Bucket *b : todo)
          if (on_planes(*b) && (refresh || (THREE && !b->split_factor)) && (rc = add_x2_scales(scales, *b))) return rc;
        if ((rc = scales.flush())) return rc;
        if (THREE)
          for (Bucket *b : todo)
            if (on_planes(*b) && b->plane_chunk == b->count && !b->cols_wait &&
                (rc = planes.add(planes_of(*b, 0, b->count, false), planes_wgs(*b, b->count))))
              return rc;
        if ((rc = planes.flush())) return rc;
      }
      // T = Lbar G, then P = T Rbar with partial sums of squares
      Batch<GemmX2Args> tall1(gemm_f16x2_kernel<256, 128, 1, X2_STORE_SPLIT>, 256, s), wide1(gemm_f16x2_kernel<128, 64, THREE ? 3 : 1, X2_STORE_SPLIT>, 256, s),
          tall2(gemm_f16x2_kernel<256, 128, 2, X2_STORE_NORM>, 256, s), wide2(gemm_f16x2_kernel<128, 64, THREE ? 3 : 2, X2_STORE_NORM>, 256, s);
      const bool fp32 = c.precond_matrix_cores == SHAMPOO_MATRIX_CORES_FP32;
      GemmBatch<EPI_STORE> first(fp32 ? gemm_kernels<ROW_CONTIG, ROW_CONTIG, float, GD, EPI_STORE, false, true>()
                                      : gemm_kernels<ROW_CONTIG, ROW_CONTIG, float, GD, EPI_STORE>(), s);
      GemmBatch<EPI_STORE_NORM> only(fp32 ? gemm_kernels<ROW_CONTIG, ROW_CONTIG, float, GD, EPI_STORE_NORM, false, true>()
                                          : gemm_kernels<ROW_CONTIG, ROW_CONTIG, float, GD, EPI_STORE_NORM>(), s),
          second(fp32 ? gemm_kernels<K_CONTIG, ROW_CONTIG, float, float, EPI_STORE_NORM, false, true>()
                      : gemm_kernels<K_CONTIG, ROW_CONTIG, float, float, EPI_STORE_NORM>(), s);
      auto x2_wgs = [](const GemmX2Args &g) { return (int64_t)g.tiles_m * g.tiles_n * g.batch; };
      // the last dimension of a tensor block, where a matrix product would be mostly padding
      auto narrow = [&](const Bucket &b) { return b.t3 && b.modes >= 3 && b.dlast() <= NARROW_MAX && !fp32; };
      int widest = 1;                      // one launch for all of them
      for (const Bucket *b : todo) if (narrow(*b)) widest = std::max(widest, (int)b->dlast());
      Batch<NarrowProductArgs> narrow_products(widest <= 4 ? product_narrow_kernel<1> : widest <= 8 ? product_narrow_kernel<2>
                                               : widest <= 12 ? product_narrow_kernel<3> : product_narrow_kernel<4>, 256, s);
      // a block of m x n times its left root, and the other way round
      auto left_product = [&](const Bucket &b, float *out, bool result) {
        GemmArgs g{};
        scale_direction(b, g, true, result);
        // (Lbar symmetric: A(i,k) read as Lbar[k][i], contiguous in i)
        g.a.base = ws + b.off_Linv; g.a.batch_stride = (int64_t)b.m * b.m; g.a.ld = b.m;
        g.b.from_table = 1; g.desc = reinterpret_cast<const BlockDesc *>(ws + b.off_desc); g.ptr_table = gd_tab;
        g.c = out; g.c_batch_stride = (int64_t)b.m * b.n; g.ldc = b.n;
        g.M = b.m; g.N = b.n; g.K = b.m; g.alpha = c1; g.beta = 0.f;
        g.batch = b.count;
        return g;
      };
      auto right_product = [&](const Bucket &b, const float *in, bool scaled) {
        GemmArgs h{};
        if (scaled) scale_direction(b, h, false, true);
        h.a.base = in; h.a.batch_stride = (int64_t)b.m * b.n; h.a.ld = b.n;
        h.b.base = ws + b.off_Rinv; h.b.batch_stride = (int64_t)b.n * b.n; h.b.ld = b.n;
        h.c = reinterpret_cast<float *>(ws + b.off_P); h.c_batch_stride = (int64_t)b.m * b.n; h.ldc = b.n;
        h.M = b.m; h.N = b.n; h.K = b.n; h.alpha = 1.f; h.beta = 0.f;
        h.batch = b.count;
        h.norm_partial = reinterpret_cast<float *>(ws + b.off_sshp);
        return h;
      };
      // Both products on the fp16 or bf16 matrix cores, float32-accurate through splits of the
      // float32 operands, each scaled by a power of two.  A bf16
      // gradient is one fp16 plane (exact: 8 significant bits), the scaled transpose made for the factor
      // update, against two of Lbar, T and Rbar; a float32 one (or a filtered or shifted one) is split into three bf16
      // planes, against three of the others.  B operands are read along k.  Tiles of 256 rows (half the operand traffic per
      // multiply; three planes do not leave room for them) unless padding the rows to 256 would add more than an eighth to the
      // work and unless there are too few of them to give every CU one.
      struct X2Shape { bool tall; int tm, tn; };
      auto x2_shape = [&](const Bucket &b) {
        const int tm128 = (b.m + 127) / 128, tn = (b.n + X2_TN - 1) / X2_TN, tm256 = (b.m + 255) / 256;
        const bool tall = !THREE && tm256 * 256 * 8 <= tm128 * 128 * 9 && (int64_t)tm256 * tn * b.count >= 256;
        return X2Shape{tall, tall ? tm256 : tm128, tn};
      };
      auto x2_args = [&](const Bucket &b, int b0, int cnt, GemmX2Args &g, GemmX2Args &h) {
        const X2Shape x = x2_shape(b);
        const int64_t mn = (int64_t)b.m * b.n, plane = cnt * mn;
        uint16_t *Tp = reinterpret_cast<uint16_t *>(bucket_t(b)) + (THREE ? 3 * plane : 0);
        g = GemmX2Args{};
        g.a_plane_stride = (int64_t)b.count * b.m * b.m; g.a_batch_stride = (int64_t)b.m * b.m; g.lda = b.m;
        g.a = reinterpret_cast<const uint16_t *>(ws + b.off_Linvp) + b0 * g.a_batch_stride;
        g.b = THREE ? reinterpret_cast<const uint16_t *>(bucket_t(b)) : reinterpret_cast<const uint16_t *>(ws + b.off_Gt);
        g.b_plane_stride = THREE ? plane : 0; g.b_batch_stride = mn; g.ldb = b.m;
        g.c2 = Tp; g.c2_plane_stride = plane; g.c_batch_stride = mn; g.ldc = b.n;
        g.M = b.m; g.N = b.n; g.K = b.m; g.alpha = c1; g.out_scale = reinterpret_cast<const float *>(ws + b.off_t_scale) + b0;
        g.tiles_m = x.tm; g.tiles_n = x.tn; g.batch = cnt;
        h = GemmX2Args{};
        h.a = Tp; h.a_plane_stride = plane; h.a_batch_stride = mn; h.lda = b.n;
        h.b_plane_stride = (int64_t)b.count * b.n * b.n; h.b_batch_stride = (int64_t)b.n * b.n; h.ldb = b.n;
        h.b = reinterpret_cast<const uint16_t *>(ws + b.off_Rinvp) + b0 * h.b_batch_stride;
        h.c = reinterpret_cast<float *>(ws + b.off_P) + b0 * mn; h.c_batch_stride = mn; h.ldc = b.n;
        h.M = b.m; h.N = b.n; h.K = b.n; h.alpha = 1.f; h.out_scale = reinterpret_cast<const float *>(ws + b.off_inv_ts) + b0;
        h.norm_partial = reinterpret_cast<float *>(ws + b.off_sshp) + (int64_t)b0 * x.tm * x.tn;
        h.tiles_m = x.tm; h.tiles_n = x.tn; h.batch = cnt;
      };
      {
        for (size_t i = 0; i < todo.size(); ++i) {
          const Bucket &b = *todo[i];
          float *T = bucket_t(b), *P = reinterpret_cast<float *>(ws + b.off_P), *ssh = reinterpret_cast<float *>(ws + b.off_sshp);
          if (on_planes(b)) {
            const X2Shape x = x2_shape(b);
            ssh_count[i] = x.tm * x.tn;
            if (THREE && b.plane_chunk < b.count) continue;      // below
            GemmX2Args g, h;
            x2_args(b, 0, b.count, g, h);
            if ((rc = (x.tall ? tall1 : wide1).add(g, x2_wgs(g))) || (rc = (x.tall ? tall2 : wide2).add(h, x2_wgs(h)))) return rc;
          } else if (b.t3) {
            // P = G x_1 Lbar_1 x_2 Lbar_2 ... x_w Lbar_w (Sec. 2.3), the first product here
            GemmArgs g = left_product(b, b.modes == 1 ? P : T, b.modes == 1);
            if (b.modes == 1) { g.norm_partial = ssh; only.add(g, &ssh_count[i]); }
            else first.add(g);
          } else if (b.whole()) {
            // diagonal Shampoo: a diagonalised side scales rows / columns instead of multiplying
            DiagScaleArgs ds{};
            ds.desc = reinterpret_cast<const BlockDesc *>(ws + b.off_desc);  ds.g_table = gd_tab; ds.m = b.m; ds.n = b.n; ds.geom = b.geom;
            const float *dl = reinterpret_cast<const float *>(ws + b.off_Linv), *dr = reinterpret_cast<const float *>(ws + b.off_Rinv);
            const unsigned ew_grid = (unsigned)b.geom.chunks * b.count;
            if (b.diagL && b.diagR) {
              ds.dl = dl; ds.dr = dr; ds.out = P; ds.norm_partial = ssh; ds.alpha = c1;
              hipLaunchKernelGGL(diag_scale_kernel<GD>, dim3(ew_grid), dim3(EW_THREADS), 0, s, ds);
              HIP_TRY(hipGetLastError());
              ssh_count[i] = b.geom.chunks;
            } else if (b.diagL) {
              // T = D_L G, then P = T Rbar with per-tile sums of squares
              ds.dl = dl; ds.out = T; ds.alpha = c1;
              hipLaunchKernelGGL(diag_scale_kernel<GD>, dim3(ew_grid), dim3(EW_THREADS), 0, s, ds);
              HIP_TRY(hipGetLastError());
              second.add(right_product(b, T, false), &ssh_count[i]);
            } else {
              // T = Lbar G, then P = T D_R
              first.add(left_product(b, T, true));
              if ((rc = first.flush())) return rc;
              ds.src = T; ds.dr = dr; ds.out = P; ds.norm_partial = ssh; ds.alpha = 1.f;
              hipLaunchKernelGGL(diag_scale_kernel<float>, dim3(ew_grid), dim3(EW_THREADS), 0, s, ds);
              HIP_TRY(hipGetLastError());
              ssh_count[i] = b.geom.chunks;
            }
          } else {
            first.add(left_product(b, T, false));
            second.add(right_product(b, T, true), &ssh_count[i]);
          }
        }
        if ((rc = tall1.flush()) || (rc = wide1.flush()) || (rc = first.flush()) || (rc = only.flush())) return rc;
        // A middle mode k of a tensor block, seen as pre x d_k x post: its first two
        // indices are swapped, the product is the plain one on d_k x (pre post), and they are
        // swapped back; then the last mode on the block as (N / d_w) x d_w.
        std::vector<int> swapped(todo.size(), 0);       // the block is in the second scratch
        for (int mid = 0; mid < 2; ++mid) {
          Batch<PermuteArgs> there(permute_12_kernel<float>, 256, s), back(permute_12_kernel<float>, 256, s);
          GemmBatch<EPI_STORE> products(fp32 ? gemm_kernels<ROW_CONTIG, ROW_CONTIG, float, float, EPI_STORE, false, true>()
                                             : gemm_kernels<ROW_CONTIG, ROW_CONTIG, float, float, EPI_STORE>(), s);
          for (size_t i = 0; i < todo.size(); ++i) {
            const Bucket &b = *todo[i];
            if (!b.t3 || mid + 2 >= b.modes) continue;
            float *cur = bucket_t(b), *other = reinterpret_cast<float *>(ws + o->off_T2 + b.off_t2);
            if (swapped[i]) std::swap(cur, other);
            const int64_t mn = (int64_t)b.m * b.n;
            const int pre = mid == 0 ? b.m : b.m * b.td[1], dk = b.td[mid + 1], post = (int)(mn / ((int64_t)pre * dk));
            PermuteArgs pm{};
            pm.src = cur; pm.dst = other; pm.d1 = pre; pm.d2 = dk; pm.d3 = post; pm.blocks = b.count;
            permute_shape(pm, tensor_chunks(b));
            if ((rc = there.add(pm, (int64_t)pm.chunks * b.count))) return rc;
            GemmArgs h{};
            h.a.base = ws + b.off_midinv[mid]; h.a.batch_stride = (int64_t)dk * dk; h.a.ld = dk;
            h.b.base = other; h.b.batch_stride = mn; h.b.ld = pre * post;
            h.c = cur; h.c_batch_stride = mn; h.ldc = pre * post;
            h.M = dk; h.N = pre * post; h.K = dk; h.alpha = 1.f; h.beta = 0.f;
            h.batch = b.count;
            products.add(h);
            if (narrow(b) && mid + 3 == b.modes) continue;      // the last product swaps back
            pm.d1 = dk; pm.d2 = pre;
            permute_shape(pm, tensor_chunks(b));
            if ((rc = back.add(pm, (int64_t)pm.chunks * b.count))) return rc;
            swapped[i] ^= 1;
          }
          if ((rc = there.flush()) || (rc = products.flush()) || (rc = back.flush())) return rc;
        }
        for (size_t i = 0; i < todo.size(); ++i) {
          const Bucket &b = *todo[i];
          if (!b.t3 || b.modes == 1) continue;
          const int dl = b.dlast();
          const int64_t mn = (int64_t)b.m * b.n;
          if (narrow(b)) {
            NarrowProductArgs na;
            na.src = swapped[i] ? reinterpret_cast<float *>(ws + o->off_T2 + b.off_t2) : bucket_t(b);
            na.root = reinterpret_cast<const float *>(ws + b.off_Rinv); na.dst = reinterpret_cast<float *>(ws + b.off_P);
            na.norm_partial = reinterpret_cast<float *>(ws + b.off_sshp);
            na.gmax = reinterpret_cast<const float *>(ws + b.off_gmax) + b.count;
            na.d = dl; na.d2 = b.td[b.modes - 2]; na.d1 = (int)(mn / dl / na.d2); na.blocks = b.count;
            na.tiles2 = (na.d2 + NARROW_T2 - 1) / NARROW_T2; na.tiles = ssh_count[i] = narrow_tiles(na.d1, na.d2);
            if ((rc = narrow_products.add(na, (int64_t)na.tiles * b.count))) return rc;
            continue;
          }
          GemmArgs q{};
          q.a.base = swapped[i] ? reinterpret_cast<float *>(ws + o->off_T2 + b.off_t2) : bucket_t(b); q.a.batch_stride = mn; q.a.ld = dl;
          q.b.base = ws + b.off_Rinv; q.b.batch_stride = (int64_t)dl * dl; q.b.ld = dl;
          q.c = reinterpret_cast<float *>(ws + b.off_P); q.c_batch_stride = mn; q.ldc = dl;
          q.M = (int)(mn / dl); q.N = dl; q.K = dl; q.alpha = 1.f; q.beta = 0.f;
          q.batch = b.count;
          q.norm_partial = reinterpret_cast<float *>(ws + b.off_sshp);
          scale_direction(b, q, false, true);
          second.add(q, &ssh_count[i]);
        }
      }
      timer.reset();
      {
        StageTimer t(o, SHAMPOO_STAGE_PRECOND2, s);
        if ((rc = tall2.flush()) || (rc = wide2.flush()) || (rc = second.flush()) || (rc = narrow_products.flush())) return rc;
      }
      // planes of more blocks than the scratch has room for: in passes
      if (THREE)
        for (Bucket *bp : todo) {
          const Bucket &b = *bp;
          if (!on_planes(b) || b.plane_chunk == b.count) continue;
          for (int b0 = 0; b0 < b.count; b0 += b.plane_chunk) {
            const int cnt = std::min(b.plane_chunk, b.count - b0);
            GemmX2Args g, h;
            x2_args(b, b0, cnt, g, h);
            {
              StageTimer t(o, SHAMPOO_STAGE_PRECOND, s);
              Batch<BlockPlanesArgs> planes(block_planes_kernel, 256, s);
              if ((rc = planes.add(planes_of(b, b0, cnt, false), planes_wgs(b, cnt))) || (rc = planes.flush())) return rc;
              if ((rc = wide1.add(g, x2_wgs(g))) || (rc = wide1.flush())) return rc;
            }
            StageTimer t(o, SHAMPOO_STAGE_PRECOND2, s);
            if ((rc = wide2.add(h, x2_wgs(h))) || (rc = wide2.flush())) return rc;
          }
        }
    }
    {
      StageTimer t(o, SHAMPOO_STAGE_UPDATE, s);
      Batch<ScaleArgs> scales(scale_kernel, 64, s);
      Batch<EwArgs> updates(update_kernel<GD>, EW_THREADS, s);
      for (size_t i = 0; i < todo.size(); ++i) {
        const Bucket &b = *todo[i];
        float *scale = reinterpret_cast<float *>(ws + b.off_scale);
        if (use_shampoo) {
          ScaleArgs sa;
          sa.sg_partial = reinterpret_cast<const float *>(ws + b.off_sgp); sa.sg_count = b.geom.chunks;
          sa.ssh_partial = reinterpret_cast<const float *>(ws + b.off_sshp); sa.ssh_count = ssh_count[i];
          sa.scale = scale; sa.norms = reinterpret_cast<float *>(ws + b.off_norms); sa.blocks = b.count;
          if ((rc = scales.add(sa, b.count))) return rc;
        }
        EwArgs e{};
        fill_ew(e, b);
        e.p = reinterpret_cast<float *>(ws + b.off_P); e.scale = scale;
        e.wd_decoupled = wd_dec; e.nesterov = c.use_nesterov ? 1 : 0;
        e.graft_only = use_shampoo ? 0 : 1;
        if ((rc = updates.add(e, (int64_t)b.geom.chunks * b.count))) return rc;
      }
      if ((rc = scales.flush()) || (rc = updates.flush())) return rc;
    }
  }
  if (o->has_tensor) {
    // the updated block-contiguous copies go back into the caller's tensors
    StageTimer t(o, SHAMPOO_STAGE_UPDATE, s);
    for (int i = 0; i < c.n_params; ++i) {
      if (p.pshape[i].kind != P_TENSOR) continue;
      add_copy(i, o->last_w[i], ws + o->off_Wb[i], 4, true);
    }
    send_copies(true);
    HIP_TRY(hipGetLastError());
  }
  if (!p.diag_chunks.empty() && !small_ok) {
    StageTimer t(o, SHAMPOO_STAGE_DIAG, s);
    hipLaunchKernelGGL(diag_kernel<GT>, dim3((unsigned)p.diag_chunks.size()), dim3(EW_THREADS), 0, s, d);
    HIP_TRY(hipGetLastError());
  }
  return helper.join();
}

}  // namespace

// ---------------------------------------------------------------------------
// extern "C" boundary
// ---------------------------------------------------------------------------
// No entry point throws: host memory that runs out is the only exception there is, and an error like a launch that fails.
extern "C" {

int shampoo_plan(const shampoo_config *cfg, int64_t *table, int64_t cap, int64_t *n_blocks, int64_t *n_buckets) try {
  const int rc = check_config(cfg);
  if (rc) return rc;
  if (cap < 0 || (cap > 0 && !table)) return SHAMPOO_ERR_NULL;
  Plan p;
  make_plan(cfg, p);
  if (const int rp = check_plan(p)) return rp;
  if (n_blocks) *n_blocks = (int64_t)p.blocks.size();
  if (n_buckets) *n_buckets = (int64_t)p.buckets.size();
  const int64_t cnt = std::min<int64_t>(cap, (int64_t)p.blocks.size());
  for (int64_t i = 0; i < cnt; ++i) {
    const Block &b = p.blocks[i];
    int64_t *row = table + 12 * i;
    row[0] = b.param; row[1] = b.row0; row[2] = b.col0; row[3] = b.m; row[4] = b.n;
    row[5] = b.bucket; row[6] = b.slot;
    row[7] = (p.buckets[b.bucket].diagL ? 1 : 0) | (p.buckets[b.bucket].diagR ? 2 : 0) | (b.tensor ? 4 | (p.buckets[b.bucket].modes << 4) : 0);
    row[8] = b.s3; row[9] = b.d3; row[10] = b.s4; row[11] = b.d4;
  }
  return SHAMPOO_OK;
} catch (const std::exception &) {
  return SHAMPOO_ERR_HIP;
}

size_t shampoo_workspace_bytes(const shampoo_config *cfg) try {
  if (check_config(cfg)) return 0;
  Plan p;
  make_plan(cfg, p);
  if (check_plan(p)) return 0;
  return layout(cfg, p, nullptr);
} catch (const std::exception &) {
  return 0;
}

int shampoo_create(const shampoo_config *cfg, void *workspace, size_t workspace_bytes, void *stream,
                   shampoo_opt **out) try {
  if (!out) return SHAMPOO_ERR_NULL;
  *out = nullptr;
  int rc = check_config(cfg);
  if (rc) return rc;
  std::unique_ptr<shampoo_opt> own(new shampoo_opt());
  shampoo_opt *o = own.get();
  o->cfg = *cfg;
  o->ndim.assign(cfg->ndim, cfg->ndim + cfg->n_params);
  o->shape.assign(cfg->shape, cfg->shape + (size_t)SHAMPOO_MAX_NDIM * cfg->n_params);
  o->cfg.ndim = o->ndim.data();
  o->cfg.shape = o->shape.data();
  o->last_w.assign(cfg->n_params, nullptr);
  o->last_g.assign(cfg->n_params, nullptr);
  make_plan(&o->cfg, o->plan);
  if ((rc = check_plan(o->plan))) return rc;
  const size_t need = layout(&o->cfg, o->plan, o);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % ALIGN) != 0 || workspace_bytes < need)
    return SHAMPOO_ERR_WORKSPACE;
  o->ws = static_cast<unsigned char *>(workspace);
  o->ws_bytes = workspace_bytes;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (hipSetDevice(cfg->device) != hipSuccess) return SHAMPOO_ERR_HIP;
  Plan &p = o->plan;
  // state: A = M = 0, L = R = 0, roots = I
  if ((rc = launch_fill(reinterpret_cast<float *>(o->ws + o->off_A), 0.f, p.total_elems, s))) return rc;
  if (cfg->momentum > 0.f)
    if ((rc = launch_fill(reinterpret_cast<float *>(o->ws + o->off_M), 0.f, p.total_elems, s))) return rc;
  if ((rc = launch_fill(reinterpret_cast<float *>(o->ws + o->off_count), 0.f, 16, s))) return rc;
  if (o->use_b1)
    if ((rc = launch_fill(reinterpret_cast<float *>(o->ws + o->off_Gf), 0.f, p.total_elems, s))) return rc;
  {
    // pointer tables of the library-owned gradient buffers (same layout as A / M)
    std::vector<void *> t1(cfg->n_params), t2(cfg->n_params);
    for (int i = 0; i < cfg->n_params; ++i) {
      t1[i] = o->use_l2 ? reinterpret_cast<float *>(o->ws + o->off_G1) + p.param_state_offset[i] : nullptr;
      t2[i] = o->use_b1 ? reinterpret_cast<float *>(o->ws + o->off_Gf) + p.param_state_offset[i] : nullptr;
    }
    if (hipMemcpyAsync(o->ws + o->off_g1tab, t1.data(), t1.size() * sizeof(void *), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(o->ws + o->off_gftab, t2.data(), t2.size() * sizeof(void *), hipMemcpyHostToDevice, s) != hipSuccess)
      return SHAMPOO_ERR_HIP;
    if ((o->use_l2 || o->use_b1) && !p.prep_chunks.empty())
      if (hipMemcpyAsync(o->ws + o->off_prep, p.prep_chunks.data(), p.prep_chunks.size() * sizeof(DiagChunk),
                         hipMemcpyHostToDevice, s) != hipSuccess)
        return SHAMPOO_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return SHAMPOO_ERR_HIP;   // t1, t2 go out of scope
  }
  std::vector<std::vector<BlockDesc>> descs(p.buckets.size()), descs3(p.buckets.size());
  for (size_t i = 0; i < p.buckets.size(); ++i) {
    descs[i].resize(p.buckets[i].count);
    if (p.buckets[i].t3) descs3[i].resize((size_t)p.buckets[i].count * p.buckets[i].split3);
  }
  for (const Block &b : p.blocks) {
    BlockDesc d;
    d.param = b.param;
    if (b.tensor) {
      // a block of the block-contiguous copy, as a d1 x (d2 d3) matrix; the second descriptor
      // shows the same memory as the (d1 d2) x d3 matrix of the third dimension
      d.ld = b.n * b.d3 * b.d4;
      d.offset = b.voff;
      d.state_offset = p.param_state_offset[b.param] + d.offset;
      // (one entry per row range of the split Gram product, see split3)
      const int sp = p.buckets[b.bucket].split3;
      for (int k = 0; k < sp; ++k) {
        BlockDesc d3 = d;
        d3.ld = p.buckets[b.bucket].dlast();
        d3.offset = b.voff + (int64_t)k * (b.m / sp) * d.ld;
        descs3[b.bucket][(size_t)b.slot * sp + k] = d3;
      }
    } else {
      d.ld = (int32_t)p.pshape[b.param].cols;
      d.offset = b.row0 * d.ld + b.col0;
      d.state_offset = p.param_state_offset[b.param] + d.offset;
    }
    descs[b.bucket][b.slot] = d;
  }
  for (size_t i = 0; i < p.buckets.size(); ++i) {
    Bucket &b = p.buckets[i];
    const int64_t B = b.count;
    if ((rc = launch_fill(reinterpret_cast<float *>(o->ws + b.off_L), 0.f, B * (int64_t)b.l_elems(), s))) return rc;
    if ((rc = launch_fill(reinterpret_cast<float *>(o->ws + b.off_R), 0.f, B * (int64_t)b.r_elems(), s))) return rc;
    if ((rc = launch_fill(reinterpret_cast<float *>(o->ws + b.off_P), 0.f, B * b.m * b.n, s))) return rc;
    if ((rc = launch_fill(reinterpret_cast<float *>(o->ws + b.off_norms), 0.f, B * 2, s))) return rc;
    if ((rc = launch_fill(reinterpret_cast<float *>(o->ws + b.off_gmax), 0.f, B * 2, s))) return rc;
    if (b.t3) {
      for (int k = 0; k + 2 < b.modes; ++k) {
        const int64_t t2 = B * b.td[k + 1] * b.td[k + 1];
        if ((rc = launch_fill(reinterpret_cast<float *>(o->ws + b.off_mid[k]), 0.f, t2, s))) return rc;
        hipLaunchKernelGGL(eye_kernel, dim3((unsigned)((t2 + 255) / 256)), dim3(256), 0, s,
                           reinterpret_cast<float *>(o->ws + b.off_midinv[k]), b.td[k + 1], t2);
      }
      if (hipMemcpyAsync(o->ws + b.off_desc3, descs3[i].data(), descs3[i].size() * sizeof(BlockDesc),
                         hipMemcpyHostToDevice, s) != hipSuccess)
        return SHAMPOO_ERR_HIP;
    }
    // roots start as the identity (a diagonalised side: the vector of ones)
    const int64_t tl = B * b.m * b.m, tr = B * (int64_t)b.rdim() * b.rdim();
    if (b.diagL) { if ((rc = launch_fill(reinterpret_cast<float *>(o->ws + b.off_Linv), 1.f, B * b.m, s))) return rc; }
    else hipLaunchKernelGGL(eye_kernel, dim3((unsigned)((tl + 255) / 256)), dim3(256), 0, s,
                            reinterpret_cast<float *>(o->ws + b.off_Linv), b.m, tl);
    if (b.diagR) { if ((rc = launch_fill(reinterpret_cast<float *>(o->ws + b.off_Rinv), 1.f, B * b.n, s))) return rc; }
    else hipLaunchKernelGGL(eye_kernel, dim3((unsigned)((tr + 255) / 256)), dim3(256), 0, s,
                            reinterpret_cast<float *>(o->ws + b.off_Rinv), b.rdim(), tr);
    if (hipGetLastError() != hipSuccess) return SHAMPOO_ERR_HIP;
    if (hipMemcpyAsync(o->ws + b.off_desc, descs[i].data(), descs[i].size() * sizeof(BlockDesc),
                       hipMemcpyHostToDevice, s) != hipSuccess)
      return SHAMPOO_ERR_HIP;
  }
  if ((rc = split_roots(o, s))) return rc;
  if (o->n_small > 0) {
    // largest blocks first, so that the tail of the launch is made of the cheapest workgroups
    std::vector<SmallBlock> small;
    std::vector<char> only_small(cfg->n_params, 1);
    for (const Block &b : p.blocks) if (!p.buckets[b.bucket].small()) only_small[b.param] = 0;
    for (size_t i = 0; i < p.buckets.size(); ++i) {
      const Bucket &b = p.buckets[i];
      if (!b.small()) continue;
      for (int64_t k = 0; k < b.count; ++k) {
        SmallBlock sb;
        sb.d = descs[i][k]; sb.m = b.m; sb.n = b.n; sb.filter = only_small[sb.d.param];
        sb.off_L = (int64_t)(b.off_L + (size_t)k * b.m * b.m * 4); sb.off_R = (int64_t)(b.off_R + (size_t)k * b.n * b.n * 4);
        sb.off_Linv = (int64_t)(b.off_Linv + (size_t)k * b.m * b.m * 4);
        sb.off_Rinv = (int64_t)(b.off_Rinv + (size_t)k * b.n * b.n * 4);
        sb.off_P = (int64_t)(b.off_P + (size_t)k * b.m * b.n * 4); sb.off_norms = (int64_t)(b.off_norms + (size_t)k * 8);
        small.push_back(sb);
      }
    }
    std::stable_sort(small.begin(), small.end(), [](const SmallBlock &x, const SmallBlock &y) {
      return (int64_t)x.m * x.n > (int64_t)y.m * y.n;
    });
    if (hipMemcpy(o->ws + o->off_small, small.data(), small.size() * sizeof(SmallBlock), hipMemcpyHostToDevice) != hipSuccess)
      return SHAMPOO_ERR_HIP;
  }
  if (!p.diag_chunks.empty())
    if (hipMemcpyAsync(o->ws + o->off_diag, p.diag_chunks.data(), p.diag_chunks.size() * sizeof(DiagChunk),
                       hipMemcpyHostToDevice, s) != hipSuccess)
      return SHAMPOO_ERR_HIP;
  if (hipStreamSynchronize(s) != hipSuccess) return SHAMPOO_ERR_HIP;
  // Helper streams now and not by the first step that wants them: a millisecond there, and a step that is recorded first would stay
  // without them in every replay.
  int64_t staged = 0;
  bool large = false;
  for (const Bucket &b : p.buckets) {
    if (!b.small()) staged += (int64_t)b.m * b.n * b.count;
    large = large || (!b.diagL && b.m > JAC_SMALL_MAX) || (!b.diagR && b.rdim() > JAC_SMALL_MAX) || (b.t3 && std::max(b.td[1], b.td[2]) > JAC_SMALL_MAX);
  }
  o->overlap = o->n_small > 0 && staged >= OVERLAP_STAGED;
  if (o->overlap || large) (void)o->aux.ready();
  *out = own.release();
  return SHAMPOO_OK;
} catch (const std::exception &) {
  return SHAMPOO_ERR_HIP;
}

int shampoo_step(shampoo_opt *o, void *const *params, const void *const *grads, float lr, int64_t step,
                 void *stream) try {
  if (!o || !params || !grads) return SHAMPOO_ERR_NULL;
  const int np = o->cfg.n_params;
  for (int i = 0; i < np; ++i)
    if (!params[i] || !grads[i]) return SHAMPOO_ERR_NULL;
  if (step < 0 || step <= o->last_step) return SHAMPOO_ERR_STEP;
  if (!std::isfinite(lr)) return SHAMPOO_ERR_HYPER;
  hipStream_t s = static_cast<hipStream_t>(stream);
  HIP_TRY(hipSetDevice(o->cfg.device));
  // pointer tables: re-sent only when they have changed, by the first step that reads them
  const size_t tab_bytes = (size_t)np * sizeof(void *);
  const bool same = std::memcmp(o->last_w.data(), params, tab_bytes) == 0 && std::memcmp(o->last_g.data(), grads, tab_bytes) == 0;
  if (!same) {
    std::memcpy(o->last_w.data(), params, tab_bytes);
    std::memcpy(o->last_g.data(), grads, tab_bytes);
    uintptr_t bits = 0;
    for (int i = 0; i < np; ++i) bits |= reinterpret_cast<uintptr_t>(grads[i]);
    o->ptrs_aligned16 = bits % 16 == 0;
    o->tables_stale = true;
  }
  int rc;
  if (o->cfg.grad_dtype == SHAMPOO_GRAD_BF16) {
    if (o->use_l2) rc = step_impl<uint16_t, float, float>(o, lr, step, s);
    else if (o->use_b1) rc = step_impl<uint16_t, uint16_t, float>(o, lr, step, s);
    else rc = step_impl<uint16_t, uint16_t, uint16_t>(o, lr, step, s);
  } else {
    rc = step_impl<float, float, float>(o, lr, step, s);
  }
  // A step whose launches failed (SHAMPOO_ERR_HIP) leaves the state partly updated; the step
  // counter then stays where it was, so the error is not masked by SHAMPOO_ERR_STEP on a retry.
  if (rc == SHAMPOO_OK) o->last_step = step;
  return rc;
} catch (const std::exception &) {
  return SHAMPOO_ERR_HIP;
}

int shampoo_get(shampoo_opt *o, int32_t param, int32_t block, int32_t which, void *dst, size_t bytes,
                void *stream) try {
  if (!o || !dst) return SHAMPOO_ERR_NULL;
  if (param < 0 || param >= o->cfg.n_params) return SHAMPOO_ERR_SHAPE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  HIP_TRY(hipSetDevice(o->cfg.device));
  Plan &p = o->plan;
  unsigned char *ws = o->ws;
  if (p.param_blocks[param].empty()) {   // 1-D, or a matrix on the diagonal-method path
    if (block != 0 || (which != SHAMPOO_GET_A && which != SHAMPOO_GET_M && which != SHAMPOO_GET_GF)) return SHAMPOO_ERR_SHAPE;
    if (which == SHAMPOO_GET_M && !(o->cfg.momentum > 0.f)) return SHAMPOO_ERR_SHAPE;
    if (which == SHAMPOO_GET_GF && !o->use_b1) return SHAMPOO_ERR_SHAPE;
    const size_t len = (size_t)p.pshape[param].elems();
    if (bytes != len * 4) return SHAMPOO_ERR_SHAPE;
    const size_t off_state = which == SHAMPOO_GET_A ? o->off_A : (which == SHAMPOO_GET_M ? o->off_M : o->off_Gf);
    const float *src = reinterpret_cast<const float *>(ws + off_state) + p.param_state_offset[param];
    HIP_TRY(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, s));
    return SHAMPOO_OK;
  }
  if (block < 0 || block >= (int32_t)p.param_blocks[param].size()) return SHAMPOO_ERR_SHAPE;
  const Block &b = p.blocks[p.param_blocks[param][block]];
  const Bucket &bk = p.buckets[b.bucket];
  const size_t m = b.m, n = b.n;
  const unsigned char *src = nullptr;
  size_t need = 0;
  switch (which) {
    case SHAMPOO_GET_L:
    case SHAMPOO_GET_R: {
      Batch<MirrorArgs> mirrors(mirror_upper_tiles_kernel, 256, s);
      // of this block alone: a program that reads all factors asks for one after the other
      int rcf = complete_factor(o, (size_t)b.bucket, which == SHAMPOO_GET_L ? 0 : 1, b.slot, 1, o->half_stale[b.bucket], mirrors);
      if (rcf || (rcf = mirrors.flush())) return rcf;
      need = (which == SHAMPOO_GET_L ? bk.l_elems() : bk.r_elems()) * 4;
      src = ws + (which == SHAMPOO_GET_L ? bk.off_L : bk.off_R) + (size_t)b.slot * need;
      break;
    }
    case SHAMPOO_GET_LINV: need = bk.l_elems() * 4; src = ws + bk.off_Linv + (size_t)b.slot * need; break;
    case SHAMPOO_GET_RINV: need = bk.r_elems() * 4; src = ws + bk.off_Rinv + (size_t)b.slot * need; break;
    case SHAMPOO_GET_L2:
    case SHAMPOO_GET_L2INV:
    case SHAMPOO_GET_L3:
    case SHAMPOO_GET_L3INV: {
      const int k = (which == SHAMPOO_GET_L2 || which == SHAMPOO_GET_L2INV) ? 0 : 1;
      if (!bk.t3 || k + 2 >= bk.modes) return SHAMPOO_ERR_SHAPE;
      need = (size_t)bk.td[k + 1] * bk.td[k + 1] * 4;
      src = ws + ((which == SHAMPOO_GET_L2 || which == SHAMPOO_GET_L3) ? bk.off_mid[k] : bk.off_midinv[k]) + (size_t)b.slot * need;
      break;
    }
    case SHAMPOO_GET_PSH: need = m * n * (size_t)b.d3 * b.d4 * 4; src = ws + bk.off_P + (size_t)b.slot * need; break;
    case SHAMPOO_GET_NORMS: src = ws + bk.off_norms + (size_t)b.slot * 8; need = 8; break;
    case SHAMPOO_GET_A:
    case SHAMPOO_GET_M:
    case SHAMPOO_GET_GF: {
      if (which == SHAMPOO_GET_M && !(o->cfg.momentum > 0.f)) return SHAMPOO_ERR_SHAPE;
      if (which == SHAMPOO_GET_GF && !o->use_b1) return SHAMPOO_ERR_SHAPE;
      const size_t off_state = which == SHAMPOO_GET_A ? o->off_A : (which == SHAMPOO_GET_M ? o->off_M : o->off_Gf);
      if (b.tensor) {   // state of a tensor parameter is kept block-contiguous
        const size_t need_t = m * n * (size_t)b.d3 * b.d4 * 4;
        if (bytes != need_t) return SHAMPOO_ERR_SHAPE;
        const float *base_t = reinterpret_cast<const float *>(ws + off_state) + p.param_state_offset[param] + b.voff;
        HIP_TRY(hipMemcpyAsync(dst, base_t, need_t, hipMemcpyDeviceToDevice, s));
        return SHAMPOO_OK;
      }
      if (bytes != m * n * 4) return SHAMPOO_ERR_SHAPE;
      const int64_t ld = p.pshape[param].cols;
      const float *base = reinterpret_cast<const float *>(ws + off_state) +
                          p.param_state_offset[param] + b.row0 * ld + b.col0;
      HIP_TRY(hipMemcpy2DAsync(dst, n * 4, base, (size_t)ld * 4, n * 4, m, hipMemcpyDeviceToDevice, s));
      return SHAMPOO_OK;
    }
    default: return SHAMPOO_ERR_SHAPE;
  }
  if (bytes != need) return SHAMPOO_ERR_SHAPE;
  HIP_TRY(hipMemcpyAsync(dst, src, need, hipMemcpyDeviceToDevice, s));
  return SHAMPOO_OK;
} catch (const std::exception &) {
  return SHAMPOO_ERR_HIP;
}

int shampoo_status(shampoo_opt *o, void *stream, int64_t *n_refreshes, int64_t *n_failed_roots) {
  if (!o) return SHAMPOO_ERR_NULL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  HIP_TRY(hipSetDevice(o->cfg.device));
  unsigned long long cnt = 0;
  HIP_TRY(hipMemcpyAsync(&cnt, o->ws + o->off_count, sizeof(cnt), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  if (n_refreshes) *n_refreshes = o->n_refresh;
  if (n_failed_roots) *n_failed_roots = (int64_t)cnt;
  return SHAMPOO_OK;
}

int shampoo_set_timing(shampoo_opt *o, int32_t enable) {
  if (!o) return SHAMPOO_ERR_NULL;
  o->timing = enable != 0;
  return SHAMPOO_OK;
}

int shampoo_get_timing(shampoo_opt *o, int32_t stage, double *ms_total, int64_t *intervals) {
  if (!o || !ms_total || !intervals) return SHAMPOO_ERR_NULL;
  if (stage < 0 || stage >= SHAMPOO_STAGE_COUNT) return SHAMPOO_ERR_SHAPE;
  double total = 0.0;
  int64_t cnt = 0;
  int rc = SHAMPOO_OK;
  for (auto &iv : o->intervals[stage]) {
    float ms = 0.f;
    if (hipEventSynchronize(iv.b) != hipSuccess || hipEventElapsedTime(&ms, iv.a, iv.b) != hipSuccess)
      rc = SHAMPOO_ERR_HIP;
    else { total += ms; ++cnt; }
    (void)hipEventDestroy(iv.a);
    (void)hipEventDestroy(iv.b);
  }
  o->intervals[stage].clear();
  *ms_total = total;
  *intervals = cnt;
  return rc;
}

int shampoo_destroy(shampoo_opt *o) {
  if (!o) return SHAMPOO_ERR_NULL;
  for (auto &v : o->intervals)
    for (auto &iv : v) { (void)hipEventDestroy(iv.a); (void)hipEventDestroy(iv.b); }
  if (o->aux.state == 1) { (void)hipSetDevice(o->cfg.device); o->aux.release(); }
  delete o;
  return SHAMPOO_OK;
}

size_t shampoo_root_inverse_workspace_bytes(int32_t n, int32_t batch) {
  if (n < 1 || batch < 1 || n > MAX_BLOCK_SIZE) return 0;
  return eig_layout(n, batch, true).bytes;   // for every exponent, and whether eigenvalues are asked for or not
}

int shampoo_root_inverse(const float *a, int32_t n, int32_t batch, float epsilon, float r, float *x,
                         float *lambda, int32_t *failed, void *workspace, size_t workspace_bytes, void *stream) try {
  if (!a || !x) return SHAMPOO_ERR_NULL;
  if (n < 1 || batch < 1) return SHAMPOO_ERR_SHAPE;
  if (n > MAX_BLOCK_SIZE) return SHAMPOO_ERR_UNSUPPORTED;
  if (!(epsilon > 0.f) || !std::isfinite(epsilon) || !(r > 0.f) || !std::isfinite(r)) return SHAMPOO_ERR_HYPER;
  const EigLayout e = eig_layout(n, batch, !lambda && band_serves(n, r));
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % ALIGN) != 0 || workspace_bytes < e.bytes)
    return SHAMPOO_ERR_WORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (failed) {
    const int rc = launch_fill(reinterpret_cast<float *>(failed), 0.f, batch, s);
    if (rc) return rc;
  }
  // The helper streams of the stand-alone call are shared by every caller of a device: the
  // lock keeps one call's fork / join events together while its work is enqueued.
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= MAX_DEVICES || n <= JAC_SMALL_MAX)
    return root_inverse_batched(a, n, batch, epsilon, r, 1.f, x, lambda, failed, nullptr,
                                static_cast<unsigned char *>(workspace), e, s, nullptr);
  std::lock_guard<std::mutex> lock(per_device[dev].mutex);
  return root_inverse_batched(a, n, batch, epsilon, r, 1.f, x, lambda, failed, nullptr,
                              static_cast<unsigned char *>(workspace), e, s, &per_device[dev].aux);
} catch (const std::exception &) {
  return SHAMPOO_ERR_HIP;
}

size_t shampoo_root_inverse_warm_workspace_bytes(int32_t n, int32_t batch) {
  if (n <= JAC_SMALL_MAX || batch < 1 || n > MAX_BLOCK_SIZE) return 0;
  return eig_layout(n, batch, false).bytes;
}

int shampoo_root_inverse_warm(const float *a, int32_t n, int32_t batch, float epsilon, float r, float *x,
                              float *lambda, int32_t *failed, float *qt, int32_t start, int32_t *sweeps,
                              void *workspace, size_t workspace_bytes, void *stream) try {
  if (!a || !x || !qt) return SHAMPOO_ERR_NULL;
  if (n < 1 || batch < 1) return SHAMPOO_ERR_SHAPE;
  if (n > MAX_BLOCK_SIZE || n <= JAC_SMALL_MAX) return SHAMPOO_ERR_UNSUPPORTED;
  if (!(epsilon > 0.f) || !std::isfinite(epsilon) || !(r > 0.f) || !std::isfinite(r)) return SHAMPOO_ERR_HYPER;
  const EigLayout e = eig_layout(n, batch, false);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % ALIGN) != 0 || workspace_bytes < e.bytes)
    return SHAMPOO_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(qt) % 16 != 0) return SHAMPOO_ERR_WORKSPACE;   // the kernels move it 16 bytes at a time
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (failed) {
    const int rc = launch_fill(reinterpret_cast<float *>(failed), 0.f, batch, s);
    if (rc) return rc;
  }
  WarmStart w;
  w.qt = qt; w.start = start != 0; w.sweeps = sweeps;
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= MAX_DEVICES)
    return root_inverse_batched(a, n, batch, epsilon, r, 1.f, x, lambda, failed, nullptr,
                                static_cast<unsigned char *>(workspace), e, s, nullptr, nullptr, w);
  std::lock_guard<std::mutex> lock(per_device[dev].mutex);
  return root_inverse_batched(a, n, batch, epsilon, r, 1.f, x, lambda, failed, nullptr,
                              static_cast<unsigned char *>(workspace), e, s, &per_device[dev].aux, nullptr, w);
} catch (const std::exception &) {
  return SHAMPOO_ERR_HIP;
}

int shampoo_root_inverse_static(const float *a, int32_t n, int32_t batch, float epsilon, float r, float *x,
                                float *lambda, int32_t *failed, void *stream) try {
  if (!a || !x) return SHAMPOO_ERR_NULL;
  if (n < 1 || batch < 1) return SHAMPOO_ERR_SHAPE;
  if (n > SHAMPOO_STATIC_MAX_N) return SHAMPOO_ERR_UNSUPPORTED;
  if (!(epsilon > 0.f) || !std::isfinite(epsilon) || !(r > 0.f) || !std::isfinite(r)) return SHAMPOO_ERR_HYPER;
  const EigLayout e = eig_layout(n, batch, false, SHAMPOO_STATIC_SCRATCH_BYTES, SHAMPOO_STATIC_SCRATCH_BYTES);
  if (e.bytes == 0 || e.bytes > SHAMPOO_STATIC_SCRATCH_BYTES) return SHAMPOO_ERR_UNSUPPORTED;
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= MAX_DEVICES) return SHAMPOO_ERR_UNSUPPORTED;
  unsigned char *ws = nullptr;
  {
    // every GPU holds its own copy of the array at its own address: looked up once per device
    std::lock_guard<std::mutex> lock(per_device[dev].mutex);
    if (!per_device[dev].scratch) {
      void *ptr = nullptr;
      HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
      if (!ptr) return SHAMPOO_ERR_HIP;
      per_device[dev].scratch = static_cast<unsigned char *>(ptr);
    }
    ws = per_device[dev].scratch;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (failed) {
    const int rc = launch_fill(reinterpret_cast<float *>(failed), 0.f, batch, s);   // a fill kernel, not a memset node
    if (rc) return rc;
  }
  // everything on the caller's stream: no helper streams are created on this path
  return root_inverse_batched(a, n, batch, epsilon, r, 1.f, x, lambda, failed, nullptr, ws, e, s, nullptr);
} catch (const std::exception &) {
  return SHAMPOO_ERR_HIP;
}

size_t shampoo_root_inverse_newton_workspace_bytes(int32_t n, int32_t batch) {
  if (n < 1 || batch < 1 || n > MAX_BLOCK_SIZE) return 0;
  return newton_layout(n, batch).bytes;
}

int shampoo_root_inverse_newton(const float *a, int32_t n, int32_t batch, float epsilon, int32_t p, float tolerance,
                                int32_t max_iterations, float *x, int32_t *iterations, int32_t *failed,
                                void *workspace, size_t workspace_bytes, void *stream) try {
  if (!a || !x) return SHAMPOO_ERR_NULL;
  if (n < 1 || batch < 1) return SHAMPOO_ERR_SHAPE;
  if (n > MAX_BLOCK_SIZE || !newton_p_supported(p)) return SHAMPOO_ERR_UNSUPPORTED;
  if (!(epsilon >= 0.f) || !std::isfinite(epsilon) || !(tolerance > 0.f) || !std::isfinite(tolerance) ||
      max_iterations < 1 || max_iterations > 1000)
    return SHAMPOO_ERR_HYPER;
  const NewtonLayout e = newton_layout(n, batch);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % ALIGN) != 0 || workspace_bytes < e.bytes)
    return SHAMPOO_ERR_WORKSPACE;
  return newton_root_batched(a, n, batch, epsilon, p, 1.f, tolerance, max_iterations, x, iterations, failed, nullptr,
                             static_cast<unsigned char *>(workspace), e, static_cast<hipStream_t>(stream));
} catch (const std::exception &) {
  return SHAMPOO_ERR_HIP;
}

int shampoo_jacobi_pair(int32_t s, int32_t halves, int32_t round, int32_t k, int32_t *p, int32_t *q) {
  if (!p || !q) return SHAMPOO_ERR_NULL;
  if (s < 2 || (s & 1) || round < 0 || round >= s - 1 || k < 0 || k >= s / 2) return SHAMPOO_ERR_SHAPE;
  if (halves == 1 && (s < 4 || ((s / 2) & (s / 2 - 1)) != 0)) return SHAMPOO_ERR_SHAPE;
  if (halves == 2 && s % 4 != 0) return SHAMPOO_ERR_SHAPE;
  if (halves < 0 || halves > 2) return SHAMPOO_ERR_SHAPE;
  int pp, qq;
  if (halves == 2) grouped_pair(s, 2, round, k, pp, qq);
  else if (halves) halves_pair(s, round, k, pp, qq); else rr_pair(s, round, k, pp, qq);
  *p = pp; *q = qq;
  return SHAMPOO_OK;
}

const char *shampoo_strerror(int code) {
  switch (code) {
    case SHAMPOO_OK: return "success";
    case SHAMPOO_ERR_NULL: return "a required pointer is NULL";
    case SHAMPOO_ERR_SHAPE: return "bad shape, dimension count, block size, index or byte count";
    case SHAMPOO_ERR_HYPER: return "hyper-parameter out of range";
    case SHAMPOO_ERR_WORKSPACE: return "workspace NULL, misaligned or too small";
    case SHAMPOO_ERR_STEP: return "step must be non-negative and strictly increasing";
    case SHAMPOO_ERR_HIP: return "a HIP runtime call failed or host memory ran out";
    case SHAMPOO_ERR_UNSUPPORTED: return "size outside the supported range";
    default: return "unknown error code";
  }
}

}  // extern "C"
