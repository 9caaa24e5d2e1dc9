// FP64 HODLR matrix products, gradient assembly and refinement helpers.
//
// Matrix product (eq. "e:rank"): y_a = D_a x_a + sum_l U_a (V_b^T x_b) over
// the level-l ancestor-or-self a of each leaf and its sibling b.  The V^T x
// projections come from the level-pass product (per leaf tile, all R columns
// at once) followed by a pairwise tree sum; the apply kernel then forms
// [D_a | U(I_a, :)] [x_a ; G_a] on MFMA, G_a gathering each level's sibling
// projection.  A^T swaps U and V and transposes the leaf blocks.
//
// Gradients (dL/dA = -Lambda X^T restricted to D, U, V):
//   dD_a = -Lambda_a X_a^T,  dU(I_a, level l) = -Lambda_a (V_b^T X_b)^T,
//   dV(I_b, level l) = -X_b (U_a^T Lambda_a)^T.
#include "mfma.h"

#include <algorithm>

namespace hodlr {

constexpr int kMvThreads = 256;

__device__ __forceinline__ d4 mma64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// A operand row of lane li such that register t of the product holds row 4 lq + t:
// four consecutive rows of a lane's column
__device__ __forceinline__ int row4(int li) { return 4 * (li & 3) + (li >> 2); }

// Sums over the projection tree: node i of level l = nodes 2 i + node 2 i + 1 of
// level l + 1, blocks of `elems`.  One launch forms up to three levels: a thread
// takes one element of the 2^DEPTH blocks below one node and keeps the sums in
// between, so these are not read again and a tree of 10 levels takes 3 launches
// (one a level: 9; N = 131072, R = 240, one vector: 56 us, now 10; N = 524288, R = 704,
// 32 vectors: 225, now 132).
template <int DEPTH>
__global__ __launch_bounds__(256) void tree_sum_kernel(int l, int nblk, int64_t elems, double* __restrict__ tree) {
  const int64_t e = (int64_t)(blockIdx.x % nblk) * 256 + threadIdx.x;
  const int i = blockIdx.x / nblk;  // node of level l - DEPTH, from the blocks of level l
  if (e >= elems) return;
  double v[1 << DEPTH];
#pragma unroll
  for (int k = 0; k < 1 << DEPTH; ++k) v[k] = tree[(tree_slot(l, (i << DEPTH) + k)) * elems + e];
#pragma unroll
  for (int d = DEPTH - 1; d >= 0; --d) {
#pragma unroll
    for (int k = 0; k < 1 << d; ++k) {
      v[k] = v[2 * k] + v[2 * k + 1];
      tree[tree_slot(l - DEPTH + d, (i << d) + k) * elems + e] = v[k];
    }
  }
}

hipError_t launch_tree_sums(hipStream_t s, int L, int64_t elems, double* tree) {
  if (elems == 0) return hipSuccess;
  const int64_t nblk = (elems + 255) / 256;
  for (int l = L; l > 1;) {
    const int depth = std::min(l - 1, 3);
    const int64_t wgs = nblk << (l - depth);
    if (wgs > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)wgs);
    if (depth == 3)
      hipLaunchKernelGGL(tree_sum_kernel<3>, grid, dim3(256), 0, s, l, (int)nblk, elems, tree);
    else if (depth == 2)
      hipLaunchKernelGGL(tree_sum_kernel<2>, grid, dim3(256), 0, s, l, (int)nblk, elems, tree);
    else
      hipLaunchKernelGGL(tree_sum_kernel<1>, grid, dim3(256), 0, s, l, (int)nblk, elems, tree);
    l -= depth;
  }
  return hipGetLastError();
}

// y(leaf rows, chunk) = op(D_a) x_a + U(I_a, :) G_a     (op = identity or transpose)
// Bound by the latency of streaming D and U for few right-hand sides.  Waves
// stand WR x WK = 4 over 64-row blocks and groups of 16 K columns (WK = 1, 2, 4 for
// leaves above 128, up to 128 and up to 64 rows, so that every wave has rows);
// partial sums meet in LDS in a fixed order.  A lane holds K columns
// 4 lq + s of a group, contiguous in x, G and a transposed D.  Loads in flight come
// from the workgroups of a CU (4 to 6): with the next group's operands prefetched
// they were fewer and it was slower.  FULL: whole 64-row blocks; otherwise rows
// past the leaf re-read its last one (their results are not stored).
// N = 131072, leaf 128, R = 240, FP32 storage, one vector: 67 us, transposed 83
// (four row blocks for every leaf, element loads of a transposed D: 137 and
// 230); N = 2^20, leaf 256, FP64: 0.93 ms, 5.7 TB/s, as before.
template <typename S, int TRANS, int NCB, int WK, bool FULL>
__global__ __launch_bounds__(kMvThreads) void matvec_apply_kernel(
    const int64_t* __restrict__ leaf_off, int L, const int32_t* __restrict__ rpre, int R, const S* __restrict__ D,
    int64_t ldd, const S* __restrict__ Ua, int64_t lda, const double* __restrict__ X, int64_t ldx,
    const double* __restrict__ tree, double* __restrict__ Y, int64_t ldy, int nrhs, int zchunks) {
  constexpr int WR = 4 / WK;
  const int leaf = blockIdx.x / zchunks;
  const int zc = blockIdx.x % zchunks;
  const int64_t o = leaf_off[leaf];
  const int m = (int)(leaf_off[leaf + 1] - o);
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), kp = w / WR, wr0 = 64 * (w % WR);
  const int c0 = zc * 64;
  d4 acc[4][NCB];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) acc[rb][cb] = d4{0, 0, 0, 0};

  // the K columns: the leaf block (l = 0, rows of x), then every level (the
  // sibling's projections V^T x), in groups of 16
  int l = 0, k0 = 0, kend = m;
  const S* Ap = D + o;
  int64_t ldA = ldd, ldB = ldx;
  const double* Bp = X + o;
  auto advance = [&](int steps) {
    for (; steps > 0 && l <= L; --steps) {
      k0 += 16;
      while (l <= L && k0 >= kend) {
        if (++l > L) break;
        const int cl0 = rpre[l - 1];
        k0 = 0;
        kend = rpre[l] - cl0;
        Ap = Ua + o + (int64_t)cl0 * lda;
        ldA = lda;
        Bp = tree + tree_slot(l, (leaf >> (L - l)) ^ 1) * R * nrhs + cl0;
        ldB = R;
      }
    }
  };
  auto load = [&](double (&av)[4][4], double (&bv)[NCB][4]) {
    const bool tr = TRANS && l == 0, whole = k0 + 16 <= kend;  // uniform
    const int kq = k0 + 4 * lq;
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
      const int row = wr0 + 16 * rb + row4(li), rc = FULL ? row : min(row, m - 1);
      if (whole && tr) {
        load_run(Ap + kq + (int64_t)rc * ldA, av[rb]);
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int kc = whole ? kq + s : min(kq + s, kend - 1);
          const double v = tr ? (double)Ap[kc + (int64_t)rc * ldA] : (double)Ap[rc + (int64_t)kc * ldA];
          av[rb][s] = whole || kq + s < kend ? v : 0.0;
        }
      }
    }
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const double* col = Bp + (int64_t)min(c0 + 16 * cb + li, nrhs - 1) * ldB;
      if (whole) {
        load_run(col + kq, bv[cb]);
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const double v = col[min(kq + s, kend - 1)];
          bv[cb][s] = kq + s < kend ? v : 0.0;
        }
      }
    }
  };
  auto use = [&](const double (&av)[4][4], const double (&bv)[NCB][4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) acc[rb][cb] = mma64(av[rb][s], bv[cb][s], acc[rb][cb]);
  };
  if (wr0 < m) {
    advance(kp);
#pragma unroll 1
    while (l <= L) {
      double av[4][4], bv[NCB][4];
      load(av, bv);
      use(av, bv);
      advance(WK);
    }
  }
  if constexpr (WK > 1) {
    __shared__ double red[4 - WR][NCB][4][64];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
      if (rb > 0) __syncthreads();
      if (kp > 0) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
          for (int t = 0; t < 4; ++t) red[w - WR][cb][t][lane] = acc[rb][cb][t];
      }
      __syncthreads();
      if (kp == 0) {
#pragma unroll
        for (int u = 1; u < WK; ++u)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[rb][cb][t] += red[w + (u - 1) * WR][cb][t][lane];
      }
    }
    if (kp > 0) return;
  }
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int row = wr0 + 16 * rb + 4 * lq + t;
        const int col = c0 + 16 * cb + li;
        if (row < m && col < nrhs) Y[o + row + (int64_t)col * ldy] = acc[rb][cb][t];
      }
}

template <typename S>
hipError_t launch_matvec_apply(hipStream_t s, int trans, int nleaf, int L, const int64_t* d_leaf_off,
                               const int32_t* d_rpre, int R, const S* D, int64_t ldd, const S* Ua, int64_t lda,
                               const double* X, int64_t ldx, const double* tree, double* Y, int64_t ldy, int nrhs,
                               TileShape sh) {
  if (nleaf == 0 || nrhs == 0) return hipSuccess;
  if (sh.rows > 256) return hipErrorInvalidValue;
  const int zchunks = (nrhs + 63) / 64;
  dim3 grid((unsigned)(nleaf * zchunks));
#define HODLR_MV(TR, NC, WKV, FULLV)                                                                                \
  hipLaunchKernelGGL((matvec_apply_kernel<S, TR, NC, WKV, FULLV>), grid, dim3(kMvThreads), 0, s, d_leaf_off, L, d_rpre, \
                     R, D, ldd, Ua, lda, X, ldx, tree, Y, ldy, nrhs, zchunks)
  // chunks of 64 columns; up to 16 or 32 columns a narrower instance (one chunk, no padded MFMA columns)
#define HODLR_MVC(TR, WKV, FULLV)                                                                   \
  if (nrhs <= 16) HODLR_MV(TR, 1, WKV, FULLV); else if (nrhs <= 32) HODLR_MV(TR, 2, WKV, FULLV); else HODLR_MV(TR, 4, WKV, FULLV)
#define HODLR_MVW(TR)                                                                \
  if (sh.rows > 128) {                                                               \
    if (sh.mult(64)) { HODLR_MVC(TR, 1, true); } else { HODLR_MVC(TR, 1, false); }   \
  } else if (sh.rows > 64) {                                                         \
    if (sh.mult(64)) { HODLR_MVC(TR, 2, true); } else { HODLR_MVC(TR, 2, false); }   \
  } else {                                                                           \
    HODLR_MVC(TR, 4, false);                                                         \
  }
  if (trans) { HODLR_MVW(1) } else { HODLR_MVW(0) }
#undef HODLR_MVW
#undef HODLR_MVC
#undef HODLR_MV
  return hipGetLastError();
}
template hipError_t launch_matvec_apply<double>(hipStream_t, int, int, int, const int64_t*, const int32_t*, int,
                                                const double*, int64_t, const double*, int64_t, const double*,
                                                int64_t, const double*, double*, int64_t, int, TileShape);
template hipError_t launch_matvec_apply<float>(hipStream_t, int, int, int, const int64_t*, const int32_t*, int,
                                               const float*, int64_t, const float*, int64_t, const double*, int64_t,
                                               const double*, double*, int64_t, int, TileShape);

// ---------------------------------------------------------------------------
// gradients
// ---------------------------------------------------------------------------
// out(I_leaf, c) = [add(I_leaf, c) -] sum_k Left(I_leaf, k) B_c(k) with, per column c,
//   LEAF  B_c(k) = X(o + c, k), c < m: the outer products on the leaf block
//   GEN   B_c(k) = S(c, k) of the sibling of the leaf's ancestor at c's level, c < R;
//         tri = 1: over the columns k of the levels above c's level only
//   MIX   k over the columns of c's own level, B_c(k) = M(k, c), M the r x r matrix
//         of the leaf's ancestor there (Pd at pdoff[l] + node r^2; tri = 1: M^T)
// Bound by memory for few k (the written columns) and by MFMA for many.  Waves
// stand WR x WC = 4 over 64-row and 64-column blocks of the leaf's rows and a
// chunk of columns (WC = 1, 2, 4 for leaves above 128, up to 128 and up to 64
// rows); a wave past the leaf or the columns ends, its k range is that of
// its columns, and a lane stores 4 consecutive rows.  N = 131072, leaf 128,
// R = 240, FP32, one vector: GEN 35 us, LEAF 19 (four row blocks for every leaf and
// stores of single rows: 249 and 111); N = 32768, leaf 128, 192 columns, FP64: the two
// GEN (tri), LEAF and the two MIX of a gradient of log|det A| together 331 us
// (before, with an element-wise MIX: 1504).
enum LeftMode { kLeftLeaf, kLeftGen, kLeftMix };
struct LeftArgs {
  int ncols = 0;  // GEN and MIX: R
  int nk = 0;     // columns of Left
  int tri = 0;
  const double* B = nullptr;  // X, the tree or Pd
  int64_t ldb = 0;            // of X
  const int64_t* pdoff = nullptr;
};

template <typename S, int WC, int MODE>
__global__ __launch_bounds__(kMvThreads, 2) void left_product_kernel(const int64_t* __restrict__ leaf_off, int L,
                                                                     const int32_t* __restrict__ rpre, int nchunks,
                                                                     const double* __restrict__ Left, int64_t ldl,
                                                                     LeftArgs g, S* __restrict__ out, int64_t ldo,
                                                                     const double* __restrict__ add, int64_t ldadd) {
  constexpr int WR = 4 / WC;
  __shared__ int rs[HODLR_MAX_LEVELS + 1];
  const int leaf = blockIdx.x / nchunks, ch = blockIdx.x % nchunks;
  const int64_t o = leaf_off[leaf];
  const int m = (int)(leaf_off[leaf + 1] - o);
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr0 = 64 * (w % WR), c0 = 64 * (WC * ch + w / WR);
  const int ncols = MODE == kLeftLeaf ? m : g.ncols;
  if constexpr (MODE != kLeftLeaf) {
    if (tid <= L) rs[tid] = rpre[tid];
    __syncthreads();
  }
  if (wr0 >= m || c0 >= ncols) return;
  auto level = [&](int c) {  // of column c: 1 .. L
    int l = 1;
    for (int i = 1; i < L; ++i) l += c >= rs[i];
    return l;
  };
  // per column block: the lane's column of B, its stride and range of k
  const double* bp[4];
  int klo[4], khi[4], ks[4];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) {
    const int c = min(c0 + 16 * cb + li, ncols - 1);
    klo[cb] = 0;
    khi[cb] = g.nk;
    if constexpr (MODE == kLeftLeaf) {
      bp[cb] = g.B + o + c;
    } else {
      const int l = level(c), node = leaf >> (L - l);
      if constexpr (MODE == kLeftGen) {
        bp[cb] = g.B + tree_slot(l, node ^ 1) * ncols * g.nk + c;
        ks[cb] = ncols;
        if (g.tri) khi[cb] = min(g.nk, rs[l - 1]);
      } else {
        const int r0 = rs[l - 1], r = rs[l] - r0;
        klo[cb] = r0;
        khi[cb] = rs[l];
        ks[cb] = g.tri ? 1 : r;
        bp[cb] = g.B + g.pdoff[l] + (int64_t)node * r * r + (int64_t)(c - r0) * (g.tri ? r : 1);
      }
    }
  }
  // the wave's range of k: levels rise with c
  const int kbeg = MODE == kLeftMix ? rs[level(c0) - 1] & ~3 : 0;
  int kend = g.nk;
  if (MODE == kLeftMix) kend = rs[level(min(c0 + 63, ncols - 1))];
  if (MODE == kLeftGen && g.tri) kend = min(kend, rs[level(min(c0 + 63, ncols - 1)) - 1]);
  d4 acc[4][4];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) acc[rb][cb] = d4{0, 0, 0, 0};
  const double* Lw = Left + o + wr0;
  auto load = [&](int k0, double (&av)[4], double (&bv)[4]) {
    const int kk = k0 + lq, kc = min(kk, g.nk - 1);
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
      const double v = Lw[min(16 * rb + row4(li), m - 1 - wr0) + (int64_t)kc * ldl];
      av[rb] = kk < g.nk ? v : 0.0;
    }
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const bool in = kk >= klo[cb] && kk < khi[cb];
      bv[cb] = in ? bp[cb][(kk - klo[cb]) * (MODE == kLeftLeaf ? g.ldb : (int64_t)ks[cb])] : 0.0;
    }
  };
  double av[4], bv[4];
  if (kbeg < kend) load(kbeg, av, bv);
#pragma unroll 1
  for (int k0 = kbeg; k0 < kend; k0 += 4) {
    double an[4], bn[4];
    if (k0 + 4 < kend) load(k0 + 4, an, bn);
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) acc[rb][cb] = mma64(av[rb], bv[cb], acc[rb][cb]);
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      av[x] = an[x];
      bv[x] = bn[x];
    }
  }
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) {
    const int c = c0 + 16 * cb + li;
    if (c >= ncols) continue;
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
      const int row = wr0 + 16 * rb + 4 * lq;
      S* po = out + o + row + (int64_t)c * ldo;
      if (row + 4 <= m) {
        double base[4] = {0.0, 0.0, 0.0, 0.0};
        if (add) load_run(add + o + row + (int64_t)c * ldadd, base);
        typename Vec<S, 4>::type v;
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = (S)(MODE == kLeftMix ? acc[rb][cb][t] : base[t] - acc[rb][cb][t]);
        *reinterpret_cast<typename Vec<S, 4>::type*>(po) = v;
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (row + t < m) {
            const double base = add ? add[o + row + t + (int64_t)c * ldadd] : 0.0;
            po[t] = (S)(MODE == kLeftMix ? acc[rb][cb][t] : base - acc[rb][cb][t]);
          }
      }
    }
  }
}

template <typename S, int MODE>
static hipError_t launch_left(hipStream_t s, int nleaf, int m_max, int L, const int64_t* d_leaf_off,
                              const int32_t* d_rpre, const double* Left, int64_t ldl, const LeftArgs& g, int ncols,
                              S* out, int64_t ldo, const double* add, int64_t ldadd) {
  if (nleaf == 0 || ncols == 0) return hipSuccess;
  if (m_max > 256 || L > HODLR_MAX_LEVELS) return hipErrorInvalidValue;
#define HODLR_LEFT(WCV)                                                                                             \
  {                                                                                                                 \
    const int nchunks = (ncols + 64 * WCV - 1) / (64 * WCV);                                                        \
    hipLaunchKernelGGL((left_product_kernel<S, WCV, MODE>), dim3((unsigned)(nleaf * nchunks)), dim3(kMvThreads), 0, \
                       s, d_leaf_off, L, d_rpre, nchunks, Left, ldl, g, out, ldo, add, ldadd);                      \
  }
  if (m_max > 128) HODLR_LEFT(1)
  else if (m_max > 64) HODLR_LEFT(2)
  else HODLR_LEFT(4)
#undef HODLR_LEFT
  return hipGetLastError();
}

template <typename S>
hipError_t launch_grad_leaf(hipStream_t s, int nleaf, int m_max, const int64_t* d_leaf_off, int nrhs,
                            const double* X, int64_t ldx, const double* Lam, int64_t ldl, S* dD, int64_t ldd,
                            const double* add, int64_t ldadd) {
  LeftArgs g;
  g.nk = nrhs;
  g.B = X;
  g.ldb = ldx;
  return launch_left<S, kLeftLeaf>(s, nleaf, m_max, 0, d_leaf_off, nullptr, Lam, ldl, g, m_max, dD, ldd, add, ldadd);
}
template hipError_t launch_grad_leaf<double>(hipStream_t, int, int, const int64_t*, int, const double*, int64_t,
                                             const double*, int64_t, double*, int64_t, const double*, int64_t);
template hipError_t launch_grad_leaf<float>(hipStream_t, int, int, const int64_t*, int, const double*, int64_t,
                                            const double*, int64_t, float*, int64_t, const double*, int64_t);

template <typename S>
hipError_t launch_grad_gen(hipStream_t s, int nleaf, int m_max, int L, const int64_t* d_leaf_off, const int32_t* d_rpre,
                           int R, int nrhs, const double* Left, int64_t ldl, const double* tree, S* out, int64_t ldo,
                           const double* add, int64_t ldadd, int tri) {
  LeftArgs g;
  g.ncols = R;
  g.nk = nrhs;
  g.tri = tri;
  g.B = tree;
  return launch_left<S, kLeftGen>(s, nleaf, m_max, L, d_leaf_off, d_rpre, Left, ldl, g, R, out, ldo, add, ldadd);
}
template hipError_t launch_grad_gen<double>(hipStream_t, int, int, int, const int64_t*, const int32_t*, int, int,
                                            const double*, int64_t, const double*, double*, int64_t, const double*,
                                            int64_t, int);
template hipError_t launch_grad_gen<float>(hipStream_t, int, int, int, const int64_t*, const int32_t*, int, int,
                                           const double*, int64_t, const double*, float*, int64_t, const double*,
                                           int64_t, int);

hipError_t launch_node_mix(hipStream_t s, int64_t n, int nleaf, int m_max, int L, int R, const int64_t* d_leaf_off,
                           const int32_t* d_rpre, const int64_t* d_pdoff, const double* Pd, int trans,
                           const double* in, double* out) {
  LeftArgs g;
  g.ncols = g.nk = R;
  g.tri = trans;
  g.B = Pd;
  g.pdoff = d_pdoff;
  return launch_left<double, kLeftMix>(s, nleaf, m_max, L, d_leaf_off, d_rpre, in, n, g, R, out, n, nullptr, 0);
}

// ---------------------------------------------------------------------------
// refinement helpers (FP64)
// ---------------------------------------------------------------------------
constexpr int kNormBlocks = 256;

// per (block, column): partial sum of squares and max |.| over a strided row range
__global__ void colnorm_partial_kernel(int64_t n, const double* __restrict__ X, int64_t ldx, double* __restrict__ part) {
  __shared__ double s2[256], si[256];
  const int j = blockIdx.y;
  double a2 = 0.0, ai = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const double v = X[i + (int64_t)j * ldx];
    a2 += v * v;
    ai = fmax(ai, fabs(v));
  }
  s2[threadIdx.x] = a2;
  si[threadIdx.x] = ai;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) {
      s2[threadIdx.x] += s2[threadIdx.x + off];
      si[threadIdx.x] = fmax(si[threadIdx.x], si[threadIdx.x + off]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[((int64_t)j * gridDim.x + blockIdx.x) * 2] = s2[0];
    part[((int64_t)j * gridDim.x + blockIdx.x) * 2 + 1] = si[0];
  }
}
// one wave per column: its lanes load the partials (all in flight), then halve
// (a thread a column, walking them: a norm of 131072 rows took 33 us, now 11)
__global__ __launch_bounds__(64) void colnorm_final_kernel(int nblk, const double* __restrict__ part,
                                                           double* __restrict__ out2, double* __restrict__ outinf) {
  const int j = blockIdx.x;
  double a2 = 0.0, ai = 0.0;
  for (int b = threadIdx.x; b < nblk; b += 64) {
    a2 += part[((int64_t)j * nblk + b) * 2];
    ai = fmax(ai, part[((int64_t)j * nblk + b) * 2 + 1]);
  }
#pragma unroll
  for (int h = 32; h > 0; h >>= 1) {
    a2 += __shfl_down(a2, h);
    ai = fmax(ai, __shfl_down(ai, h));
  }
  if (threadIdx.x == 0) {
    out2[j] = sqrt(a2);
    outinf[j] = ai;
  }
}

hipError_t launch_colnorms(hipStream_t s, int64_t n, int nrhs, const double* X, int64_t ldx, double* part,
                           double* out2, double* outinf) {
  if (nrhs == 0) return hipSuccess;
  hipLaunchKernelGGL(colnorm_partial_kernel, dim3(kNormBlocks, nrhs), dim3(256), 0, s, n, X, ldx, part);
  hipLaunchKernelGGL(colnorm_final_kernel, dim3(nrhs), dim3(64), 0, s, kNormBlocks, part, out2, outinf);
  return hipGetLastError();
}

template <typename T>
__global__ void scale_down_kernel(int64_t n, const double* __restrict__ Rr, int64_t ldr,
                                  const double* __restrict__ sc, T* __restrict__ out, int64_t ldo) {
  const int j = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double d = sc[j] > 0.0 ? sc[j] : 1.0;
  out[i + (int64_t)j * ldo] = (T)(Rr[i + (int64_t)j * ldr] / d);
}
template <typename T>
hipError_t launch_scale_down(hipStream_t s, int64_t n, int nrhs, const double* Rr, int64_t ldr, const double* sc,
                             T* out, int64_t ldo) {
  if (nrhs == 0 || n == 0) return hipSuccess;
  hipLaunchKernelGGL(scale_down_kernel<T>, dim3((unsigned)((n + 255) / 256), nrhs), dim3(256), 0, s, n, Rr, ldr, sc,
                     out, ldo);
  return hipGetLastError();
}
template hipError_t launch_scale_down<double>(hipStream_t, int64_t, int, const double*, int64_t, const double*,
                                              double*, int64_t);
template hipError_t launch_scale_down<float>(hipStream_t, int64_t, int, const double*, int64_t, const double*, float*,
                                             int64_t);

template <typename T>
__global__ void axpy_up_kernel(int64_t n, const T* __restrict__ d, int64_t ldd, const double* __restrict__ sc,
                               double* __restrict__ X, int64_t ldx) {
  const int j = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double f = sc[j] > 0.0 ? sc[j] : 1.0;
  X[i + (int64_t)j * ldx] += (double)d[i + (int64_t)j * ldd] * f;
}
template <typename T>
hipError_t launch_axpy_up(hipStream_t s, int64_t n, int nrhs, const T* d, int64_t ldd, const double* sc, double* X,
                          int64_t ldx) {
  if (nrhs == 0 || n == 0) return hipSuccess;
  hipLaunchKernelGGL(axpy_up_kernel<T>, dim3((unsigned)((n + 255) / 256), nrhs), dim3(256), 0, s, n, d, ldd, sc, X,
                     ldx);
  return hipGetLastError();
}
template hipError_t launch_axpy_up<double>(hipStream_t, int64_t, int, const double*, int64_t, const double*, double*,
                                           int64_t);
template hipError_t launch_axpy_up<float>(hipStream_t, int64_t, int, const float*, int64_t, const double*, double*,
                                          int64_t);

// AX <- B - AX
__global__ void residual_kernel(int64_t n, const double* __restrict__ B, int64_t ldb, double* __restrict__ AX,
                                int64_t ldax) {
  const int j = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  AX[i + (int64_t)j * ldax] = B[i + (int64_t)j * ldb] - AX[i + (int64_t)j * ldax];
}
hipError_t launch_residual(hipStream_t s, int64_t n, int nrhs, const double* B, int64_t ldb, double* AX, int64_t ldax) {
  if (nrhs == 0 || n == 0) return hipSuccess;
  hipLaunchKernelGGL(residual_kernel, dim3((unsigned)((n + 255) / 256), nrhs), dim3(256), 0, s, n, B, ldb, AX, ldax);
  return hipGetLastError();
}

template <typename T, typename S>
__global__ void convert_kernel(int64_t rows, const S* __restrict__ in, int64_t ldi, int64_t gsi, T* __restrict__ out,
                               int64_t ldo) {
  const int j = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows) return;
  out[i + (int64_t)j * ldo] = (T)in[group_row(i, gsi) + (int64_t)j * ldi];
}
template <typename T, typename S>
hipError_t launch_convert(hipStream_t s, int64_t rows, int cols, const S* in, int64_t ldi, T* out, int64_t ldo,
                          int64_t gsi) {
  if (rows == 0 || cols == 0) return hipSuccess;
  hipLaunchKernelGGL((convert_kernel<T, S>), dim3((unsigned)((rows + 255) / 256), cols), dim3(256), 0, s, rows, in, ldi,
                     gsi, out, ldo);
  return hipGetLastError();
}
template hipError_t launch_convert<double, double>(hipStream_t, int64_t, int, const double*, int64_t, double*, int64_t, int64_t);
template hipError_t launch_convert<double, float>(hipStream_t, int64_t, int, const float*, int64_t, double*, int64_t, int64_t);
template hipError_t launch_convert<float, double>(hipStream_t, int64_t, int, const double*, int64_t, float*, int64_t, int64_t);

}  // namespace hodlr
