// HODLR construction from a kernel function (Section II-B; the entries of
// Section I "Kernel matrices" and of the Laplace double layer, Section IV-B
// eq. "e:laplace_int"): exact leaf blocks, and every sibling block
// A(I_a, I_b) compressed by cross approximation with partial pivoting taken
// for r_l steps (the approximate partial-pivoted LU that the experiments of
// Section IV-A use):
//   for k = 1 .. r:
//     v = A(i_k, :) - sum_{l<k} u_l(i_k) v_l,   j_k = argmax |v|,  v_k = v / v(j_k)
//     u_k = A(:, j_k) - sum_{l<k} v_l(j_k) u_l,  i_{k+1} = argmax over unused rows |u_k|
// with i_1 = the block's first row, the lowest index on ties, and an
// exhausted step (v(j_k) = 0) giving u_k = v_k = 0.  U_a = [u_k] goes to rows
// I_a, V_b = [v_k] to rows I_b of the level's columns of U_big / V_big.
//
// Blocks of up to kCbRows rows and columns and ranks up to kCbRank take all their
// steps in one workgroup (aca_block_kernel) where that pays (aca_own_launches).
// The others advance together: step k is one launch for the residual rows (a
// workgroup per 1024-column tile of a block, writing v unnormalized and the
// tile's largest modulus) and one for the residual columns (each workgroup first
// reduces its block's row partials to j_k and the pivot value, normalizes its
// tile of v, then forms its tile of u and the tile's largest modulus over unused
// rows); the next row launch reduces those to i_{k+1}.  Partials are reduced in a
// fixed order (deterministic).
#include "wave.h"

#include <algorithm>
#include <climits>

namespace hodlr {

namespace {

constexpr int kCsThreads = 256;
constexpr int kCsEpt = 4;
constexpr int kCsTile = kCsThreads * kCsEpt;  // elements of a block row / column per workgroup
constexpr double kPi = 3.141592653589793238462643383279502884;

// the entry of points p and q from |x_p - x_q|^2 (Gaussian, Matern)
__device__ __forceinline__ double radial_value(const ConstructKernel& k, double d2) {
  if (k.kind == HODLR_KERNEL_GAUSS) return exp(-d2 / (2.0 * (k.ell * k.ell)));
  const double s = sqrt(3.0) * sqrt(d2) / k.ell;
  return (1.0 + s) * exp(-s);
}
// Laplace double layer, w_q n_q . (x_p - x_q) / (2 pi |x_p - x_q|^2), from the
// two differences and the normal and weight of q.  The sum of two products is
// written out as the fused operation that is meant: left to the compiler, one
// kernel fused the first product and another the second, and an ulp decides the
// pivots of a block that has used up its numerical rank.
__device__ __forceinline__ double layer_value(double d2, double dx0, double dx1, double n0, double n1, double wq) {
  const double num = fma(n0, dx0, n1 * dx1);
  return num / (2.0 * kPi * d2) * wq;
}

__device__ __forceinline__ double kernel_offdiag(const ConstructKernel& k, int64_t p, int64_t q) {
  double d2 = 0.0, dx0 = 0.0, dx1 = 0.0;
  for (int d = 0; d < k.dim; ++d) {
    const double t = k.pts[p + d * k.ldp] - k.pts[q + d * k.ldp];
    d2 += t * t;
    if (d == 0) dx0 = t;
    if (d == 1) dx1 = t;
  }
  if (k.kind != HODLR_KERNEL_LAPLACE_DL) return radial_value(k, d2);
  return layer_value(d2, dx0, dx1, k.nrm[q], k.nrm[q + k.ldp], k.w[q]);
}

__device__ __forceinline__ double kernel_entry(const ConstructKernel& k, int64_t p, int64_t q) {
  if (p != q) return kernel_offdiag(k, p, q);
  const double d = k.kind == HODLR_KERNEL_LAPLACE_DL ? k.w[p] * k.kap[p] / (4.0 * kPi) : 1.0;
  return d + k.shift;
}

// (modulus, index) pairs: the larger modulus wins, the lower index on ties
__device__ __forceinline__ bool better(double a, int ia, double b, int ib) { return a > b || (a == b && ia < ib); }

// block-wide argmax of (a, idx, val) over kCsThreads threads; result in slot 0
__device__ __forceinline__ void block_argmax(double* sa, int* si, double* sv, int tid) {
  for (int s = kCsThreads / 2; s > 0; s >>= 1) {
    __syncthreads();
    if (tid < s && better(sa[tid + s], si[tid + s], sa[tid], si[tid])) {
      sa[tid] = sa[tid + s];
      si[tid] = si[tid + s];
      if (sv) sv[tid] = sv[tid + s];
    }
  }
  __syncthreads();
}

}  // namespace

// leaf blocks: D(s0 + p, q) = A(s0 + p, s0 + q) for q < m, zero for m <= q < m_max
template <typename TS>
__global__ __launch_bounds__(kCsThreads) void construct_leaves_kernel(ConstructKernel k, const int64_t* __restrict__ off,
                                                                      int m_max, int ccols, TS* D, int64_t ldd) {
  const int a = blockIdx.x;
  const int64_t s0 = off[a];
  const int m = (int)(off[a + 1] - s0);
  const int p = threadIdx.x;
  if (p >= m) return;
  const int q0 = blockIdx.y * ccols;
  const int q1 = min(m_max, q0 + ccols);
  for (int q = q0; q < q1; ++q) D[(s0 + p) + (int64_t)q * ldd] = q < m ? (TS)kernel_entry(k, s0 + p, s0 + q) : TS(0);
}

// step k, residual rows: v(j) = A(i_k, j) - sum_{l<k} U(i_k, l) V(j, l) for the tile's columns
__global__ __launch_bounds__(kCsThreads) void aca_row_kernel(ConstructKernel kd, const AcaBlock* __restrict__ blocks,
                                                             const AcaTile* __restrict__ tiles, int k, int kmax,
                                                             const double* __restrict__ U, int64_t ldu, double* V,
                                                             int64_t ldv, const double* __restrict__ cp_abs,
                                                             const int* __restrict__ cp_idx, double* __restrict__ rp_abs,
                                                             double* __restrict__ rp_val, int* __restrict__ rp_idx,
                                                             int* __restrict__ piv) {
  const AcaTile tl = tiles[blockIdx.x];
  const AcaBlock b = blocks[tl.blk];
  if (k >= b.rank) return;
  __shared__ double sa[kCsThreads], sv[kCsThreads];
  __shared__ int si[kCsThreads];
  __shared__ double uk[HODLR_MAX_RANK];
  const int tid = threadIdx.x;
  int i = 0;
  if (k > 0) {  // i_k from the previous step's column partials of this block
    double best = -2.0;
    int bi = INT_MAX;
    for (int t = tid; t < b.ntile; t += kCsThreads)
      if (better(cp_abs[b.tile0 + t], cp_idx[b.tile0 + t], best, bi)) {
        best = cp_abs[b.tile0 + t];
        bi = cp_idx[b.tile0 + t];
      }
    sa[tid] = best;
    si[tid] = bi;
    block_argmax(sa, si, nullptr, tid);
    i = si[0];
  }
  if (tl.t == 0 && tid == 0) piv[(int64_t)tl.blk * kmax + k] = i;
  if (tid < k) uk[tid] = U[(b.r0 + i) + (int64_t)(b.col + tid) * ldu];
  __syncthreads();
  double best = -1.0, bval = 0.0;
  int bj = INT_MAX;
  const int64_t p = b.r0 + i;
  // the thread's kCsEpt columns advance together through l (independent
  // loads in flight); each column's terms are still subtracted in order of l
  double v[kCsEpt];
  const double* Vb = V + b.c0 + (int64_t)b.col * ldv;
  const int j0 = tl.t * kCsTile + tid;
  if (j0 + (kCsEpt - 1) * kCsThreads < b.n) {  // full tile (uniform)
#pragma unroll
    for (int e = 0; e < kCsEpt; ++e) v[e] = kernel_offdiag(kd, p, b.c0 + j0 + e * kCsThreads);
    for (int l = 0; l < k; ++l) {
      const double c = uk[l];
      const double* Vl = Vb + (int64_t)l * ldv + j0;
#pragma unroll
      for (int e = 0; e < kCsEpt; ++e) v[e] -= c * Vl[e * kCsThreads];
    }
  } else {
#pragma unroll
    for (int e = 0; e < kCsEpt; ++e) {
      const int j = j0 + e * kCsThreads;
      v[e] = 0.0;
      if (j < b.n) {
        v[e] = kernel_offdiag(kd, p, b.c0 + j);
        for (int l = 0; l < k; ++l) v[e] -= uk[l] * Vb[j + (int64_t)l * ldv];
      }
    }
  }
#pragma unroll
  for (int e = 0; e < kCsEpt; ++e) {
    const int j = j0 + e * kCsThreads;
    if (j < b.n) {
      V[(b.c0 + j) + (int64_t)(b.col + k) * ldv] = v[e];
      const double av = fabs(v[e]);
      if (av > best) {  // j increases along e: the first of equal moduli stays
        best = av;
        bj = j;
        bval = v[e];
      }
    }
  }
  sa[tid] = best;
  si[tid] = bj;
  sv[tid] = bval;
  block_argmax(sa, si, sv, tid);
  if (tid == 0) {
    rp_abs[tl.gtile] = sa[0];
    rp_idx[tl.gtile] = si[0];
    rp_val[tl.gtile] = sv[0];
  }
}

// step k, residual columns: j_k and the pivot value from the row partials,
// v_k = v / v(j_k) on the tile's columns, u(i) = A(i, j_k) - sum_{l<k} V(j_k, l) U(i, l)
// on the tile's rows, and the tile's largest |u| over rows not yet pivots
__global__ __launch_bounds__(kCsThreads) void aca_col_kernel(ConstructKernel kd, const AcaBlock* __restrict__ blocks,
                                                             const AcaTile* __restrict__ tiles, int k, int kmax,
                                                             double* U, int64_t ldu, double* V, int64_t ldv,
                                                             const double* __restrict__ rp_abs,
                                                             const double* __restrict__ rp_val,
                                                             const int* __restrict__ rp_idx, double* __restrict__ cp_abs,
                                                             int* __restrict__ cp_idx, const int* __restrict__ piv) {
  const AcaTile tl = tiles[blockIdx.x];
  const AcaBlock b = blocks[tl.blk];
  if (k >= b.rank) return;
  __shared__ double sa[kCsThreads], sv[kCsThreads];
  __shared__ int si[kCsThreads];
  __shared__ double vk[HODLR_MAX_RANK];
  __shared__ unsigned char used[kCsTile];
  const int tid = threadIdx.x;
  {
    double best = -2.0, bval = 0.0;
    int bj = INT_MAX;
    for (int t = tid; t < b.ntile; t += kCsThreads)
      if (better(rp_abs[b.tile0 + t], rp_idx[b.tile0 + t], best, bj)) {
        best = rp_abs[b.tile0 + t];
        bj = rp_idx[b.tile0 + t];
        bval = rp_val[b.tile0 + t];
      }
    sa[tid] = best;
    si[tid] = bj;
    sv[tid] = bval;
    block_argmax(sa, si, sv, tid);
  }
  const int j = si[0];
  const double delta = sv[0];
  const bool exhausted = delta == 0.0;
  const int row0 = tl.t * kCsTile;
#pragma unroll
  for (int e = 0; e < kCsEpt; ++e) {
    const int jj = row0 + e * kCsThreads + tid;
    if (jj < b.n) {
      double* pv = V + (b.c0 + jj) + (int64_t)(b.col + k) * ldv;
      *pv = exhausted ? 0.0 : *pv / delta;
    }
  }
  if (tid < k && !exhausted) vk[tid] = V[(b.c0 + j) + (int64_t)(b.col + tid) * ldv];
  for (int x = tid; x < kCsTile; x += kCsThreads) used[x] = 0;
  __syncthreads();
  if (tid <= k) {
    const int rel = piv[(int64_t)tl.blk * kmax + tid] - row0;
    if (rel >= 0 && rel < kCsTile) used[rel] = 1;
  }
  __syncthreads();
  double best = -2.0;
  int bi = INT_MAX;
  double u[kCsEpt];
  const double* Ub = U + b.r0 + (int64_t)b.col * ldu;
  const int i0 = row0 + tid;
  if (exhausted) {
#pragma unroll
    for (int e = 0; e < kCsEpt; ++e) u[e] = 0.0;
  } else if (i0 + (kCsEpt - 1) * kCsThreads < b.m) {  // full tile (uniform)
#pragma unroll
    for (int e = 0; e < kCsEpt; ++e) u[e] = kernel_offdiag(kd, b.r0 + i0 + e * kCsThreads, b.c0 + j);
    for (int l = 0; l < k; ++l) {
      const double c = vk[l];
      const double* Ul = Ub + (int64_t)l * ldu + i0;
#pragma unroll
      for (int e = 0; e < kCsEpt; ++e) u[e] -= c * Ul[e * kCsThreads];
    }
  } else {
#pragma unroll
    for (int e = 0; e < kCsEpt; ++e) {
      const int ii = i0 + e * kCsThreads;
      u[e] = 0.0;
      if (ii < b.m) {
        u[e] = kernel_offdiag(kd, b.r0 + ii, b.c0 + j);
        for (int l = 0; l < k; ++l) u[e] -= vk[l] * Ub[ii + (int64_t)l * ldu];
      }
    }
  }
#pragma unroll
  for (int e = 0; e < kCsEpt; ++e) {
    const int ii = row0 + e * kCsThreads + tid;
    if (ii < b.m) {
      U[(b.r0 + ii) + (int64_t)(b.col + k) * ldu] = u[e];
      const double sc = used[ii - row0] ? -1.0 : fabs(u[e]);
      if (sc > best) {
        best = sc;
        bi = ii;
      }
    }
  }
  sa[tid] = best;
  si[tid] = bi;
  block_argmax(sa, si, nullptr, tid);
  if (tid == 0) {
    cp_abs[tl.gtile] = sa[0];
    cp_idx[tl.gtile] = si[0];
  }
}

// All steps of one block, one row and one column of it per thread: the generators
// stay in registers (2 x 32 doubles a thread), the points in LDS, and memory sees
// only the finished columns.  (The tiled steps read every earlier column again:
// 496 of them per generator at rank 32, and run at 4.2 TB/s.)  Each wave publishes
// its best candidate with its generator row, so a half step is one barrier;
// bound by that chain (entry, subtractions in order of l, search).  Entries,
// order of subtractions and choice of pivots are those of the tiled steps, and so
// are the results, to the bit.  N = 262144, leaf 128, rank 32: 0.22 ms a level
// (tiled 0.53); the whole construction 4.78 ms (tiled 5.85).  The limits: two
// generators of rank 32 take half of the registers at 512 threads.
constexpr int kCbRank = 32;
constexpr int kCbRows = 512;

template <int NT>
__global__ __launch_bounds__(NT, 2) void aca_block_kernel(ConstructKernel kd, const AcaBlock* __restrict__ blocks,
                                                          double* __restrict__ U, int64_t ldu,
                                                          double* __restrict__ V, int64_t ldv) {
  constexpr int NW = NT / 64;
  const AcaBlock b = blocks[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  __shared__ double rpt[3][NT], cpt[6][NT];                   // row points; column points, normals, weights
  __shared__ __align__(16) double hist[2][NW][kCbRank];       // per wave: its candidate's generator row
  __shared__ unsigned long long ckey[2][NW];                  // order of moduli (see below)
  __shared__ int cidx[2][NW];
  __shared__ double cval[2][NW];
  const bool isrow = tid < b.m, iscol = tid < b.n, dl = kd.kind == HODLR_KERNEL_LAPLACE_DL;
  for (int d = 0; d < kd.dim; ++d) {
    if (isrow) rpt[d][tid] = kd.pts[b.r0 + tid + d * kd.ldp];
    if (iscol) cpt[d][tid] = kd.pts[b.c0 + tid + d * kd.ldp];
  }
  if (dl && iscol) {
    cpt[3][tid] = kd.nrm[b.c0 + tid];
    cpt[4][tid] = kd.nrm[b.c0 + tid + kd.ldp];
    cpt[5][tid] = kd.w[b.c0 + tid];
  }
  __syncthreads();

  auto entry = [&](int i, int j) {
    double d2 = 0.0, dx0 = 0.0, dx1 = 0.0;
    for (int d = 0; d < kd.dim; ++d) {
      const double t = rpt[d][i] - cpt[d][j];
      d2 += t * t;
      if (d == 0) dx0 = t;
      if (d == 1) dx1 = t;
    }
    if (!dl) return radial_value(kd, d2);
    return layer_value(d2, dx0, dx1, cpt[3][j], cpt[4][j], cpt[5][j]);
  };
  // x - sum_{l<k} c_l g_l in order of l (both are zero from l = k on)
  auto residual = [&](double x, const double* c, const double (&g)[kCbRank], int k) {
#pragma unroll
    for (int l0 = 0; l0 < kCbRank; l0 += 8)
      if (l0 < k) {
#pragma unroll
        for (int l = l0; l < l0 + 8; ++l) x -= c[l] * g[l];
      }
    return x;
  };
  // The largest modulus, lowest index on ties, of candidates x (absent: NaN or
  // out of the block; last: before these): published per wave with its row g
  // (whole groups of 8 below k), then chosen from the waves; a wave without
  // candidates offers zero.  Moduli are compared as integers.
  auto pick = [&](int sb, double x, bool in, bool last, const double (&g)[kCbRank], int k, int& wave) {
    const unsigned long long bits = __builtin_bit_cast(unsigned long long, x) & 0x7fffffffffffffffull;
    const bool open = in && (last || x == x);
    const uint32_t hi = !open ? 0u : last ? 1u : (uint32_t)(bits >> 32) + 2u;
    const uint32_t lo = open && !last ? (uint32_t)bits : 0u;
    const uint32_t mh = wave_max(hi);
    bool best = hi == mh;
    const uint32_t ml = wave_max(best ? lo : 0u);  // (lane moves: every lane takes part)
    best = best && lo == ml;
    const unsigned long long hit = __ballot(best);  // indices ascend with the lane
    if (lane == (int)__builtin_ctzll(hit)) {
      ckey[sb][w] = ((unsigned long long)mh << 32) | ml;
      cidx[sb][w] = tid;
      cval[sb][w] = mh ? x : 0.0;
#pragma unroll
      for (int l0 = 0; l0 < kCbRank; l0 += 8)
        if (l0 < k) {
#pragma unroll
          for (int l = l0; l < l0 + 8; ++l) hist[sb][w][l] = g[l];
        }
    }
    __syncthreads();
    unsigned long long key = ckey[sb][0];
    wave = 0;
#pragma unroll
    for (int o = 1; o < NW; ++o) {
      const unsigned long long ko = ckey[sb][o];
      if (ko > key) {
        key = ko;
        wave = o;
      }
    }
    wave = __builtin_amdgcn_readfirstlane(wave);
  };

  double u[kCbRank], v[kCbRank];
#pragma unroll
  for (int l = 0; l < kCbRank; ++l) u[l] = v[l] = 0.0;
  int i = 0, wi = 0;
  bool used = false;
#pragma unroll 1
  for (int k = 0; k < b.rank; ++k) {
    used = used || tid == i;
    double x = 0.0;
    if (iscol) x = residual(entry(i, tid), hist[1][wi], v, k);
    int wj;
    pick(0, x, iscol, false, v, k, wj);
    const int j = cidx[0][wj];
    const double delta = cval[0][wj];
    const bool exhausted = delta == 0.0;
    const double vk = exhausted ? 0.0 : x / delta;
    if (iscol) V[(b.c0 + tid) + (int64_t)(b.col + k) * ldv] = vk;
    double y = 0.0;
    if (isrow && !exhausted) y = residual(entry(tid, j), hist[0][wj], u, k);
    if (isrow) U[(b.r0 + tid) + (int64_t)(b.col + k) * ldu] = y;
#pragma unroll
    for (int l0 = 0; l0 < kCbRank; l0 += 8)
      if (l0 == (k & ~7)) {
#pragma unroll
        for (int l = l0; l < l0 + 8; ++l) {
          v[l] = l == k ? (iscol ? vk : 0.0) : v[l];
          u[l] = l == k ? y : u[l];
        }
      }
    pick(1, y, isrow, used, u, k + 1, wi);
    i = cidx[1][wi];
  }
}

// FP64 n x c (ld lds) to the storage type (ld ldd)
template <typename TS>
__global__ __launch_bounds__(kCsThreads) void store_cols_kernel(int64_t n, const double* __restrict__ src, int64_t lds,
                                                                TS* dst, int64_t ldd) {
  const int64_t i = (int64_t)blockIdx.x * kCsThreads + threadIdx.x;
  if (i < n) dst[i + (int64_t)blockIdx.y * ldd] = (TS)src[i + (int64_t)blockIdx.y * lds];
}

template <typename TS>
hipError_t launch_construct_leaves(hipStream_t s, const ConstructKernel& k, int nleaf, const int64_t* d_off, int m_max,
                                   TS* D, int64_t ldd) {
  if (nleaf == 0 || m_max > kCsThreads) return hipErrorInvalidValue;
  constexpr int ccols = 16;
  hipLaunchKernelGGL(construct_leaves_kernel<TS>, dim3(nleaf, (m_max + ccols - 1) / ccols), dim3(kCsThreads), 0, s, k,
                     d_off, m_max, ccols, D, ldd);
  return hipGetLastError();
}
template hipError_t launch_construct_leaves<double>(hipStream_t, const ConstructKernel&, int, const int64_t*, int,
                                                    double*, int64_t);
template hipError_t launch_construct_leaves<float>(hipStream_t, const ConstructKernel&, int, const int64_t*, int,
                                                   float*, int64_t);

int aca_tile_elems() { return kCsTile; }

int aca_block_class(int m, int n, int rank) {
  const int rows = std::max(m, n);
  if (rank > kCbRank || rows > kCbRows) return 3;
  return rows <= 128 ? 0 : rows <= 256 ? 1 : 2;
}

// A class's launch is a chain of 2 rank half steps (one a round of its workgroups:
// 512 threads a CU) in front of the tiled steps.  These are bound by their 2 rank
// launches, about 20 us a step, until their tiles fill the chip (8 of 256 threads
// a CU), and by memory beyond; below that a few more tiles cost nothing and the
// chain is time added.  So a class, the shortest blocks first, gets its launch
// where enough work stays behind to keep the tiled steps above their launches:
// rows times rank of 2^24 for every round; the shortest blocks, whose tiles are
// nearly empty, as soon as all tiles together fill the chip.  Gaussian kernel, rank
// 32, us with none, the first, the first two and all three classes:
//   leaf 128, N = 2^13: 681, 743, -, 929; 2^16: 1319, 1330, -, 1442;
//     2^17: 2741, 2566, 2408, 2293; rank 16, 2^17: 936, 876, 842, 861
//   leaf 64, N = 2^15: 962, 1000, -, 1150; 2^16: 1606, 1415, 1460, 1533
//   leaf 256 (no first), N = 2^17: 2502, -, 2324, 2217; rank 16: 858, -, 818, 833
// Where every block has a class there are no other launches (N = 1024, leaf
// 128, rank 32: 516 and 308).
int aca_own_launches(const int64_t (&blocks)[4], const int64_t (&tiles)[4], const int64_t (&work)[4]) {
  if (blocks[3] == 0) return 7;
  const int64_t all = tiles[0] + tiles[1] + tiles[2] + tiles[3];
  int64_t left = work[0] + work[1] + work[2] + work[3];
  int own = 0;
  for (int c = 0; c < 3; ++c) {
    if (blocks[c] == 0) continue;
    left -= work[c];
    const double rounds = std::max(1.0, (double)blocks[c] * (128 << c) / (256 * 512));
    if (c == 0 ? all < 256 * 8 : left < rounds * (1 << 24)) break;
    own |= 1 << c;
  }
  return own;
}

hipError_t launch_aca_blocks(hipStream_t s, const ConstructKernel& k, int cls, int nblocks, const AcaBlock* blocks,
                             double* U, int64_t ldu, double* V, int64_t ldv) {
  if (nblocks == 0) return hipSuccess;
  if (cls == 0)
    hipLaunchKernelGGL(aca_block_kernel<128>, dim3(nblocks), dim3(128), 0, s, k, blocks, U, ldu, V, ldv);
  else if (cls == 1)
    hipLaunchKernelGGL(aca_block_kernel<256>, dim3(nblocks), dim3(256), 0, s, k, blocks, U, ldu, V, ldv);
  else if (cls == 2)
    hipLaunchKernelGGL(aca_block_kernel<kCbRows>, dim3(nblocks), dim3(kCbRows), 0, s, k, blocks, U, ldu, V, ldv);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_aca_step(hipStream_t s, const ConstructKernel& k, int ntiles, const AcaBlock* blocks,
                           const AcaTile* tiles, int step, int kmax, double* U, int64_t ldu, double* V, int64_t ldv,
                           AcaPartials p) {
  if (ntiles == 0) return hipSuccess;
  if (kmax > HODLR_MAX_RANK) return hipErrorInvalidValue;
  hipLaunchKernelGGL(aca_row_kernel, dim3(ntiles), dim3(kCsThreads), 0, s, k, blocks, tiles, step, kmax,
                     (const double*)U, ldu, V, ldv, (const double*)p.cp_abs, (const int*)p.cp_idx, p.rp_abs, p.rp_val,
                     p.rp_idx, p.piv);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(aca_col_kernel, dim3(ntiles), dim3(kCsThreads), 0, s, k, blocks, tiles, step, kmax, U, ldu, V,
                     ldv, (const double*)p.rp_abs, (const double*)p.rp_val, (const int*)p.rp_idx, p.cp_abs, p.cp_idx,
                     (const int*)p.piv);
  return hipGetLastError();
}

template <typename TS>
hipError_t launch_store_cols(hipStream_t s, int64_t n, int ncols, const double* src, int64_t lds, TS* dst,
                             int64_t ldd) {
  if (n == 0 || ncols == 0) return hipSuccess;
  hipLaunchKernelGGL(store_cols_kernel<TS>, dim3((unsigned)((n + kCsThreads - 1) / kCsThreads), ncols),
                     dim3(kCsThreads), 0, s, n, src, lds, dst, ldd);
  return hipGetLastError();
}
template hipError_t launch_store_cols<float>(hipStream_t, int64_t, int, const double*, int64_t, float*, int64_t);

}  // namespace hodlr
