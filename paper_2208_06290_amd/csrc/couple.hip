// Coupling systems (Section III-A eq. "e:k"; Alg. "a:gpuf" form K / factor K /
// solve W; Alg. "a:gpus" solve w):
//
//   K_g = [[V_a^T Y_a, I], [I, V_b^T Y_b]]   for the children a, b of parent g
//
// The products V^T Y arrive as per-tile partial sums (level pass), summed in
// fixed order (segment_reduce) to one item per node.
//
// couple_factor: one workgroup per parent; K is formed in LDS from the
//   children's products and inverted by a blocked Gauss-Jordan elimination with
//   partial pivoting, K^{-1} is stored (kp x kp, kp = 2r rounded up to 16, zero
//   padding), and W = K^{-1} rhs, the
//   right-hand sides [V_a^T Y_big(I_a, 1:R_l); V_b^T Y_big(I_b, 1:R_l)] of
//   eq. "e:node1", is formed on MFMA.
// couple_solve: w = K^{-1} [V_a^T x_a; V_b^T x_b] (eq. "e:node3"), or the
//   transposed product used by the adjoint.
#include "mfma.h"
#include "wave.h"

#include <algorithm>

namespace hodlr {

// ---------------------------------------------------------------------------
// segment sums: out[s] = sum of tiles [desc[s].x, desc[s].x + desc[s].y)
// ---------------------------------------------------------------------------
template <typename T, int NT>
__global__ void segment_reduce_kernel(const int2* __restrict__ desc, int64_t elems, const T* __restrict__ P,
                                      T* __restrict__ out) {
  const int sg = blockIdx.y;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= elems) return;
  const int2 d = desc[sg];  // d.y <= NT items
  // all loads in flight at once (clamped to the segment), summed in item order
  T v[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) v[t] = P[(int64_t)(d.x + min(t, d.y - 1)) * elems + e];
  T acc = v[0];
#pragma unroll
  for (int t = 1; t < NT; ++t)
    if (t < d.y) acc += v[t];
  out[(int64_t)sg * elems + e] = acc;
}

// maxy: largest item count of a segment (<= kSegTiles); the kernel issues that many loads
template <typename T>
hipError_t launch_segment_reduce(hipStream_t s, int nsegs, const int2* d_desc, int64_t elems, const T* P, T* out,
                                 int maxy) {
  if (nsegs == 0 || elems == 0) return hipSuccess;
  if (maxy < 1 || maxy > kSegTiles) return hipErrorInvalidValue;
  dim3 grid((unsigned)((elems + 255) / 256), (unsigned)nsegs);
  if (maxy <= 2)
    hipLaunchKernelGGL((segment_reduce_kernel<T, 2>), grid, dim3(256), 0, s, d_desc, elems, P, out);
  else if (maxy <= 4)
    hipLaunchKernelGGL((segment_reduce_kernel<T, 4>), grid, dim3(256), 0, s, d_desc, elems, P, out);
  else if (maxy <= 8)
    hipLaunchKernelGGL((segment_reduce_kernel<T, 8>), grid, dim3(256), 0, s, d_desc, elems, P, out);
  else
    hipLaunchKernelGGL((segment_reduce_kernel<T, kSegTiles>), grid, dim3(256), 0, s, d_desc, elems, P, out);
  return hipGetLastError();
}
template hipError_t launch_segment_reduce<double>(hipStream_t, int, const int2*, int64_t, const double*, double*, int);
template hipError_t launch_segment_reduce<float>(hipStream_t, int, const int2*, int64_t, const float*, float*, int);

template <typename T>
__device__ __forceinline__ T bcast(T v, int srclane);
template <>
__device__ __forceinline__ double bcast<double>(double v, int srclane) {
  int2 u = __builtin_bit_cast(int2, v);
  u.x = __builtin_amdgcn_readlane(u.x, srclane);
  u.y = __builtin_amdgcn_readlane(u.y, srclane);
  return __builtin_bit_cast(double, u);
}
template <>
__device__ __forceinline__ float bcast<float>(float v, int srclane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), srclane));
}

constexpr int kCfMaxRows = 128;  // rows of a padded K (r <= 64)

// Element e = tid + u * NT (u = 0, 1, ...) of an n2-row column-major block as
// (row, column), stepped without a division per element.
struct BlockWalk {
  int k, c, dq, dr, n2;
  __device__ __forceinline__ BlockWalk(int tid, int nt, int n2_) : n2(n2_) {
    k = tid % n2;
    c = tid / n2;
    dq = nt / n2;
    dr = nt % n2;
  }
  __device__ __forceinline__ void next() {
    k += dr;
    c += dq;
    if (k >= n2) {
      k -= n2;
      ++c;
    }
  }
};

// One panel of the in-place Gauss-Jordan elimination: columns 16 jb .. + 15 of
// K (LDS, column-major, ld ldk) by one wave, lane i holding rows i and (NS = 2)
// 64 + i of the panel in registers.  Step j takes the largest |K(., j)| among
// rows not pivoted yet (the lowest current position on ties, a NaN counts as
// infinite: the rule of LU with partial pivoting) and exchanges column j with
// the pivot's unit vector: K(i, c) -= K(i, j) / pv * K(p, c) for the other rows
// and columns of the panel, K(i, j) = -K(i, j) / pv.  The pivot row is divided
// by its pivot when the panel ends (the later steps are linear in it); its
// entry j is 1 until then.
//
// A step is one dependency chain (about 0.25 us in FP64), so nothing but the
// chain is left in it: the moduli are compared as integers, high words first
// (six one-instruction steps; low words and positions only on a tie), every
// lane divides its own candidate while the maximum is found, and what is
// recorded of a pivot stays in its lane until the panel ends.  The loop is
// rolled: the columns rotate, step j works on x[0] and the elimination of
// x[c + 1] is written to x[c], so they are back in place after 16 steps.
//   s_pos  row -> current position (the step it was pivoted at, once pivoted)
//   s_pan  row -> panel in which it was pivoted (-1: not yet)
//   s_prow step -> pivot row
//   spiv, sud (global): LAPACK-style interchange (plus p0) and 1 / pivot of step j
// Columns j >= nid are unit vectors e_j: nothing to search.  A zero pivot in
// column j is reported as column j - (j >= cut ? skip : 0) + c0 of K.
struct PanelInfo {
  unsigned long long* info;
  unsigned long long base;
  int cut, skip, c0;
};
template <typename T, int NS>
__device__ __forceinline__ void gj_panel(T* K, int ldk, int kp, int nid, int jb, int lane, int* s_pos, int* s_pan,
                                         int* s_prow, int32_t* spiv, int p0, T* sud, PanelInfo pi) {
  T x[NS][16];
  int pos[NS], from[NS];  // current position; position at the time it was pivoted
  bool open[NS], here[NS], zero[NS];
  T myrp[NS];
#pragma unroll
  for (int sl = 0; sl < NS; ++sl) {
    const int row = 64 * sl + lane;
    const bool in = row < kp;
#pragma unroll
    for (int c = 0; c < 16; ++c) x[sl][c] = in ? K[row + (16 * jb + c) * ldk] : T(0);
    pos[sl] = in ? s_pos[row] : 0x7fffffff;
    open[sl] = in && s_pan[row] < 0;
    here[sl] = zero[sl] = false;
    myrp[sl] = T(1);
    from[sl] = 0;
  }
#pragma unroll 1
  for (int j = 16 * jb; j < 16 * jb + 16; ++j) {
    int plane = j & 63, pslot = j >> 6, bk = j;
    bool nz = true;
    T rpv = T(1);
    if (j < nid) {  // uniform
      uint32_t hi[NS], lo[NS];
      T rp[NS];
#pragma unroll
      for (int sl = 0; sl < NS; ++sl) {
        modulus_words(x[sl][0], open[sl], hi[sl], lo[sl]);
        rp[sl] = T(1) / x[sl][0];
      }
      // keeps the divisions ahead of the search, whose waits they fill
      if constexpr (NS == 1) asm volatile("" : "+v"(rp[0]));
      else asm volatile("" : "+v"(rp[0]), "+v"(rp[NS - 1]));
      const uint32_t mx = wave_max(NS == 2 ? max(hi[0], hi[NS - 1]) : hi[0]);
      unsigned long long hit[NS];
      int nhit = 0;
#pragma unroll
      for (int sl = 0; sl < NS; ++sl) {
        hit[sl] = __ballot(hi[sl] == mx);
        nhit += __builtin_popcountll(hit[sl]);
      }
      if (nhit > 1) {  // uniform: low words, then the lowest position
        if constexpr (sizeof(T) == 8) {
          uint32_t c0 = hi[0] == mx ? lo[0] : 0u;
          if (NS == 2) c0 = max(c0, hi[NS - 1] == mx ? lo[NS - 1] : 0u);
          const uint32_t ml = wave_max(c0);
#pragma unroll
          for (int sl = 0; sl < NS; ++sl) hit[sl] = __ballot(hi[sl] == mx && lo[sl] == ml);
        }
        int c = 0x7fffffff;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) c = min(c, (hit[sl] >> lane) & 1 ? pos[sl] : 0x7fffffff);
        const int mp = wave_min(c);
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) hit[sl] &= __ballot(pos[sl] == mp);
      }
      pslot = NS == 2 && hit[0] == 0 ? 1 : 0;
      plane = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(pslot ? hit[NS - 1] : hit[0]));
      nz = bcast(pslot ? x[NS - 1][0] : x[0][0], plane) != T(0);
      rpv = nz ? bcast(pslot ? rp[NS - 1] : rp[0], plane) : T(0);  // no elimination after a zero pivot
      bk = __builtin_amdgcn_readlane(pslot ? pos[NS - 1] : pos[0], plane);
    }
    T g[NS];
    bool me[NS];
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) {
      me[sl] = lane == plane && sl == pslot;
      g[sl] = me[sl] ? T(0) : x[sl][0] * rpv;
      if (open[sl] && pos[sl] == j) pos[sl] = bk;  // the row displaced by the interchange
      open[sl] = open[sl] && !me[sl];
      here[sl] = here[sl] || me[sl];
      pos[sl] = me[sl] ? j : pos[sl];
      from[sl] = me[sl] ? bk : from[sl];
      myrp[sl] = me[sl] && nz ? rpv : myrp[sl];
      zero[sl] = zero[sl] || (me[sl] && !nz);
    }
#pragma unroll
    for (int c = 0; c < 15; ++c) {
      const T pc = bcast(pslot ? x[NS - 1][c + 1] : x[0][c + 1], plane);
#pragma unroll
      for (int sl = 0; sl < NS; ++sl) x[sl][c] = x[sl][c + 1] - g[sl] * pc;  // g = 0 in the pivot row
    }
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) x[sl][15] = me[sl] ? T(1) : -g[sl];
  }
#pragma unroll
  for (int sl = 0; sl < NS; ++sl) {
    const int row = 64 * sl + lane;
    if (row < kp) {
#pragma unroll
      for (int c = 0; c < 16; ++c) K[row + (16 * jb + c) * ldk] = x[sl][c] * myrp[sl];
      s_pos[row] = pos[sl];
      if (here[sl]) {
        s_pan[row] = jb;
        s_prow[pos[sl]] = row;
        spiv[pos[sl]] = p0 + from[sl];
        sud[pos[sl]] = zero[sl] ? T(INFINITY) : myrp[sl];
        if (zero[sl])
          atomicMin(pi.info, pi.base | (unsigned long long)(pos[sl] - (pos[sl] >= pi.cut ? pi.skip : 0) + pi.c0));
      }
    }
  }
}

// The row (of 16) that lane li feeds as MFMA A operand so that register t of
// lane group lq of the result holds row 4 lq + t.
template <typename T>
__device__ __forceinline__ int row4_of_lane(int li) {
  return sizeof(T) == 8 ? 4 * (li & 3) + (li >> 2) : li;
}

// Four consecutive rows i0 .. of a column of a child's product (r rows,
// zero past them).  vec: r % 4 = 0, one access.
template <typename T>
__device__ __forceinline__ void load_col4(const T* col, int r, int i0, bool vec, T (&v)[4]) {
  if (vec) {
    typedef T V4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));
    const V4 x = *reinterpret_cast<const V4*>(col + min(i0, r - 4));
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = i0 < r ? x[s] : T(0);
  } else {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const T x = col[min(i0 + s, r - 1)];
      v[s] = i0 + s < r ? x : T(0);
    }
  }
}
// Four consecutive rows i0 .. (below r) of a column of a child's W.
template <typename T, typename V>
__device__ __forceinline__ void store_col4(T* col, int r, int i0, bool vec, const V& acc) {
  if (vec) {
    typedef T V4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));
    if (i0 < r) {
      V4 x;
#pragma unroll
      for (int t = 0; t < 4; ++t) x[t] = acc[t];
      *reinterpret_cast<V4*>(col + i0) = x;
    }
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (i0 + t < r) col[i0 + t] = acc[t];
  }
}

// 16 x 16 tile of a product of two LDS matrices (ld ldk): sum over 16 nt of A(li, k) B(k, li)
template <typename T>
__device__ __forceinline__ typename Mfma<T>::V tile_mm(const T* A, const T* B, int ldk, int nt, int li, int lq) {
  typename Mfma<T>::V acc = vzero<typename Mfma<T>::V>();
  for (int q = 0; q < nt; ++q) {
    T av[4], bv[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = 16 * q + 4 * s + lq;
      av[s] = A[li + k * ldk];
      bv[s] = B[k + li * ldk];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = Mfma<T>::mma(av[s], bv[s], acc);
  }
  return acc;
}

// In-place Gauss-Jordan inversion of the n x n matrix at K (n % 16 = 0, LDS),
// 16-column panels: one wave runs a panel in registers, then every other wave
// applies the panel's exchanges to its own 16 columns as one product,
// K(i, c) = [i not a pivot row] K(i, c) + sum_j P(i, j) K(p_j, c), on MFMA.
// The wave of the next panel goes straight on to it: one barrier per panel.
// Entry (p_j, c) ends as K^{-1}(j, p_c); permuted() puts it in place.
template <typename T, int NW, int NS, int NB>
__device__ __forceinline__ void gj_invert(T* K, int ldk, int n, int nid, int tid, int w, int* s_pos, int* s_pan,
                                          int* s_prow, int32_t* spiv, int p0, T* sud, PanelInfo pi) {
  using M = Mfma<T>;
  using V = typename M::V;
  constexpr int NT = 64 * NW;
  const int lane = tid & 63, li = lane & 15, lq = lane >> 4, nb = n >> 4;
  for (int jb = 0; jb < nb; ++jb) {
    if (w == jb) gj_panel<T, NS>(K, ldk, n, nid, jb, lane, s_pos, s_pan, s_prow, spiv, p0, sud, pi);
    __syncthreads();
    if (w != jb && w < nb) {
      T* Kc = K + (16 * w + li) * ldk;
      T bv[4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) bv[ks] = Kc[s_prow[16 * jb + 4 * ks + lq]];
#pragma unroll
      for (int rb = 0; rb < NB; ++rb) {
        if (rb >= nb) continue;
        V acc;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int row = 16 * rb + M::crow(lq, t);
          const T x = Kc[row];
          acc[t] = s_pan[row] == jb ? T(0) : x;
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) acc = M::mma(K[16 * rb + li + (16 * jb + 4 * ks + lq) * ldk], bv[ks], acc);
#pragma unroll
        for (int t = 0; t < 4; ++t) Kc[16 * rb + M::crow(lq, t)] = acc[t];
      }
    }
  }
  __syncthreads();
  constexpr int NPT = 16 * NB * 16 * NB / NT;
  T v[NPT];
  BlockWalk it(tid, NT, n);
#pragma unroll
  for (int u = 0; u < NPT; ++u) {
    v[u] = it.c < n ? K[it.k + it.c * ldk] : T(0);
    it.next();
  }
  __syncthreads();
  BlockWalk st(tid, NT, n);
#pragma unroll
  for (int u = 0; u < NPT; ++u) {
    if (st.c < n) K[s_pos[st.k] + s_prow[st.c] * ldk] = v[u];
    st.next();
  }
  __syncthreads();
}

// Coupling factor (any r <= 64), K in LDS with both halves padded to
// h = r rounded up to 16: [[T_a, I], [I, T_b]] of size 2h, the padding of T_a
// and T_b zero.  The elimination is a chain of dependent steps, 0.5 us each in
// FP64 whatever the number of parents, so the number of steps decides.  When
// every |T| < 1, partial pivoting on K takes the identity's ones for its first
// h pivots (row h + j in column j, no other candidate reaches 1), which leaves
// S = I - T_a T_b for the other h; so S is formed on MFMA, inverted with h
// steps, and with M = S^{-1}
//   K^{-1} = [[-T_b M, I + T_b M T_a], [M, -M T_a]].
// Otherwise all 2h steps run on K.  Pivots, interchanges and a singular K are
// those of LU with partial pivoting on K in both cases.  Rank 32, FP64, one
// parent: 41 us with 64 steps (one barrier per step on four waves: 53 us);
// a factorization's 12 levels at N = 2^20: 0.78 ms (1.37 ms), 9 levels of rank
// 64 at N = 2^17: 0.95 ms (1.93 ms).  NW = 4 waves up to
// 2h = 64, 8 up to 128.  W = K^{-1} rhs then streams 16 columns per wave from
// and to memory, K^{-1} read from LDS.
// (Ranks that correct their products, couple_corrects, leave W to
// couple_apply_kernel and keep T_a and T_b in Kt for it.  W is null where no
// level has columns above it, Kt where no rank corrects.)
template <typename T, int NW>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 3 : 1) void couple_factor_kernel(
    int r, int kp, int Rp, const T* __restrict__ segs, const int32_t* __restrict__ seg_start, T* __restrict__ Kinv,
    int32_t* __restrict__ Kpiv, T* __restrict__ Kud, T* __restrict__ Kt, T* __restrict__ W, unsigned long long* info,
    int level, int L) {
  using M = Mfma<T>;
  using V = typename M::V;
  constexpr int NT = 64 * NW, NB = NW, TPW = NW / 4;  // threads, 16-row blocks of K, tiles of S per wave
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* K = reinterpret_cast<T*>(smem_raw);
  __shared__ int s_pos[16 * NB], s_pan[16 * NB], s_prow[16 * NB];
  const int g = blockIdx.x;
  const int h = (r + 15) & ~15, n = 2 * h, n2 = 2 * r;
  const int ldk = n + 1;  // rows and columns of a block on different banks
  const int64_t elems = (int64_t)r * (Rp + r);
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const T* Pa = segs + (int64_t)seg_start[2 * g] * elems;
  const T* Pb = segs + (int64_t)seg_start[2 * g + 1] * elems;
  int32_t* pvg = Kpiv + (int64_t)g * n;
  T* udg = Kud + (int64_t)g * n;
  bool small = true;
  {
    // K from the products' last r columns, loads in batches
    constexpr int B = 8;
    BlockWalk it(tid, NT, n);
    while (it.c < n) {
      T v[B];
      BlockWalk st = it;
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int i = it.k, j = it.c;
        T x = i - j == h || j - i == h ? T(1) : T(0);
        if (i < r && j < r) x = Pa[i + (int64_t)(Rp + j) * r];
        else if (i >= h && j >= h && i < h + r && j < h + r) x = Pb[(i - h) + (int64_t)(Rp + j - h) * r];
        v[u] = x;
        it.next();
      }
#pragma unroll
      for (int u = 0; u < B; ++u) {
        if (st.c < n) {
          K[st.k + st.c * ldk] = v[u];
          if ((st.k < h) == (st.c < h)) small = small && fabs(v[u]) < T(1);
        }
        st.next();
      }
    }
    for (int i = tid; i < n; i += NT) {
      s_pos[i] = i;
      s_pan[i] = -1;
    }
  }
  small = __syncthreads_and(small);
  const unsigned long long base = ((unsigned long long)(L - level) << 44) | ((unsigned long long)g << 16);
  const int nt = h >> 4;
  if (small) {
    T* S = K + h * ldk;         // rows 0 .., columns h ..
    T* X = K + h;               // rows h .., columns 0 ..
    T* Tb = K + h + h * ldk;
    int ti[TPW], tj[TPW];
    bool have[TPW];
#pragma unroll
    for (int u = 0; u < TPW; ++u) {
      const int id = w + NW * u;
      have[u] = id < nt * nt;
      ti[u] = 16 * (have[u] ? id % nt : 0);
      tj[u] = 16 * (have[u] ? id / nt : 0);
    }
#pragma unroll
    for (int u = 0; u < TPW; ++u)
      if (have[u]) {
        const V c = tile_mm(K + ti[u], Tb + tj[u] * ldk, ldk, nt, li, lq);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int i = ti[u] + M::crow(lq, t), j = tj[u] + li;
          S[i + j * ldk] = (i == j ? T(1) : T(0)) - c[t];
        }
      }
    for (int j = tid; j < h; j += NT) {
      pvg[j] = h + j;
      udg[j] = T(1);
    }
    __syncthreads();
    gj_invert<T, NW, 1, NW / 2>(S, ldk, h, r, tid, w, s_pos, s_pan, s_prow, pvg + h, h, udg + h,
                                PanelInfo{info, base, h, 0, r});
#pragma unroll
    for (int u = 0; u < TPW; ++u)
      if (have[u]) {
        const V c = tile_mm(S + ti[u], K + tj[u] * ldk, ldk, nt, li, lq);
#pragma unroll
        for (int t = 0; t < 4; ++t) X[ti[u] + M::crow(lq, t) + (tj[u] + li) * ldk] = c[t];  // M T_a
      }
    __syncthreads();
    V x2[TPW], x3[TPW], m[TPW], x1[TPW];
#pragma unroll
    for (int u = 0; u < TPW; ++u)
      if (have[u]) {
        x2[u] = tile_mm(Tb + ti[u], S + tj[u] * ldk, ldk, nt, li, lq);
        x3[u] = tile_mm(Tb + ti[u], X + tj[u] * ldk, ldk, nt, li, lq);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int e = ti[u] + M::crow(lq, t) + (tj[u] + li) * ldk;
          m[u][t] = S[e];
          x1[u][t] = X[e];
        }
      }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < TPW; ++u)
      if (have[u]) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int i = ti[u] + M::crow(lq, t), j = tj[u] + li, e = i + j * ldk;
          K[e] = -x2[u][t];
          S[e] = (i == j ? T(1) : T(0)) + x3[u][t];
          X[e] = m[u][t];
          Tb[e] = -x1[u][t];
        }
      }
    __syncthreads();
  } else {
    gj_invert<T, NW, NW / 4, NB>(K, ldk, n, n, tid, w, s_pos, s_pan, s_prow, pvg, 0, udg,
                                 PanelInfo{info, base, h, h - r, 0});
  }
  // K^{-1} without the padding of the halves
  T* Kg = Kinv + (int64_t)g * kp * kp;
  for (BlockWalk e(tid, NT, kp); e.c < kp; e.next()) {
    const int i = e.k < r ? e.k : e.k + h - r, j = e.c < r ? e.c : e.c + h - r;
    Kg[e.k + e.c * kp] = e.k < n2 && e.c < n2 ? K[i + j * ldk] : T(0);
  }
  if (couple_corrects(r)) {
    T* Tg = Kt + (int64_t)g * 2 * r * r;
    for (int e = tid; e < r * r; e += NT) {
      Tg[e] = Pa[(int64_t)Rp * r + e];
      Tg[r * r + e] = Pb[(int64_t)Rp * r + e];
    }
    return;
  }
  // W = K^{-1} rhs: wave w takes the column blocks w, w + NW, ..; row blocks
  // 0 .. nt - 1 are the first child's, nt .. 2 nt - 1 the second's (r % 8 = 0 here)
  T* Wg = W + (int64_t)g * n2 * Rp;
  for (int c0 = 16 * w; c0 < Rp; c0 += 16 * NW) {
    const int64_t c = min(c0 + li, Rp - 1);
    T bv[NB][4];
#pragma unroll
    for (int q = 0; q < NB; ++q)
      if (q < 2 * nt) load_col4((q < nt ? Pa : Pb) + c * r, r, 16 * (q < nt ? q : q - nt) + 4 * lq, true, bv[q]);
#pragma unroll 2
    for (int rb = 0; rb < 2 * nt; ++rb) {
      V acc = vzero<V>();
#pragma unroll
      for (int q = 0; q < NB; ++q)
        if (q < 2 * nt) {
#pragma unroll
          for (int s = 0; s < 4; ++s)
            acc = M::mma(K[16 * rb + row4_of_lane<T>(li) + (16 * q + 4 * lq + s) * ldk], bv[q][s], acc);
        }
      if (c0 + li < Rp)
        store_col4(Wg + c * n2 + (rb < nt ? 0 : r), r, 16 * (rb < nt ? rb : rb - nt) + 4 * lq, true, acc);
    }
  }
}

// ---------------------------------------------------------------------------
// couple_solve
// ---------------------------------------------------------------------------
// Four waves per parent, wave w on the 16-row blocks w, w + 4 of the result
// (blocks of either child's rows); K^{-1} (or its transpose) comes from memory
// as MFMA A operand, all of a block's loads in flight together, and serves
// every 16-column block of the right-hand sides.  Bound by that one latency:
// 11 levels of 32-column adjoint solves at N = 2^18, rank 32 take 125 us (one
// wave per parent with four columns at a time: 320 us), and one column gains
// too (rank 64, 9 levels: 116 against 312 us).
// REF: w -> w + K^{-1} (rhs - K w) once, the waves exchanging w and the
// residual through LDS.  A product with K^{-1} leaves an error of cond(K)^2
// roundings where substitution with an LU leaves cond(K); the correction
// brings it back.  With it W and the factors of an uneven tree (N = 102846,
// ranks 37 .. 31) take 1.01 ms and a 3-column solve's levels 0.15 ms (LU and
// substitution: 1.84 and 0.32 ms).
template <typename T, int TRANS, int NB, bool REF>
__global__ __launch_bounds__(256) void couple_apply_kernel(int r, int kp, int nrhs, int64_t elems,
                                                           const T* __restrict__ segs, const int32_t* __restrict__ seg_start,
                                                           const T* __restrict__ Kinv, const T* __restrict__ Kt,
                                                           T* __restrict__ w_) {
  using M = Mfma<T>;
  using V = typename M::V;
  constexpr int NR = NB / 4;  // row blocks of a wave
  __shared__ T xs[REF ? 2 : 1][REF ? NB * 256 : 1];  // [w, residual]: block, lane, 4 rows
  const int g = blockIdx.x;
  const int n2 = 2 * r, nt = (r + 15) >> 4;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const T* Pa = segs + (int64_t)seg_start[2 * g] * elems;
  const T* Pb = segs + (int64_t)seg_start[2 * g + 1] * elems;
  const T* Kg = Kinv + (int64_t)g * kp * kp;
  T* wg = w_ + (int64_t)g * n2 * nrhs;
  const bool vec = r % 4 == 0;
  T av[NR][NB][4];
#pragma unroll
  for (int u = 0; u < NR; ++u) {
    const int rb = w + 4 * u;
    if (rb >= 2 * nt) continue;
    const int half = rb >= nt, row = half * r + min(16 * (half ? rb - nt : rb) + row4_of_lane<T>(li), r - 1);
#pragma unroll
    for (int q = 0; q < NB; ++q)
      if (q < 2 * nt) {
        const int kh = q >= nt, k0 = 16 * (kh ? q - nt : q) + 4 * lq;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int k = kh * r + min(k0 + s, r - 1);
          av[u][q][s] = TRANS ? Kg[k + row * kp] : Kg[row + k * kp];
        }
      }
  }
  for (int c0 = 16 * blockIdx.y; c0 < nrhs; c0 += 16 * gridDim.y) {
    const int64_t c = min(c0 + li, nrhs - 1);
    T bv[NB][4];
#pragma unroll
    for (int q = 0; q < NB; ++q)
      if (q < 2 * nt) load_col4((q < nt ? Pa : Pb) + c * r, r, 16 * (q < nt ? q : q - nt) + 4 * lq, vec, bv[q]);
    V x[NR];
#pragma unroll
    for (int u = 0; u < NR; ++u) {
      x[u] = vzero<V>();
      if (w + 4 * u < 2 * nt) {
#pragma unroll
        for (int q = 0; q < NB; ++q)
          if (q < 2 * nt) {
#pragma unroll
            for (int s = 0; s < 4; ++s) x[u] = M::mma(av[u][q][s], bv[q][s], x[u]);
          }
      }
    }
    if constexpr (REF) {
#pragma unroll
      for (int u = 0; u < NR; ++u)
        if (w + 4 * u < 2 * nt) {
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int rb = w + 4 * u, i = 16 * (rb >= nt ? rb - nt : rb) + 4 * lq + s;
            xs[0][(rb * 64 + lane) * 4 + s] = i < r ? x[u][s] : T(0);
          }
        }
      __syncthreads();
      // rhs - K x (K^T x): T x of the own child, x of the other
#pragma unroll
      for (int u = 0; u < NR; ++u) {
        const int rb = w + 4 * u;
        if (rb >= 2 * nt) continue;
        const int half = rb >= nt, i0 = 16 * (half ? rb - nt : rb), other = half ? rb - nt : rb + nt;
        const T* Tg = Kt + (int64_t)g * 2 * r * r + half * r * r;
        const int i = min(i0 + row4_of_lane<T>(li), r - 1);
        V acc = vzero<V>();
        for (int q = 0; q < nt; ++q) {
          T xv[4], tv[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int k = min(16 * q + 4 * lq + s, r - 1);
            tv[s] = TRANS ? Tg[k + i * r] : Tg[i + k * r];
            xv[s] = xs[0][((q + half * nt) * 64 + lane) * 4 + s];
          }
#pragma unroll
          for (int s = 0; s < 4; ++s) acc = M::mma(tv[s], xv[s], acc);
        }
        T rhs[4];
        load_col4((half ? Pb : Pa) + c * r, r, i0 + 4 * lq, vec, rhs);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const T res = rhs[s] - xs[0][(other * 64 + lane) * 4 + s] - acc[s];
          xs[1][(rb * 64 + lane) * 4 + s] = i0 + 4 * lq + s < r ? res : T(0);
        }
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < NR; ++u)
        if (w + 4 * u < 2 * nt) {
#pragma unroll
          for (int q = 0; q < NB; ++q)
            if (q < 2 * nt) {
#pragma unroll
              for (int s = 0; s < 4; ++s) bv[q][s] = xs[1][(q * 64 + lane) * 4 + s];
            }
          V d = vzero<V>();
#pragma unroll
          for (int q = 0; q < NB; ++q)
            if (q < 2 * nt) {
#pragma unroll
              for (int s = 0; s < 4; ++s) d = M::mma(av[u][q][s], bv[q][s], d);
            }
          x[u] += d;
        }
    }
#pragma unroll
    for (int u = 0; u < NR; ++u) {
      const int rb = w + 4 * u, half = rb >= nt;
      if (rb < 2 * nt && c0 + li < nrhs)
        store_col4(wg + c * n2 + half * r, r, 16 * (half ? rb - nt : rb) + 4 * lq, vec, x[u]);
    }
  }
}

template <typename T>
static hipError_t launch_apply(hipStream_t s, int trans, int nparents, int r, int kp, int ncols, int64_t elems,
                               const T* segs, const int32_t* d_seg_start, const T* Kinv, const T* Kt, T* w) {
  if (nparents == 0 || r == 0 || ncols == 0) return hipSuccess;
  if (r > kCfMaxRows / 2 || kp < 2 * r) return hipErrorInvalidValue;
  // few parents: column blocks over workgroups too
  const int blocks = (ncols + 15) / 16;
  const dim3 grid(nparents, std::min(blocks, std::max(1, 1024 / nparents)));
#define HODLR_CA(TR, NB, REF)                                                                                     \
  hipLaunchKernelGGL((couple_apply_kernel<T, TR, NB, REF>), grid, dim3(256), 0, s, r, kp, ncols, elems, segs,      \
                     d_seg_start, Kinv, Kt, w)
#define HODLR_CAT(NB, REF)          \
  if (trans) HODLR_CA(1, NB, REF);  \
  else HODLR_CA(0, NB, REF)
  if (couple_corrects(r)) {
    if (r > 32) {
      HODLR_CAT(8, true);
    } else {
      HODLR_CAT(4, true);
    }
  } else if (r > 32) {
    HODLR_CAT(8, false);
  } else {
    HODLR_CAT(4, false);
  }
#undef HODLR_CAT
#undef HODLR_CA
  return hipGetLastError();
}

template <typename T>
hipError_t launch_couple_factor(hipStream_t s, int nparents, int r, int kp, int Rp, const T* segs,
                                const int32_t* d_seg_start, T* Kinv, int32_t* Kpiv, T* Kud, T* Kt, T* W,
                                unsigned long long* info, int level, int L) {
  if (nparents == 0 || r == 0) return hipSuccess;
  const int n = 2 * ((r + 15) & ~15);
  if (n > kCfMaxRows || kp < 2 * r || kp > n) return hipErrorInvalidValue;
  const size_t smem = sizeof(T) * (size_t)n * (n + 1);
#define HODLR_CF(NW)                                                                                              \
  {                                                                                                               \
    auto k = couple_factor_kernel<T, NW>;                                                                         \
    hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);      \
    if (e != hipSuccess) return e;                                                                                \
    hipLaunchKernelGGL(k, dim3(nparents), dim3(64 * NW), smem, s, r, kp, Rp, segs, d_seg_start, Kinv, Kpiv, Kud, Kt, \
                       W, info, level, L);                                                                        \
  }
  if (n <= 64) HODLR_CF(4) else HODLR_CF(8)
#undef HODLR_CF
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !couple_corrects(r)) return e;
  return launch_apply<T>(s, 0, nparents, r, kp, Rp, (int64_t)r * (Rp + r), segs, d_seg_start, Kinv, Kt, W);
}
template hipError_t launch_couple_factor<double>(hipStream_t, int, int, int, int, const double*, const int32_t*,
                                                 double*, int32_t*, double*, double*, double*, unsigned long long*, int,
                                                 int);
template hipError_t launch_couple_factor<float>(hipStream_t, int, int, int, int, const float*, const int32_t*, float*,
                                                int32_t*, float*, float*, float*, unsigned long long*, int, int);

template <typename T>
hipError_t launch_couple_solve(hipStream_t s, int trans, int nparents, int r, int kp, int nrhs, const T* segs,
                               const int32_t* d_seg_start, const T* Kinv, const T* Kt, T* w) {
  return launch_apply<T>(s, trans, nparents, r, kp, nrhs, (int64_t)r * nrhs, segs, d_seg_start, Kinv, Kt, w);
}
template hipError_t launch_couple_solve<double>(hipStream_t, int, int, int, int, int, const double*, const int32_t*,
                                                const double*, const double*, double*);
template hipError_t launch_couple_solve<float>(hipStream_t, int, int, int, int, int, const float*, const int32_t*,
                                               const float*, const float*, float*);

}  // namespace hodlr
