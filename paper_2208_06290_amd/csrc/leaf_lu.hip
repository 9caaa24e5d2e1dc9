// Batched LU with partial pivoting of the leaf diagonal blocks
// (Alg. "a:fact" leaf loop / Alg. "a:gpuf" batched_LU_factorize_inplace on D_big^L).
//
// One workgroup (256 threads = 4 waves) per leaf, left-looking by 32-column
// chunks:
//   1. the chunk's original columns are loaded into MFMA accumulators in the
//      current row order (wave w owns the 16-row blocks b with b % 4 == w);
//   2. the chunk is swept with the L blocks of all earlier chunks on MFMA
//      (X_k = inv(L_kk) B_k by the owning wave, published through LDS,
//      B_b -= L_bk X_k by every wave), which leaves the U rows above the panel
//      and the Schur-complemented panel below;
//   3. the panel (rows below, 32 columns) is factored with one thread per row,
//      the row held in registers: pivot = largest magnitude, lowest current
//      position on ties (LAPACK idamax), rows are not moved - each thread
//      tracks its position; each wave with rows publishes its best candidate's
//      row in LDS and every thread selects the winner, one barrier per column.
//      The wave's search compares moduli as words (DPP maxima of the high words,
//      low words and positions only on ties).
// Entries are stored by original row while factoring (later interchanges move
// no data); a final pass writes them in pivoted order.  Four workgroups per CU
// in FP64, five with 4-byte elements: at most 128 registers per lane and 40 KB
// of LDS, so the panel rows reach the registers 8 columns at a time.
//
// Bound by instruction issue and latency of the panels (46 % of the time; the
// sweeps 19 %, the loads 16 % at the rate of memory, the moves to rows 11 %, the
// diagonal inverses 4 %).  4096 leaves of 256: FP64 3.00 ms, FP32 from FP64
// 2.11, bfloat16 updates (2048 leaves) 0.97; with all waves in every panel, the search on
// values and the inverses on half a wave in LDS 3.95, 2.79 and 1.35 ms.
//
// Output per leaf a (block of ldl x ldl, column-major, ld = ldl; ldl = m_max
// rounded up to 16; or, in place, the leaf's own rows of D with ld = ldd,
// which needs |I_a| % 16 == 0 so no 16 x 16 block reaches past the leaf):
//   lu     unit-lower L below the diagonal, U on and above; zero outside m_a x m_a
//          (the separate layout only)
//   piv    LAPACK-style interchanges: row j was swapped with piv[j] (0-based, >= j)
//   perm   composed row order: row i of P^T A is row perm[i] of A
//   udinv  1 / U_jj (1 outside m_a)
//   inv    inverses of the 16 x 16 diagonal blocks: [0][kb] = inv(L_kb,kb) (unit
//          lower), [1][kb] = inv(U_kb,kb) (upper); padded rows act as identity
// First exactly-zero pivot -> atomicMin(info, leaf << 20 | column).
#include "mfma.h"
#include "wave.h"

namespace hodlr {

constexpr int kLuThreads = 256;
constexpr int kCW = 32;  // chunk (panel) width

template <typename T, typename S, int CW, bool BF>
__global__ __launch_bounds__(kLuThreads, sizeof(T) == 4 ? 5 : 4) void leaf_lu_kernel(int ldl, const int64_t* __restrict__ leaf_off,
                                                             const S* D, int64_t ldd, T* lu, int64_t lul,
                                                             int inplace, int32_t* __restrict__ piv,
                                                             int32_t* __restrict__ perm,
                                                             T* __restrict__ udinv, T* invl,
                                                             unsigned long long* info) {
  using M = Mfma<T>;
  using V = typename M::V;
  // staging area: the earlier chunks' diagonal-block inverses for the sweep
  // (<= 14 blocks of 256), the panel rows 8 columns at a time ([row][8]), the
  // new diagonal block and the inversion scratch (2 x 1024)
  __shared__ T stage[14 * 256];
  __shared__ T xk[2][16 * CW];   // published X_k [row][col]
  __shared__ T crow_[2][4][CW];  // per wave: the row of its best pivot candidate
  __shared__ T cval[2][4];        // per wave: |candidate|
  __shared__ int ckey[2][4];      // per wave: candidate position (INT_MAX: none)
  __shared__ int pm[256];         // position -> original (leaf-local) row

  const int a = blockIdx.x;
  const int64_t o = leaf_off[a];
  const int m = (int)(leaf_off[a + 1] - o);
  const int tid0 = threadIdx.x, w0 = __builtin_amdgcn_readfirstlane(tid0 >> 6);
  T* F = lu + (inplace ? o : (int64_t)a * ldl * ldl);  // by original row while factoring (ld lul)
  T* IL = invl + (int64_t)a * 2 * (ldl / 16) * 256;
  int32_t* pv = piv + (int64_t)a * ldl;
  const int nbk = (m + 15) >> 4;
  const int nch = (m + CW - 1) / CW;

  for (int i = tid0; i < 256; i += kLuThreads) pm[i] = i;
  // zero padding outside m x m (never touched by the factorization)
  if (m < ldl && !inplace) {
    for (int j = 0; j < ldl; ++j)
      for (int i = tid0; i < ldl; i += kLuThreads)
        if (i >= m || j >= m) F[i + (int64_t)j * lul] = T(0);
  }
  __syncthreads();

  for (int c = 0; c < nch; ++c) {
    // lane coordinates are re-derived from opaque copies in every chunk so the
    // compiler cannot hoist lane-dependent addresses and constants out of the
    // chunk loop (they would otherwise stay live and spill)
    int tid = tid0, w = w0;
    asm volatile("" : "+v"(tid));
    asm volatile("" : "+s"(w));
    const int lane = tid & 63, li = lane & 15, lq = lane >> 4;
    const int c0 = CW * c;
    const int cw = min(CW, m - c0);
    // 1. load the chunk in the current row order
    V acc[4][CW / 16];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int cb = 0; cb < CW / 16; ++cb)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int row = 16 * (4 * q + w) + M::crow(lq, t);
          const int col = 16 * cb + li;
          acc[q][cb][t] = (row < m && col < cw) ? (T)D[o + pm[row] + (int64_t)(c0 + col) * ldd] : T(0);
        }
    // 2. sweep with the L blocks of the earlier chunks; their diagonal-block
    // inverses are staged in LDS first (the panel buffer is free until the
    // panel), so the owner's step waits on no global load
    const int nk = (CW / 16) * c;
    T* ILs = stage;
    for (int e = tid; e < nk * 256; e += kLuThreads) ILs[e] = IL[e];
    __syncthreads();
    for (int k = 0; k < nk; ++k) {
      T* xb = xk[k & 1];
      if ((k & 3) == w) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (4 * q + w == k) {
#pragma unroll
            for (int cb = 0; cb < CW / 16; ++cb) {
              T lv[4], bv[4];
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                lv[t] = ILs[k * 256 + li * 16 + M::crow(lq, t)];
                bv[t] = acc[q][cb][t];
              }
              const V nv = Mma16<T, BF>::mma(lv, bv, vzero<V>());
              acc[q][cb] = nv;
#pragma unroll
              for (int t = 0; t < 4; ++t) xb[M::crow(lq, t) * CW + 16 * cb + li] = nv[t];
            }
          }
      }
      // operands of this step's update are independent of X_k: load them
      // before the barrier (rows clamped in range, used only by active blocks)
      T av[4][4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int b = min(4 * q + w, nbk - 1);
        const int prow = pm[16 * b + li];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) av[q][ks] = -F[prow + (int64_t)(16 * k + 4 * ks + lq) * lul];
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int b = 4 * q + w;
        if (b > k && b < nbk) {  // uniform
          if constexpr (BF) {
#pragma unroll
            for (int cb = 0; cb < CW / 16; ++cb) {
              T xv[4];
#pragma unroll
              for (int ks = 0; ks < 4; ++ks) xv[ks] = xb[(4 * ks + lq) * CW + 16 * cb + li];
              acc[q][cb] = Mma16<T, true>::mma(av[q], xv, acc[q][cb]);
            }
          } else {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
              for (int cb = 0; cb < CW / 16; ++cb)
                acc[q][cb] = M::mma(av[q][ks], xb[(4 * ks + lq) * CW + 16 * cb + li], acc[q][cb]);
          }
        }
      }
    }
    // U rows above the panel are final
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int cb = 0; cb < CW / 16; ++cb)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int row = 16 * (4 * q + w) + M::crow(lq, t);
          const int col = 16 * cb + li;
          if (row < m && row < c0 && col < cw) F[pm[row] + (int64_t)(c0 + col) * lul] = acc[q][cb][t];
        }
    // 3. panel factorization, one thread per panel row
    const int pr = m - c0;
    const bool own = tid < pr;
    int mypos = tid;
    bool done = false;
    const int orig = own ? pm[c0 + tid] : 0;
    // panel rows to the registers through LDS, 8 columns at a time
    T r[CW];
#pragma unroll
    for (int h = 0; h < CW / 8; ++h) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int row = 16 * (4 * q + w) + M::crow(lq, t);
          if (row < m && row >= c0 && (li >> 3) == (h & 1)) stage[(row - c0) * 8 + (li & 7)] = acc[q][h >> 1][t];
        }
      __syncthreads();
#pragma unroll
      for (int cc = 0; cc < 8; ++cc) r[8 * h + cc] = own ? stage[tid * 8 + cc] : T(0);
      __syncthreads();
    }
    // waves without rows of this panel only keep the barriers
    const int nact = (pr + 63) >> 6;
    if (w >= nact) {
      for (int j = 0; j < cw; ++j) __syncthreads();
    } else {
#pragma unroll
      for (int j = 0; j < CW; ++j) {
        if (j < cw) {
          // one barrier per column: each wave publishes its best candidate (value,
          // position, row from column j on); every thread then picks the winner
          const int sb = j & 1;
          const bool cand = own && !done;
          uint32_t hi, lo;
          modulus_words(r[j], cand, hi, lo);  // a NaN can still be chosen
          const uint32_t mh = wave_max(hi);
          bool best = hi == mh;
          if constexpr (sizeof(T) == 8) {
            if (__builtin_popcountll(__ballot(best)) > 1) {
              const uint32_t ml = wave_max(best ? lo : 0u);  // (lane moves: every lane takes part)
              best = best && lo == ml;
            }
          }
          if (__builtin_popcountll(__ballot(best)) > 1) {
            const int first = wave_min(best && cand ? mypos : 0x7fffffff);
            best = best && mypos == first;
          }
          if (mh == 0) {  // no candidates in this wave
            if (lane == 0) {
              cval[sb][w] = T(-1);
              ckey[sb][w] = 0x7fffffff;
            }
          } else if (best) {
            const T v = fabs(r[j]);
            cval[sb][w] = v == v ? v : T(INFINITY);
            ckey[sb][w] = mypos;
#pragma unroll
            for (int cc = j; cc < CW; ++cc) crow_[sb][w][cc] = r[cc];
          }
          __syncthreads();
          T bv = cval[sb][0];
          int bk = ckey[sb][0], bw = 0;
#pragma unroll
          for (int x = 1; x < 4; ++x)
            if (x < nact) {
              const T xv = cval[sb][x];
              const int xk = ckey[sb][x];
              if (xv > bv || (xv == bv && xk < bk)) {
                bv = xv;
                bk = xk;
                bw = x;
              }
            }
          const T* prow = crow_[sb][bw];
          if (cand) {
            if (mypos == bk) {  // this row is the pivot of column j
              done = true;
              pv[c0 + j] = c0 + bk;
              if (r[j] == T(0)) atomicMin(info, ((unsigned long long)a << 20) | (unsigned long long)(c0 + j));
              mypos = j;
            } else {
              if (mypos == j) mypos = bk;  // the row displaced by the interchange
              const T pivot = prow[j];
              if (pivot != T(0)) {
                const T l = r[j] * (T(1) / pivot);
                r[j] = l;
#pragma unroll
                for (int cc = j + 1; cc < CW; ++cc) r[cc] -= l * prow[cc];
              }
            }
          }
        }
      }
    }
    // store the panel by original row and record the new row order; the rows
    // that became pivot rows also go to LDS as the chunk's 32 x 32 diagonal
    // block (pivoted order), from which the diagonal-block inverses are formed
    T* dblk = stage;  // [32][32] row-major; the panel no longer reads stage
    if (own) {
#pragma unroll
      for (int cc = 0; cc < CW; ++cc)
        if (cc < cw) F[orig + (int64_t)(c0 + cc) * lul] = r[cc];
      if (mypos < CW) {
#pragma unroll
        for (int cc = 0; cc < CW; ++cc) dblk[mypos * CW + cc] = cc < cw ? r[cc] : T(0);
      }
    }
    // rows beyond m act as identity
    for (int e = cw * CW + tid; e < CW * CW; e += kLuThreads) dblk[e] = e / CW == e % CW ? T(1) : T(0);
    __syncthreads();
    if (own) pm[c0 + mypos] = orig;
    // inverses of the new 16 x 16 diagonal blocks, a column per thread in
    // registers: wave 0 the unit-lower L blocks, wave 1 the upper U blocks
    if (lane < 32 && w < 2) {
      const int half = lane >> 4, kb = (CW / 16) * c + half;
      int cc = li;
      asm volatile("" : "+v"(cc));  // keeps the identity columns from being hoisted out of the chunk loop
      const T* Bk = dblk + (16 * half) * CW + 16 * half;  // element (i, j) at Bk[i * CW + j]
      if (kb < nbk) {
        T x[16];
        if (w == 0) {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            T sacc = (i == cc) ? T(1) : T(0);
#pragma unroll
            for (int jj = 0; jj < i; ++jj) sacc -= Bk[i * CW + jj] * x[jj];
            x[i] = (i >= cc) ? sacc : T(0);
            IL[kb * 256 + i * 16 + cc] = x[i];
          }
        } else {
#pragma unroll
          for (int i = 15; i >= 0; --i) {
            T sacc = (i == cc) ? T(1) : T(0);
#pragma unroll
            for (int jj = i + 1; jj < 16; ++jj) sacc -= Bk[i * CW + jj] * x[jj];
            x[i] = (i <= cc) ? sacc / Bk[i * CW + i] : T(0);
            IL[(ldl / 16 + kb) * 256 + i * 16 + cc] = x[i];
          }
        }
      }
    } else if (w == 2 && lane < CW && c0 + lane < ldl) {
      const int j = lane;
      udinv[(int64_t)a * ldl + c0 + j] = (j < cw) ? T(1) / dblk[j * CW + j] : T(1);
    }
    __syncthreads();
  }
  const int tid = tid0;
  // pivoted order: F[i, :] <- F[perm[i], :], 32 columns at a time; nothing
  // to do when no row moved
  const bool moved = tid < m && pm[tid] != tid;
  if (__syncthreads_or(moved)) {
    const int src = tid < m ? pm[tid] : tid;
    for (int g = 0; g < nch; ++g) {
      T r[CW];
#pragma unroll
      for (int cc = 0; cc < CW; ++cc) {
        const int col = min(CW * g + cc, m - 1);
        r[cc] = F[min(src, m - 1) + (int64_t)col * lul];
      }
      __syncthreads();
      if (moved) {
#pragma unroll
        for (int cc = 0; cc < CW; ++cc)
          if (CW * g + cc < m) F[tid + (int64_t)(CW * g + cc) * lul] = r[cc];
      }
      __syncthreads();
    }
  }
  int32_t* pmo = perm + (int64_t)a * ldl;
  for (int i = tid; i < ldl; i += kLuThreads) {
    pmo[i] = i < m ? pm[i] : i;
    if (i >= m) pv[i] = i;
    if (i >= nch * CW) udinv[(int64_t)a * ldl + i] = T(1);  // beyond the last chunk of a short leaf
  }
}

template <typename T, typename S>
hipError_t launch_leaf_lu(hipStream_t s, int nleaf, int ldl, const int64_t* d_leaf_off, const S* D, int64_t ldd,
                          T* lu, int64_t lul, int inplace, int32_t* piv, int32_t* perm, T* udinv, T* invl,
                          unsigned long long* info, int bf) {
  if (nleaf == 0) return hipSuccess;
  if (ldl % 16 || ldl > 256) return hipErrorInvalidValue;
  if (inplace ? lul < ldl : lul != ldl) return hipErrorInvalidValue;
  if constexpr (sizeof(T) == 4) {
    if (bf) {
      hipLaunchKernelGGL((leaf_lu_kernel<T, S, kCW, true>), dim3(nleaf), dim3(kLuThreads), 0, s, ldl, d_leaf_off, D,
                         ldd, lu, lul, inplace, piv, perm, udinv, invl, info);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((leaf_lu_kernel<T, S, kCW, false>), dim3(nleaf), dim3(kLuThreads), 0, s, ldl, d_leaf_off, D, ldd,
                     lu, lul, inplace, piv, perm, udinv, invl, info);
  return hipGetLastError();
}

template hipError_t launch_leaf_lu<double, double>(hipStream_t, int, int, const int64_t*, const double*, int64_t,
                                                   double*, int64_t, int, int32_t*, int32_t*, double*, double*,
                                                   unsigned long long*, int);
template hipError_t launch_leaf_lu<float, double>(hipStream_t, int, int, const int64_t*, const double*, int64_t,
                                                  float*, int64_t, int, int32_t*, int32_t*, float*, float*,
                                                  unsigned long long*, int);
template hipError_t launch_leaf_lu<float, float>(hipStream_t, int, int, const int64_t*, const float*, int64_t,
                                                 float*, int64_t, int, int32_t*, int32_t*, float*, float*,
                                                 unsigned long long*, int);

}  // namespace hodlr
