// Block triangular solves with stored LU factors, on MFMA.
//
//   trans = 0:  X = U^{-1} L^{-1} P^T B     (per block: P^T B takes rows perm[i])
//   trans = 1:  X = P L^{-T} U^{-T} B       (adjoint; rows scattered through perm)
//
// Used for the leaf solves of the factorization (Alg. "a:gpuf":
// batched_LU_solve_inplace on Y_big^L, all R columns of a leaf at once) and
// of the solution stage (Alg. "a:gpus").  The inverses of the 16 x 16 diagonal
// blocks of L and U come with the factorization, so every block step is a
// contraction: X_k = inv(M_kk) B_k, then B_b -= M_bk X_k for the blocks beyond.
//
// Two kernels (launch_leaf_trsm has the rule): trsm_kernel shares the row
// blocks of a chunk of columns between the waves of a workgroup,
// trsm_wide_kernel gives every wave columns of its own.
#include "mfma.h"

namespace hodlr {

constexpr int kTwLd = 17;  // padded row length of the owner's 16 x 16 turn-around buffer

// Resident workgroups per CU: four waves with accumulators of at most 64
// registers per lane (4 blocks x 2 column blocks of FP64, or 4 x 4 of FP32)
// keep four workgroups per CU, wider chunks two; eight waves two, or one.
template <typename T, int NW, int NQ, int NCB>
constexpr int trsm_occupancy() {
  return NW == 4 ? (NQ * NCB * (int)sizeof(T) <= 64 ? 4 : 2) : (NCB <= 2 ? 2 : 1);
}

// One workgroup per (block, chunk of columns).  The chunk (<= 256 rows)
// stays in MFMA accumulators for the whole solve: wave w of NW owns the
// 16-row blocks b with b % NW == w.  The owning wave forms X_k and publishes
// it through LDS (double buffered, one barrier per step), and every wave
// applies it to its blocks; the factor operands and the next owner's inverted
// diagonal block are fetched before the barrier.  The products run transposed
// (X^T = B^T M^{-T}) so that accumulator rows are matrix rows on the lanes:
// every global load and store covers whole 128-byte lines; transposed factors come
// in runs of four rows a lane (N = 2^18, leaf 128, FP64, 32 columns: 137 us, by
// elements 182; N = 2^17, FP32, one: 33 and 86).  Leaf blocks take
// 32-column chunks with 128 registers per lane (four workgroups per CU: the
// steps are short and latency-bound, so more resident workgroups pay more than
// wider chunks).
template <typename T, typename S, int TRANS, int NW, int NQ, int NCB, bool BF>
__global__ __launch_bounds__(64 * NW, (trsm_occupancy<T, NW, NQ, NCB>())) void trsm_kernel(int ldl, const int64_t* __restrict__ leaf_off,
                                                             const T* lu, int64_t lul, int inplace, const int32_t* __restrict__ perm,
                                                             const T* __restrict__ dinv, const S* B, int64_t ldb,
                                                             T* X, int64_t ldx, int ncols, int nchunks, int64_t gsb,
                                                             int64_t gsx) {
  using M = Mfma<T>;
  using V = typename M::V;
  constexpr int kThreads = 64 * NW;
  constexpr int kBlocks = NW * NQ;  // 16-row blocks of a block (row block b is owned by wave b % NW)
  constexpr int kCwT = 16 * NCB;     // columns of a chunk
  __shared__ T xk[2][16 * kCwT];   // published block X_k: [row][col]
  __shared__ T tw[NW][16 * kTwLd];  // per-wave turn-around of the owner's block

  const int lid = (int)xcd_remap(blockIdx.x, gridDim.x);
  const int a = lid / nchunks;
  const int chunk = lid % nchunks;
  const int64_t o = leaf_off[a];
  const int m = (int)(leaf_off[a + 1] - o);
  // first row of the block in B and X (row i of an operand at (i >> 8) gs + (i & 255); a block
  // never crosses a 256-row boundary of an operand in the row-group blocked layout)
  const S* Bb = B + group_row(o, gsb);
  T* Xb = X + group_row(o, gsx);
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c0 = chunk * kCwT;
  const int nbk = (m + 15) >> 4;
  const T* F = lu + (inplace ? o : (int64_t)a * ldl * ldl);  // ld lul
  const int32_t* pm = perm + (int64_t)a * ldl;
  const int nbd = ldl >> 4;
  const T* DI = dinv + (int64_t)a * 2 * nbd * 256;  // [0][kb]: inv(L_kk), [1][kb]: inv(U_kk)
  T* twv = tw[w];

  // B operand of X_k^T = B_k^T inv(M_kk)^T: inv(M_kk)(li, 4 ks + lq) for ks = 0..3,
  // read from the factorization's inverted diagonal blocks (sweep 0 is L
  // (trans 0) or U^T (trans 1), sweep 1 is U or L^T)
  auto load_inv = [&](int sweep, int k, T (&iv)[4]) {
    const int which = TRANS ? 1 - sweep : sweep;
    const T* src = DI + ((int64_t)which * nbd + k) * 256;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int j = 4 * ks + lq;
      iv[ks] = TRANS ? src[j * 16 + li] : src[li * 16 + j];
    }
  };

  // The chunk is held transposed: accumulator block (q, cb), register t holds
  // X(16 (NW q + w) + li, c0 + 16 cb + crow(lq, t)), so the 16 lanes of a row
  // group touch 16 consecutive rows of one column (whole 128-byte lines).
  V acc[NQ][NCB];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int row = 16 * (NW * q + w) + li;
    const int rowc = min(row, m - 1);
    const int src = TRANS ? rowc : pm[rowc];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int col = c0 + 16 * cb + M::crow(lq, t);
        const T v = (T)Bb[src + (int64_t)min(col, ncols - 1) * ldb];
        acc[q][cb][t] = (row < m && col < ncols) ? v : T(0);
      }
  }
  __syncthreads();  // B may alias X: all loads of the chunk precede any store

  // X_k^T = B_k^T inv(M_kk)^T for the wave owning block k (accumulator block
  // q): the block turns around through LDS to become the A operand; the
  // result stays in the accumulators and is published as X_k[row][col]
  auto owner = [&](int q, const T (&iv)[4], T* xb) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
      for (int t = 0; t < 4; ++t) twv[li * kTwLd + M::crow(lq, t)] = acc[q][cb][t];
      T tv[4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) tv[ks] = twv[(4 * ks + lq) * kTwLd + li];
      const V nv = Mma16<T, BF>::mma(tv, iv, vzero<V>());
      acc[q][cb] = nv;
#pragma unroll
      for (int t = 0; t < 4; ++t) xb[li * kCwT + 16 * cb + M::crow(lq, t)] = nv[t];
    }
  };
  // rows of block k that K-step ks takes: transposed factors are read in runs of 4 rows
  auto krow = [&](int ks) { return TRANS ? 4 * lq + ks : 4 * ks + lq; };
  // B_b^T -= X_k^T M_bk^T on accumulator block q2
  auto update = [&](int q2, const T (&av)[NQ][4], const T* xb) {
    if constexpr (BF) {
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        T xv[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) xv[ks] = xb[krow(ks) * kCwT + 16 * cb + li];
        acc[q2][cb] = Mma16<T, true>::mma(xv, av[q2], acc[q2][cb]);
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
          acc[q2][cb] = M::mma(xb[krow(ks) * kCwT + 16 * cb + li], av[q2][ks], acc[q2][cb]);
    }
  };

  // The steps are unrolled so that every block index is a compile-time
  // constant; steps past the last block of a short leaf are skipped (uniform).
#pragma clang loop unroll(full)
  for (int sweep = 0; sweep < 2; ++sweep) {

#pragma clang loop unroll(full)
    for (int st = 0; st < kBlocks; ++st) {
      const int k = sweep == 0 ? st : kBlocks - 1 - st;
      if (k < nbk) {  // uniform
        const int q = k / NW, wk = k % NW;
        // step index within the sweep decides the X buffer (sweep 1 starts at nbk - 1)
        const int sidx = sweep == 0 ? k : nbk - 1 - k;
        T* xb = xk[sidx & 1];
        T* xn = xk[(sidx + 1) & 1];
        // the first step's X_k is formed here, later ones one step ahead (look-ahead)
        if (sidx == 0 && w == wk) {
          T iv0[4];
          load_inv(sweep, k, iv0);
          owner(q, iv0, xb);
        }
        // the factor operands M(16 b + li, 16 k + krow(ks)) of this wave's blocks
        // on the far side of k do not depend on X_k: fetched before the barrier
        // (clamped in range, no branches)
        T av[NQ][4];
#pragma unroll
        for (int q2 = 0; q2 < NQ; ++q2) {
          if (sweep == 0 ? q2 < q : q2 > q) continue;  // never on the far side: compile time
          const int b = min(NW * q2 + w, nbk - 1);
          const int i = 16 * b + li;
          if constexpr (TRANS) load_run(F + 16 * k + 4 * lq + (int64_t)i * lul, av[q2]);
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) av[q2][ks] = -(TRANS ? av[q2][ks] : F[i + (int64_t)(16 * k + 4 * ks + lq) * lul]);
        }
        // look-ahead: the wave owning the next block updates it first and forms
        // X_next at once, so the next step starts without waiting for it
        const int kn = sweep == 0 ? k + 1 : k - 1;
        const bool nxt = sweep == 0 ? kn < nbk : kn >= 0;
        const int qn = kn / NW, wn = kn % NW;
        const bool la = nxt && w == wn;  // uniform
        T ivn[4];
        if (la) load_inv(sweep, kn, ivn);  // fetched before the barrier too
        __syncthreads();
        if (la) {
          update(qn, av, xb);
          owner(qn, ivn, xn);
        }
#pragma unroll
        for (int q2 = 0; q2 < NQ; ++q2) {
          if (sweep == 0 ? q2 < q : q2 > q) continue;
          const int b = NW * q2 + w;
          const bool act = (sweep == 0 ? (q2 > q || w > wk) : (q2 < q || w < wk)) && b < nbk &&
                           !(la && q2 == qn);  // uniform
          if (act) update(q2, av, xb);
        }
      }
    }
  }

  // store (the adjoint scatters rows through the permutation)
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int row = 16 * (NW * q + w) + li;
    if (row < m) {
      const int dst = TRANS ? pm[row] : row;
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int col = c0 + 16 * cb + M::crow(lq, t);
          if (col < ncols) Xb[dst + (int64_t)col * ldx] = acc[q][cb][t];
        }
    }
  }
}

// Wide right-hand sides: four waves per workgroup, each with 16 NC columns and
// all the rows of a leaf in accumulators, from the load of B to the store of X.
// A lane holds column li and rows 4 lq + t (t = 0..3) of each 16 x 16 block
// (the rows of the factor blocks enter permuted by row4 for that), so B and X
// move as runs of four rows, and register s of block k is directly the B
// operand of K-step s in X_k = inv(M_kk) B_k and B_b -= M_bk X_k: a wave needs
// nothing from the others, and the steps' chain (eight MFMAs) hides behind the
// updates of the other blocks.  The factor's blocks of column block k go
// through LDS in fragment order (one read gives a lane its values of four
// K-steps), the next step's in flight while this one computes; one barrier
// per step.  Each step still waits for that barrier, which more resident
// workgroups cover: 64 columns and three workgroups per CU in FP64.
constexpr int kTwThreads = 256;

template <typename T, typename S, int TRANS, int NB, int NC, bool BF>
__global__ __launch_bounds__(kTwThreads, (NB * NC * (int)sizeof(T) <= 64 ? 3 : 2)) void trsm_wide_kernel(int ldl, const int64_t* __restrict__ leaf_off, const T* lu,
                                                                  int64_t lul, int inplace,
                                                                  const int32_t* __restrict__ perm,
                                                                  const T* __restrict__ dinv, const S* B, int64_t ldb,
                                                                  T* X, int64_t ldx, int ncols, int nchunks,
                                                                  int64_t gsb, int64_t gsx) {
  using M = Mfma<T>;
  using V = typename M::V;
  constexpr int kCols = 64 * NC;
  __shared__ __align__(16) T frag[2][NB * 256 / (BF ? 2 : 1)];  // block, lane, 4 K-steps
  const int lid = (int)xcd_remap(blockIdx.x, gridDim.x);
  const int a = lid / nchunks, chunk = lid % nchunks;
  const int64_t o = leaf_off[a];
  const int m = (int)(leaf_off[a + 1] - o);
  const int nbk = (m + 15) >> 4;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c0 = chunk * kCols + 16 * NC * w;
  const T* F = lu + (inplace ? o : (int64_t)a * ldl * ldl);  // ld lul
  const int32_t* pm = perm + (int64_t)a * ldl;
  const int nbd = ldl >> 4;
  const T* DI = dinv + (int64_t)a * 2 * nbd * 256;  // [0][kb]: inv(L_kk), [1][kb]: inv(U_kk), row-major
  const S* Bb = B + group_row(o, gsb);
  T* Xb = X + group_row(o, gsx);

  // element (er, ec) of a factor block, one per thread, neighbours along the
  // stored columns; its place in the fragments
  const int er = TRANS ? tid >> 4 : tid & 15, ec = TRANS ? tid & 15 : tid >> 4;
  const int row4 = sizeof(T) == 8 ? 4 * (er & 3) + (er >> 2) : er;  // the lane that feeds row er
  const int place = (16 * (ec >> 2) + row4) * 4 + (ec & 3);
  // the blocks of step (sweep, k): inv(M_kk) and -M_bk beyond it.  Sweep 0 runs
  // down with L (TRANS: U^T), sweep 1 up with U (L^T).
  auto load_panel = [&](int sweep, int k, T (&v)[NB]) {
    const T* D = DI + ((int64_t)(TRANS ? 1 - sweep : sweep) * nbd + k) * 256;
    const T* Fk = TRANS ? F + 16 * k + ec + (int64_t)er * lul : F + er + (int64_t)(16 * k + ec) * lul;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (b == k) v[b] = D[TRANS ? ec * 16 + er : er * 16 + ec];
      else if (sweep == 0 ? b > k && b < nbk : b < k) v[b] = -(TRANS ? Fk[(int64_t)(16 * b) * lul] : Fk[16 * b]);
    }
  };
  auto store_panel = [&](int buf, int sweep, int k, const T (&v)[NB]) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (b == k || (sweep == 0 ? b > k && b < nbk : b < k)) {
        if constexpr (BF) reinterpret_cast<__bf16*>(frag[buf])[b * 256 + place] = (__bf16)v[b];
        else frag[buf][b * 256 + place] = v[b];
      }
  };

  // the right-hand sides, rows through the permutation (trans 0); four
  // consecutive rows in one access where they stay together
  V acc[NB][NC];
  int64_t cb[NC];
#pragma unroll
  for (int n = 0; n < NC; ++n) cb[n] = min(c0 + 16 * n + li, ncols - 1);
  T v[NB];
  load_panel(0, 0, v);
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    if (b >= nbk) continue;
    const int r0 = 16 * b + 4 * lq;
    int src[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int rc = min(r0 + t, m - 1);
      src[t] = TRANS ? rc : pm[rc];
    }
    if (__all(src[1] == src[0] + 1 && src[2] == src[0] + 2 && src[3] == src[0] + 3)) {
#pragma unroll
      for (int n = 0; n < NC; ++n) {
        T x[4];
        load_run(Bb + src[0] + cb[n] * ldb, x);
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[b][n][t] = x[t];
      }
    } else {
#pragma unroll
      for (int n = 0; n < NC; ++n)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const T x = (T)Bb[src[t] + cb[n] * ldb];
          acc[b][n][t] = r0 + t < m ? x : T(0);
        }
    }
  }
  store_panel(0, 0, 0, v);
  __syncthreads();  // also: B may alias X, all loads of the chunk precede any store

  auto step = [&](int sweep, int k, int buf) {
    // operands of block b: the lane's four K-steps
    if constexpr (BF) {
      const s4* fr = reinterpret_cast<const s4*>(frag[buf]) + lane;
      s4 xp[NC];
#pragma unroll
      for (int n = 0; n < NC; ++n) {
        T x[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) x[s] = acc[k][n][s];
        acc[k][n] = mma_bf16(fr[k * 64], pack_bf16(x), vzero<V>());
#pragma unroll
        for (int s = 0; s < 4; ++s) x[s] = acc[k][n][s];
        xp[n] = pack_bf16(x);
      }
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (sweep == 0 ? b > k && b < nbk : b < k) {
          const s4 av = fr[b * 64];
#pragma unroll
          for (int n = 0; n < NC; ++n) acc[b][n] = mma_bf16(av, xp[n], acc[b][n]);
        }
    } else {
      const T* fr = frag[buf] + lane * 4;
      T av[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) av[s] = fr[k * 256 + s];
#pragma unroll
      for (int n = 0; n < NC; ++n) {
        V x = vzero<V>();
#pragma unroll
        for (int s = 0; s < 4; ++s) x = M::mma(av[s], acc[k][n][s], x);
        acc[k][n] = x;
      }
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (sweep == 0 ? b > k && b < nbk : b < k) {
#pragma unroll
          for (int s = 0; s < 4; ++s) av[s] = fr[b * 256 + s];
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int n = 0; n < NC; ++n) acc[b][n] = M::mma(av[s], acc[k][n][s], acc[b][n]);
        }
    }
  };
  // unrolled: every block index is a compile-time constant; steps past the
  // last block of a short leaf are skipped (uniform).  Step k of the downward
  // sweep reads buffer k & 1, of the upward one (k + 1) & 1.
#pragma unroll
  for (int k = 0; k < NB; ++k)
    if (k < nbk) {
      const bool more = k + 1 < nbk;
      if (more) load_panel(0, k + 1, v);
      else load_panel(1, nbk - 1, v);
      step(0, k, k & 1);
      if (more) store_panel((k + 1) & 1, 0, k + 1, v);
      else store_panel((k + 1) & 1, 1, nbk - 1, v);
      __syncthreads();
    }
#pragma unroll
  for (int k = NB - 1; k >= 0; --k)
    if (k < nbk) {
      if (k > 0) load_panel(1, k - 1, v);
      step(1, k, (k + 1) & 1);
      if (k > 0) {
        store_panel(k & 1, 1, k - 1, v);
        __syncthreads();
      }
    }

  // store (the adjoint scatters rows through the permutation)
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    if (b >= nbk) continue;
    const int r0 = 16 * b + 4 * lq;
    int dst[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int rc = min(r0 + t, m - 1);
      dst[t] = TRANS ? pm[rc] : rc;
    }
    if (__all(dst[1] == dst[0] + 1 && dst[2] == dst[0] + 2 && dst[3] == dst[0] + 3)) {
      typedef T V4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));
#pragma unroll
      for (int n = 0; n < NC; ++n)
        if (c0 + 16 * n + li < ncols) {
          V4 x;
#pragma unroll
          for (int t = 0; t < 4; ++t) x[t] = acc[b][n][t];
          *reinterpret_cast<V4*>(Xb + dst[0] + cb[n] * ldx) = x;
        }
    } else {
#pragma unroll
      for (int n = 0; n < NC; ++n)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (c0 + 16 * n + li < ncols && r0 + t < m) Xb[dst[t] + cb[n] * ldx] = acc[b][n][t];
    }
  }
}

template <typename T, typename S>
hipError_t launch_leaf_trsm(hipStream_t s, int trans, int nleaf, int ldl, const int64_t* d_leaf_off, const T* lu,
                            int64_t lul, int inplace, const int32_t* perm, const T* dinv, const S* B, int64_t ldb,
                            T* X, int64_t ldx, int ncols, int64_t gsb, int64_t gsx, int bf) {
  if (nleaf == 0 || ncols == 0) return hipSuccess;
  if (ldl % 16 || ldl > 256) return hipErrorInvalidValue;
  if (inplace ? lul < ldl : lul != ldl) return hipErrorInvalidValue;
  // waves with columns of their own: leaves up to 128 rows and more than 64
  // columns.  There trsm_kernel's waves have two row blocks each at most and a
  // barrier for every few MFMAs (N = 2^17, leaf 128, FP32, 240 columns: 236 us
  // against 152; leaf 64, 96 columns: 30 against 18; uneven leaves around 100
  // rows, FP64, 340 columns: 483 against 405).  With 256 rows the accumulators
  // leave two workgroups per CU and the barriers are in the open (FP64, 384
  // columns: 5.4 against 7.2 ms), and few columns leave waves without any (32
  // adjoint columns on leaf 128: 137 against 217 us).
  const bool wide = ldl <= 128 && ncols > 64;
  // blocks of at most 64 rows: one 16-row block per wave; else four blocks per
  // wave and 32 columns
  const int nq = ldl <= 64 ? 1 : 4;
  // 4-byte elements: 64-column chunks of the leaf blocks hold as many
  // accumulator registers as 32 FP64 columns (four workgroups per CU), with
  // half the chunks and half the re-reads of each leaf's factors
  const int chunk = sizeof(T) == 4 && nq == 4 && ncols > 32 ? 64 : 32;
  // two column blocks a wave with 4-byte elements or up to 64 rows
  const int nc = sizeof(T) == 4 || nq == 1 ? 2 : 1;
  const int cw = wide ? 64 * nc : ncols <= 16 ? 16 : nq == 1 ? 64 : chunk;
  const int nchunks = (ncols + cw - 1) / cw;
  const int64_t grid = (int64_t)nleaf * nchunks;
  if (grid > 0x7fffffff) return hipErrorInvalidValue;
  // bfloat16 operands (FP32 factors and accumulation): the leaf solve of a
  // BF16 factorization, leaves of more than 64 rows
  const bool use_bf = sizeof(T) == 4 && bf && !trans && nq == 4;
#define HODLR_TS_L(KERNEL, THREADS)                                                                               \
  hipLaunchKernelGGL((KERNEL), dim3((unsigned)grid), dim3(THREADS), 0, s, ldl, d_leaf_off, lu, lul, inplace, perm,  \
                     dinv, B, ldb, X, ldx, ncols, nchunks, gsb, gsx)
#define HODLR_TS(TR, NW, NQ, NC, BFV) HODLR_TS_L((trsm_kernel<T, S, TR, NW, NQ, NC, BFV>), 64 * NW)
#define HODLR_TW(TR, NB, NC, BFV) HODLR_TS_L((trsm_wide_kernel<T, S, TR, NB, NC, BFV>), kTwThreads)
  // up to 64 rows: 4 waves, one block each; up to 256 rows: 4 waves with four
  // blocks each for wide right-hand sides, 8 waves with two each for narrow ones
#define HODLR_TS_W(TR)                                    \
  if (wide) {                                             \
    if (nq == 1) HODLR_TW(TR, 4, 2, false);               \
    else HODLR_TW(TR, 8, (sizeof(T) == 4 ? 2 : 1), false); \
  } else if (nq == 1) {                                   \
    if (cw == 64) HODLR_TS(TR, 4, 1, 4, false);           \
    else HODLR_TS(TR, 4, 1, 1, false);                    \
  } else if (cw == 64) {                                  \
    if constexpr (sizeof(T) == 4) HODLR_TS(TR, 4, 4, 4, false); \
  } else if (cw == 32) {                                  \
    HODLR_TS(TR, 4, 4, 2, false);                         \
  } else {                                                \
    HODLR_TS(TR, 8, 2, 1, false);                         \
  }
  if (use_bf) {
    if constexpr (sizeof(T) == 4) {
      if (wide) HODLR_TW(0, 8, 2, true);
      else if (cw == 64) HODLR_TS(0, 4, 4, 4, true);
      else if (cw == 32) HODLR_TS(0, 4, 4, 2, true);
      else HODLR_TS(0, 8, 2, 1, true);
    }
  } else if (trans) {
    HODLR_TS_W(1)
  } else {
    HODLR_TS_W(0)
  }
#undef HODLR_TS_W
#undef HODLR_TW
#undef HODLR_TS
#undef HODLR_TS_L
  return hipGetLastError();
}

template hipError_t launch_leaf_trsm<double, double>(hipStream_t, int, int, int, const int64_t*, const double*,
                                                     int64_t, int, const int32_t*, const double*, const double*,
                                                     int64_t, double*, int64_t, int, int64_t, int64_t, int);
template hipError_t launch_leaf_trsm<float, double>(hipStream_t, int, int, int, const int64_t*, const float*,
                                                    int64_t, int, const int32_t*, const float*, const double*,
                                                    int64_t, float*, int64_t, int, int64_t, int64_t, int);
template hipError_t launch_leaf_trsm<float, float>(hipStream_t, int, int, int, const int64_t*, const float*,
                                                   int64_t, int, const int32_t*, const float*, const float*,
                                                   int64_t, float*, int64_t, int, int64_t, int64_t, int);

}  // namespace hodlr
