// Fused per-level pass over row tiles (Alg. "a:gpuf" batched GEMMs and
// Alg. "a:gpus" batched GEMMs, restated on row tiles):
//
//   update : Z(tile, 0:nz) -= A1(tile, 0:ka) * W_node(0:ka, 0:nz)
//            factor: Y_big(I_a, 1:R_l) -= Y_a W_a        (eq. "e:node2")
//            solve : x(I_a) -= Y_a w_a                    (eq. "e:node4")
//   product: P_tile(0:kb, 0:nz) = B1(tile, 0:kb)^T * Z(tile, 0:nz)
//            the partial sums of V^T Y (eq. "e:node1" right side and the T
//            blocks of eq. "e:k") or of V^T x (eq. "e:node3") for the next level
//
// Two kernels, both 256 threads = 4 waves on a tile of <= 256 rows and a chunk
// of <= 64 columns of Z: level_pass_block_kernel for wide Z on shapes made of
// whole 16-row and 16-column blocks, level_pass_rows_kernel for everything
// else (launch_level_pass has the rule).
#include "mfma.h"

#include <algorithm>
#include <type_traits>

namespace hodlr {

constexpr int kLpThreads = 256;

// Rows of the accumulators.  A group of 16 RP rows (RP elements are 16 bytes)
// is RP MFMA blocks; register t of lane group lq in block h is row
// RP (4 t + lq) + h, so for each t a lane holds 16 contiguous bytes of its
// column and the four lane groups 64.  Lane li feeds rows
// RP row_of_lane(li) + h as MFMA A operands: 256 contiguous bytes over the 16.
template <typename T>
constexpr int kRp = 16 / (int)sizeof(T);
template <typename T>
__device__ __forceinline__ int row_of_lane(int li) {
  return sizeof(T) == 8 ? li : 4 * (li & 3) + (li >> 2);
}

// Resident workgroups per CU asked of the register allocator: a wave's part
// of Z takes 4 NCB accumulators (of 4 elements), the product NCB more.
template <typename T, int NCB, bool FULL>
constexpr int lp_occupancy() {
  return sizeof(T) == 8 ? (NCB >= 3 || (NCB == 2 && !FULL) ? 2 : 3) : (FULL ? 4 : 3);
}

// Row kernel (any shape).  Bound by memory latency: few MFMAs per byte for
// narrow Z, partial blocks for ragged trees; so it keeps whole parts of Z in
// registers and all operand loads wide and independent.  On an uneven tree
// (N = 102846, rank 37 .. 31, FP64) the passes of a factorization take 1.62 ms
// and those of a 3-column solve 0.25 ms (clamped element loads: 3.75 and
// 1.02 ms).  Workgroup = 4 waves on one tile and one chunk of
// columns of Z; a wave owns 64 rows of the tile and NCB 16-column blocks.  The
// waves stand WR x WC = 4 over rows x columns: tiles of more than 128 rows
// take 4 x 1, shorter ones 2 x 2 or 1 x 4, so that no wave is left without
// rows.  A wave holds its part of Z in accumulators with lanes on columns (see
// kRp): Z and B1 move as 16-byte accesses, and register t of an accumulator
// is directly the B operand of one 4-row K-step of the product, whose A
// operand is B1 read in the same layout, so neither passes through LDS.  The
// update takes A1 straight from memory and W from LDS in fragment order (one
// read gives a lane its values of four K-steps).  Only the waves' partial
// products meet in LDS, 16 rows of P at a time, and are summed in a fixed
// order.  BF (4-byte Z): four consecutive K-steps of a lane are one
// 16 x 16 x 16 bfloat16 MFMA; W is packed when staged, A1, B1 and Z once per
// use.
//
// FULL: the tile heights are multiples of 64, so a wave has 64 rows or none;
// otherwise a wave with fewer reads its last row in the place of those past
// the end, never stores them, and zeroes them in B1 and Z before the product (an
// infinity in the last row would make the sums of its column NaN).  K is padded with zero rows of
// W (A1 re-reads its last column).  Columns past nz and B1 columns past kb
// re-read the last one; their results are not stored.
//
// CPL (one chunk of up to 16 columns): W is not read but formed here, from the
// parent's K^{-1} (CPL = 2: its transpose) and the children's products: every
// workgroup sums its parent's items (a node's tile partials, in order), and wave
// w forms the 16-row block w of its own child's rows, in the layout and order
// of couple_apply_kernel.  That repeats a few thousand multiply-adds per tile
// and saves the launches that would form W and, up to kCplLoads item columns,
// the reduction before them: a launch is 4 us, as long as a narrow pass over a
// small system (N = 4096, one vector: 19 launches and 83 us without, 8 and
// 51 us with).
template <typename T>
struct CoupleArgs {
  const T* Kinv = nullptr;  // of the level's first parent, kp x kp each
  int kp = 0;
  const T* items = nullptr;  // r x nz each, child c's: start[c] .. start[c + 1]
  const int32_t* start = nullptr;
};

//
// NT: threads; one column block (narrow Z) on tiles up to 128 or 64 rows takes
// two waves or one, as waves without rows would only hold places of the CU.
// Products of N = 131072 rows in tiles of 128 with 240 FP32 columns, one
// vector: 43 us (four waves: 57).
template <typename TZ, typename SA, typename SB, int WC, int NCB, bool FULL, bool BF, int CPL = 0, int NT = kLpThreads>
__global__ __launch_bounds__(NT, (lp_occupancy<TZ, NCB, FULL>())) void level_pass_rows_kernel(
    const Tile* __restrict__ tiles, int zchunks, int c_base, int bchunks, int kbc, TZ* Z, int64_t ldz, int nz,
    const SA* A1, int64_t lda, int ka, const TZ* __restrict__ W, int64_t w_ld, int64_t w_pstride, int node_shift,
    const SB* __restrict__ B1, int64_t ldb, int kb_total, TZ* __restrict__ P, GroupStrides gs, int red_off,
    CoupleArgs<TZ> cpl) {
  static_assert(CPL == 0 || (WC == 1 && NCB == 1 && !BF), "the fused coupling solve is for one narrow chunk");
  using M = Mfma<TZ>;
  using V = typename M::V;
  constexpr int WR = NT / 64 / WC;
  constexpr int kCw = 16 * NCB * WC;  // columns of a chunk
  constexpr int kWc = 16 * NCB;       // columns of a wave
  constexpr int RP = kRp<TZ>, kGr = 16 * RP, NG = 4 / RP;  // rows of a group, groups of a wave
  // one column block: operands of the next step are in flight while this one
  // computes (wider parts need the registers and hide latency by their MFMAs)
  constexpr bool PF = NCB == 1;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  TZ* Ws = reinterpret_cast<TZ*>(smem_raw);

  const int lid = (int)xcd_remap(blockIdx.x, gridDim.x);  // grid < 2^31: 32-bit index math
  const int bchunk = lid % bchunks;
  const int zchunk = (lid / bchunks) % zchunks;
  const int tile = lid / (bchunks * zchunks);
  const Tile tl = tiles[tile];
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = w / WC, wc = w % WC;
  const int c0 = c_base + zchunk * kCw;
  const int wr0 = 64 * wr;                                        // first tile row of this wave
  const int wrows = tl.nrows - wr0;                               // its rows (64 and more: 64; <= 0: none)
  const int ng = (ka + 15) >> 4;                                  // K groups of the update
  const int k0 = bchunk * kbc, k1 = min(kb_total, k0 + kbc);      // columns of B1

  // W chunk to LDS, negated: element (k, c) of the chunk, k = 16 g + 4 q + s, in slot s of
  // lane 16 q + c % 16 of fragment (g, c / 16)
  if constexpr (CPL > 0) {
    const int nd = tl.node >> node_shift, half = nd & 1, nt = ng, r = ka;  // r % 8 = 0
    // K^{-1} rows of this wave's block (half r + 16 w + row), all columns
    const TZ* Kg = cpl.Kinv + (int64_t)(nd >> 1) * cpl.kp * cpl.kp;
    const int row = half * r + min(16 * w + (sizeof(TZ) == 8 ? 4 * (li & 3) + (li >> 2) : li), r - 1);
    TZ kv[8][4];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (w < nt && q < 2 * nt) {
        const int kh = q >= nt, i0 = 16 * (kh ? q - nt : q) + 4 * lq;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int k = kh * r + min(i0 + t, r - 1);
          kv[q][t] = CPL == 2 ? Kg[k + row * cpl.kp] : Kg[row + k * cpl.kp];
        }
      }
    // the children's product sums as B fragments: group q, lane, 4 rows
    TZ* Ts = reinterpret_cast<TZ*>(smem_raw) + (red_off / sizeof(TZ)) * 2;
    for (int e = tid; e < 2 * nt * 64; e += NT) {
      const int q = e >> 6, h = q >= nt, c = e & 15, i0 = 16 * (h ? q - nt : q) + 4 * ((e >> 4) & 3);
      TZ sum[4] = {TZ(0), TZ(0), TZ(0), TZ(0)};
      if (c < nz && i0 < r) {
        const int child = (nd & ~1) + h, i1 = cpl.start[child + 1];
        for (int it = cpl.start[child], first = it; it < i1; it += 4) {
          TZ v[4][4];  // four items' loads in flight
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const TZ* col = cpl.items + ((int64_t)min(it + u, i1 - 1) * nz + c) * r;
            load_run(col + i0, v[u]);
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (it + u < i1) {
#pragma unroll
              for (int t = 0; t < 4; ++t) sum[t] = it + u == first ? v[u][t] : sum[t] + v[u][t];
            }
        }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) Ts[e * 4 + t] = sum[t];
    }
    __syncthreads();
    if (w < nt) {
      V acc = vzero<V>();
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (q < 2 * nt) {
#pragma unroll
          for (int t = 0; t < 4; ++t) acc = M::mma(kv[q][t], Ts[(q * 64 + lane) * 4 + t], acc);
        }
#pragma unroll
      for (int t = 0; t < 4; ++t) Ws[(w * 64 + lane) * 4 + t] = 16 * w + 4 * lq + t < r ? -acc[t] : TZ(0);
    }
  } else if (ka > 0) {
    const int nd = tl.node >> node_shift;
    const TZ* Wn = W + (int64_t)(nd >> 1) * w_pstride + (int64_t)(nd & 1) * ka;
    for (int e = tid; e < ng * 4 * kCw; e += NT) {
      const int q = e & 3, c = (e >> 2) % kCw, g = e / (4 * kCw);
      const int k = 16 * g + 4 * q;
      const TZ* src = Wn + (int64_t)min(c0 + c, nz - 1) * w_ld;
      TZ v[4];
      if (k + 4 <= ka) {
        load_run(src + k, v);
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const TZ x = src[min(k + s, ka - 1)];
          v[s] = k + s < ka ? x : TZ(0);
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) v[s] = -v[s];
      const int slot = (g * (kCw / 16) + (c >> 4)) * 64 + 16 * q + (c & 15);
      if constexpr (BF) {
        reinterpret_cast<s4*>(Ws)[slot] = pack_bf16(v);
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) Ws[slot * 4 + s] = v[s];
      }
    }
  }

  // the wave's work, with 64 rows (whole) or fewer
  auto body = [&](auto whole_t) {
    constexpr bool whole = decltype(whole_t)::value;
    const int nrg = whole ? NG : FULL ? 0 : min(NG, max(0, (wrows + kGr - 1) / kGr));  // row groups
    const int last = max(wrows - 1, 0);
    // RP rows of a column from row r of the wave's part
    auto load_rows = [&](const auto* col, int r, TZ (&v)[RP]) {
      if constexpr (whole) {
        load_run(col + r, v);
      } else {
#pragma unroll
        for (int h = 0; h < RP; ++h) v[h] = (TZ)col[min(r + h, last)];
      }
    };
    // A1(row, 16 g + 4 lq + s) of the lane's rows
    const SA* Aw = A1 + (ka > 0 ? group_row(tl.row0, gs.a) + wr0 : 0);
    auto load_a = [&](int g, TZ (&av)[4][4]) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const SA* col = Aw + (int64_t)min(16 * g + 4 * lq + s, ka - 1) * lda;
#pragma unroll
        for (int rg = 0; rg < NG; ++rg) {
          if (rg >= nrg) continue;
          TZ v[RP];
          load_rows(col, kGr * rg + RP * row_of_lane<TZ>(li), v);
#pragma unroll
          for (int h = 0; h < RP; ++h) av[RP * rg + h][s] = v[h];
        }
      }
    };
    // B1(rows of the lane, kr0 + li), zero in rows past the tile
    const SB* Bw = B1 + (kb_total > 0 ? group_row(tl.row0, gs.b) + wr0 : 0);
    auto load_b = [&](int kr0, TZ (&bv)[4][4]) {
      const SB* col = Bw + (int64_t)min(kr0 + li, kb_total - 1) * ldb;
#pragma unroll
      for (int rg = 0; rg < NG; ++rg) {
        if (rg >= nrg) continue;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int r = kGr * rg + 4 * RP * t + RP * lq;
          TZ v[RP];
          load_rows(col, r, v);
#pragma unroll
          for (int h = 0; h < RP; ++h) bv[RP * rg + h][t] = whole || r + h <= last ? v[h] : TZ(0);
        }
      }
    };

    TZ* Zw = Z + group_row(tl.row0, gs.z) + wr0;
    int64_t zcol[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) zcol[cb] = (int64_t)min(c0 + kWc * wc + 16 * cb + li, nz - 1) * ldz;
    V acc[4][NCB];
    TZ av[4][4];
    if (PF && ka > 0) load_a(0, av);
#pragma unroll
    for (int rg = 0; rg < NG; ++rg) {
      if (rg >= nrg) continue;
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          TZ v[RP];
          load_rows(Zw + zcol[cb], kGr * rg + 4 * RP * t + RP * lq, v);
#pragma unroll
          for (int h = 0; h < RP; ++h) acc[RP * rg + h][cb][t] = v[h];
        }
      }
    }

    if (ka > 0) {
      __syncthreads();  // W staged
#pragma unroll 1
      for (int g = 0; g < ng; ++g) {
        TZ an[4][4];
        if (PF) {
          if (g + 1 < ng) load_a(g + 1, an);
          else if (kb_total > 0) load_b(k0, an);
        } else {
          load_a(g, av);
        }
        if constexpr (BF) {
          s4 ap[4];
#pragma unroll
          for (int rb = 0; rb < 4; ++rb)
            if (rb < RP * nrg) ap[rb] = pack_bf16(av[rb]);
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) {
            const s4 wp = reinterpret_cast<const s4*>(Ws)[(g * (kCw / 16) + wc * NCB + cb) * 64 + lane];
#pragma unroll
            for (int rb = 0; rb < 4; ++rb)
              if (rb < RP * nrg) acc[rb][cb] = mma_bf16(ap[rb], wp, acc[rb][cb]);
          }
        } else {
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) {
            TZ wv[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) wv[s] = Ws[((g * (kCw / 16) + wc * NCB + cb) * 64 + lane) * 4 + s];
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
              for (int rb = 0; rb < 4; ++rb)
                if (rb < RP * nrg) acc[rb][cb] = M::mma(av[rb][s], wv[s], acc[rb][cb]);
          }
        }
        if (PF) {
#pragma unroll
          for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int s = 0; s < 4; ++s) av[rb][s] = an[rb][s];
        }
      }
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        if (c0 + kWc * wc + 16 * cb + li < nz) {
#pragma unroll
          for (int rg = 0; rg < NG; ++rg) {
            if (rg >= nrg) continue;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const int r = kGr * rg + 4 * RP * t + RP * lq;
              TZ* dst = Zw + zcol[cb] + r;
              if constexpr (whole) {
                typename Vec<TZ, RP>::type v;
#pragma unroll
                for (int h = 0; h < RP; ++h) v[h] = acc[RP * rg + h][cb][t];
                *reinterpret_cast<typename Vec<TZ, RP>::type*>(dst) = v;
              } else {
#pragma unroll
                for (int h = 0; h < RP; ++h)
                  if (r + h <= last) dst[h] = acc[RP * rg + h][cb][t];
              }
            }
          }
        }
      }
    } else if (PF) {
      load_b(k0, av);
    }

    if (kb_total > 0) {
      if constexpr (!whole) {
#pragma unroll
        for (int rg = 0; rg < NG; ++rg)
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int h = 0; h < RP; ++h)
              if (kGr * rg + 4 * RP * t + RP * lq + h > last) {
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb) acc[RP * rg + h][cb][t] = TZ(0);
              }
      }
      // 16 rows of P at a time; the waves' partials go to one of two LDS
      // buffers in turn (the second takes the place of W, which no wave reads
      // after the first barrier), so one barrier separates two steps
      TZ* red[2] = {reinterpret_cast<TZ*>(smem_raw + red_off), Ws};
      TZ* Pt = P + (int64_t)tile * kb_total * nz;
      s4 zp[BF ? 4 : 1][NCB];  // bfloat16: Z packed once
      if constexpr (BF) {
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
            if (rb < RP * nrg) {
              TZ v[4];
#pragma unroll
              for (int t = 0; t < 4; ++t) v[t] = acc[rb][cb][t];
              zp[rb][cb] = pack_bf16(v);
            }
      }
      int buf = 0;
#pragma unroll 1
      for (int kr0 = k0; kr0 < k1; kr0 += 16) {
        TZ bn[4][4];
        if (!PF) load_b(kr0, av);
        else if (kr0 + 16 < k1) load_b(kr0 + 16, bn);
        V pacc[NCB];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) pacc[cb] = vzero<V>();
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
          if (rb >= RP * nrg) continue;
          if constexpr (BF) {
            const s4 bp = pack_bf16(av[rb]);
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) pacc[cb] = mma_bf16(bp, zp[rb][cb], pacc[cb]);
          } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
              for (int cb = 0; cb < NCB; ++cb) pacc[cb] = M::mma(av[rb][t], acc[rb][cb][t], pacc[cb]);
          }
        }
        if (PF) {
#pragma unroll
          for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int t = 0; t < 4; ++t) av[rb][t] = bn[rb][t];
        }
        // red[buf]: [WR][16 rows of P][kCw]
        TZ* rd = red[buf];
        buf ^= 1;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
          for (int t = 0; t < 4; ++t) rd[(wr * 16 + M::crow(lq, t)) * kCw + kWc * wc + 16 * cb + li] = pacc[cb][t];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < (16 * kCw + NT - 1) / NT; ++u) {
          const int e = tid + u * NT;
          const int kr = kr0 + (e & 15), c = e >> 4;
          if ((16 * kCw % NT == 0 || e < 16 * kCw) && kr < k1 && c0 + c < nz) {
            TZ sum = rd[(e & 15) * kCw + c];
#pragma unroll
            for (int x = 1; x < WR; ++x) sum += rd[(x * 16 + (e & 15)) * kCw + c];
            Pt[kr + (int64_t)(c0 + c) * kb_total] = sum;
          }
        }
      }
    }
  };
  // both sides pass the same barriers
  if (wrows >= 64) body(std::true_type());
  else body(std::false_type());
}

// Blocked kernel for wide Z without bfloat16 (tile heights, ka and kb
// multiples of 16, whole 16-column blocks): per (tile, 64 columns), wave w on
// rows 64 w .. of the tile in 16 RP-row blocks.  The update is computed
// transposed, Z^T -= W^T A1^T, so that the 16 lanes of a row group hold
// consecutive rows of one column of Z: every load and store of Z and A1
// covers whole 128-byte lines of four columns, addressed as a lane-uniform
// base plus one 32-bit lane offset (buffer addressing).  For the product the
// updated block is turned around through a per-wave LDS buffer, and B1 is
// loaded coalesced and turned around the same way.  RP = 2 (4-byte Z, tile
// heights multiples of 32): each lane holds two consecutive rows, loaded and
// stored as one 8-byte access; the even and the odd rows form two 16-row MFMA
// blocks (the product's sum over rows does not depend on their order).
constexpr int kZtLd = 17;  // padded row length of the per-wave 16 x 16 turn-around buffer

template <typename TZ, typename SA, typename SB, int MB, int NKS, int NCB, int RP, bool BF = false>
__global__ __launch_bounds__(kLpThreads, (MB > 2 || NKS > 8) ? 2 : 3) void level_pass_block_kernel(
    const Tile* __restrict__ tiles, int zchunks, int c_base, int bchunks, TZ* Z, int64_t ldz, int nz, const SA* __restrict__ A1,
    int64_t lda, const TZ* __restrict__ W, int64_t w_ld, int64_t w_pstride, int node_shift,
    const SB* __restrict__ B1, int64_t ldb, int kb_total, TZ* __restrict__ P, GroupStrides gs) {
  using M = Mfma<TZ>;
  using V = typename M::V;
  constexpr int ka = 4 * NKS;
  constexpr int kb = 16 * MB;  // B1 columns of this chunk (kb_total is a multiple of 16)
  constexpr int kCw = 16 * NCB;  // Z columns of a chunk
  constexpr int kBtLd = 16 * MB + 1;
  constexpr int kWave = 16 * kZtLd + 16 * kBtLd;
  constexpr bool prod = MB > 0;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  TZ* Ws = reinterpret_cast<TZ*>(smem_raw);   // W chunk [ka][kCw]
  TZ* red = reinterpret_cast<TZ*>(smem_raw);  // end of the product: [2][kb][kCw]

  const int lid = (int)xcd_remap(blockIdx.x, gridDim.x);  // grid < 2^31: 32-bit index math
  const int bchunk = lid % bchunks;
  const int zchunk = (lid / bchunks) % zchunks;
  const int tile = lid / (bchunks * zchunks);
  const Tile tl = tiles[tile];
  const int nrows = tl.nrows;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: addresses stay scalar
  const int c0 = c_base + zchunk * kCw;
  const int wr0 = 64 * w;
  const int nrb = max(0, min(4 / RP, (nrows - wr0) >> (RP == 2 ? 5 : 4)));  // 16 RP-row blocks of this wave
  const int kc0 = bchunk * 64;
  TZ* zt = Ws + kCw * ka + w * kWave;
  TZ* bt = zt + 16 * kZtLd;

  if (NKS > 0) {
    const int nd = tl.node >> node_shift;
    const TZ* Wn = W + (int64_t)(nd >> 1) * w_pstride + (int64_t)(nd & 1) * ka;
    for (int e = tid; e < kCw * ka; e += kLpThreads) {
      const int c = e % kCw, k = e / kCw;
      const TZ v = Wn[k + (int64_t)(c0 + c) * w_ld];
      // BF: as the update's packed A operands, element (k, c) to group k / 16, block
      // c / 16, lane (k % 4, c % 16), slot (k / 4) % 4
      if constexpr (BF)
        reinterpret_cast<__bf16*>(Ws)[((((k >> 4) * NCB + (c >> 4)) * 4 + (k & 3)) * 16 + (c & 15)) * 4 +
                                      ((k >> 2) & 3)] = (__bf16)v;
      else
        Ws[e] = v;
    }
  }

  // first row of this wave in each operand (rows inside a tile are contiguous)
  const auto zr = buf_rsrc(Z + group_row(tl.row0, gs.z) + wr0 + (int64_t)c0 * ldz);
  const auto ar = buf_rsrc(NKS > 0 ? A1 + group_row(tl.row0, gs.a) + wr0 : A1);  // A1 / B1 are null when unused
  const auto br = buf_rsrc(prod ? B1 + group_row(tl.row0, gs.b) + wr0 + (int64_t)kc0 * ldb : B1);
  const uint32_t zl = (uint32_t)(RP * li + (int64_t)M::crow_l(lq) * ldz) * (uint32_t)sizeof(TZ);
  const uint32_t al = (uint32_t)(RP * li + (int64_t)lq * lda) * (uint32_t)sizeof(SA);
  const uint32_t bl = (uint32_t)(RP * li + (int64_t)lq * ldb) * (uint32_t)sizeof(SB);
  constexpr uint32_t kRbRows = 16 * RP;  // rows of one row block
  // Z(16 rb + li, c0 + 16 cb + crow(lq, t)) is register t of the Z^T accumulator
  // block cb (RP = 2: rows 32 rb + 2 li + h of block h)
  auto zso = [&](int cb, int t) -> uint32_t {
    return (uint32_t)((int64_t)(16 * cb + M::crow_u(t)) * ldz * (int64_t)sizeof(TZ));
  };
  auto zvo = [&](int rb) -> uint32_t { return zl + kRbRows * (uint32_t)rb * (uint32_t)sizeof(TZ); };
  auto load_z = [&](int rb, V (&d0)[NCB], V (&d1)[NCB]) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        TZ v0, v1 = TZ(0);
        if (RP == 2) Buf2<TZ>::load(zr, zvo(rb), zso(cb, t), v0, v1);
        else v0 = Buf<TZ>::load(zr, zvo(rb), zso(cb, t));
        d0[cb][t] = v0;
        d1[cb][t] = v1;
      }
  };
  // B operand of the update: -A1(row, 4 ks + lq) for the lane's row(s)
  auto load_a = [&](int rb, TZ (&d0)[NKS > 0 ? NKS : 1], TZ (&d1)[NKS > 0 ? NKS : 1]) {
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const uint32_t vo = al + kRbRows * (uint32_t)rb * (uint32_t)sizeof(SA);
      const uint32_t so = (uint32_t)((int64_t)(4 * ks) * lda * (int64_t)sizeof(SA));
      SA x0, x1 = SA(0);
      if (RP == 2) Buf2<SA>::load(ar, vo, so, x0, x1);
      else x0 = Buf<SA>::load(ar, vo, so);
      d0[ks] = -(TZ)x0;
      d1[ks] = -(TZ)x1;
    }
  };
  // B1(row, kc0 + 4 i + lq); the last B1 chunk may hold fewer than kb
  // columns (a multiple of 16): the others read column kc0 and are zeroed
  const int kbc = prod ? min(kb, kb_total - kc0) : 0;
  auto load_b = [&](int rb, TZ (&d0)[MB > 0 ? 4 * MB : 1], TZ (&d1)[MB > 0 ? 4 * MB : 1]) {
#pragma unroll
    for (int i = 0; i < 4 * MB; ++i) {
      const bool ok = 4 * i < kbc;  // uniform
      const uint32_t vo = bl + kRbRows * (uint32_t)rb * (uint32_t)sizeof(SB);
      const uint32_t so = (uint32_t)((int64_t)(ok ? 4 * i : 0) * ldb * (int64_t)sizeof(SB));
      SB x0, x1 = SB(0);
      if (RP == 2) Buf2<SB>::load(br, vo, so, x0, x1);
      else x0 = Buf<SB>::load(br, vo, so);
      d0[i] = ok ? (TZ)x0 : TZ(0);
      d1[i] = ok ? (TZ)x1 : TZ(0);
    }
  };

  V pacc[MB > 0 ? MB : 1][NCB];
#pragma unroll
  for (int mb = 0; mb < (MB > 0 ? MB : 1); ++mb)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) pacc[mb][cb] = vzero<V>();

  // update of one 16-row MFMA block, and its contribution to the product
  auto update = [&](V (&acc)[NCB], const TZ (&acur)[NKS > 0 ? NKS : 1]) {
    if constexpr (BF) {  // four K-steps as one MFMA (NKS is a multiple of 4)
      const s4* Wp = reinterpret_cast<const s4*>(Ws);
#pragma unroll
      for (int g = 0; g < NKS / 4; ++g) {
        TZ av[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) av[j] = acur[4 * g + j];
        const s4 ap = pack_bf16(av);
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) acc[cb] = mma_bf16(Wp[((g * NCB + cb) * 4 + lq) * 16 + li], ap, acc[cb]);
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
          acc[cb] = M::mma(Ws[(4 * ks + lq) * kCw + 16 * cb + li], acur[ks], acc[cb]);
    }
  };
  auto stage_b = [&](const TZ (&bcur)[MB > 0 ? 4 * MB : 1]) {
#pragma unroll
    for (int i = 0; i < 4 * MB; ++i) bt[li * kBtLd + 4 * i + lq] = bcur[i];
  };
  auto product = [&](const V (&acc)[NCB]) {
    // P(j, c) += sum_r B1(r, j) Z(r, c); K-step kk takes rows 4 kk + lq; the
    // turned-around B1 block is read into registers once
    TZ bv[4][MB > 0 ? MB : 1];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) bv[kk][mb] = bt[(4 * kk + lq) * kBtLd + 16 * mb + li];
    s4 bp[BF && MB > 0 ? MB : 1];  // bfloat16: packed once for every Z block
    if constexpr (BF) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        TZ v[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) v[kk] = bv[kk][mb];
        bp[mb] = pack_bf16(v);
      }
    }
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
      for (int t = 0; t < 4; ++t) zt[li * kZtLd + M::crow(lq, t)] = acc[cb][t];
      TZ zv[4];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) zv[kk] = zt[(4 * kk + lq) * kZtLd + li];
      if constexpr (BF) {
        const s4 zp = pack_bf16(zv);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) pacc[mb][cb] = mma_bf16(bp[mb], zp, pacc[mb][cb]);
      } else {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) pacc[mb][cb] = M::mma(bv[kk][mb], zv[kk], pacc[mb][cb]);
      }
    }
  };

  if (NKS > 0) __syncthreads();  // W chunk staged
  // no software prefetch: latency is hidden by the other resident waves
#pragma unroll 1
  for (int rb = 0; rb < nrb; ++rb) {
    V acc0[NCB], acc1[NCB];
    TZ a0[NKS > 0 ? NKS : 1], a1[NKS > 0 ? NKS : 1];
    TZ b0[MB > 0 ? 4 * MB : 1], b1[MB > 0 ? 4 * MB : 1];
    load_z(rb, acc0, acc1);
    if (NKS > 0) load_a(rb, a0, a1);
    if (prod) {
      load_b(rb, b0, b1);
      stage_b(b0);
    }
    if (NKS > 0) {
      update(acc0, a0);
      if (RP == 2) update(acc1, a1);
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          if (RP == 2) Buf2<TZ>::store(acc0[cb][t], acc1[cb][t], zr, zvo(rb), zso(cb, t));
          else Buf<TZ>::store(acc0[cb][t], zr, zvo(rb), zso(cb, t));
        }
    }
    if (prod) {
      product(acc0);
      if (RP == 2) {
        stage_b(b1);  // after the even block's reads of bt (in order within the wave)
        product(acc1);
      }
    }
  }

  if (prod) {
    // partial products of the four waves, summed in the fixed order (w0 + w2) + (w1 + w3)
    // through a two-slot LDS buffer that reuses the W chunk and turn-around space
    __syncthreads();
    if (w < 2) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
          for (int t = 0; t < 4; ++t)
            red[(w * kb + 16 * mb + M::crow(lq, t)) * kCw + 16 * cb + li] = pacc[mb][cb][t];
    }
    __syncthreads();
    if (w >= 2) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            TZ* r = red + ((w - 2) * kb + 16 * mb + M::crow(lq, t)) * kCw + 16 * cb + li;
            *r = *r + pacc[mb][cb][t];
          }
    }
    __syncthreads();
    TZ* Pt = P + (int64_t)tile * kb_total * nz;
    for (int e = tid; e < kb * kCw; e += kLpThreads) {
      const int kr = e % kb, cw = e / kb;
      if (kr < kbc)
        Pt[(kc0 + kr) + (int64_t)(c0 + cw) * kb_total] = red[kr * kCw + cw] + red[(kb + kr) * kCw + cw];
    }
  }
}


template <typename TZ, typename SA, typename SB, int WC, int NCB, bool FULL, bool BF, int NT = kLpThreads>
static hipError_t launch_rows_part(hipStream_t s, int ntiles, int zchunks, int c_base, int bchunks, int kbc,
                                   const Tile* tiles, TZ* Z, int64_t ldz, int nz, const SA* A1, int64_t lda, int ka,
                                   const TZ* W, int64_t w_ld, int64_t w_pstride, int node_shift, const SB* B1,
                                   int64_t ldb, int kb, TZ* P, GroupStrides gs) {
  if (zchunks == 0) return hipSuccess;
  constexpr int WR = NT / 64 / WC, kCw = 16 * NCB * WC;
  const size_t red = kb > 0 ? sizeof(TZ) * WR * 16 * kCw : 0;
  const size_t wsz = std::max(red, (BF ? 2 : sizeof(TZ)) * (size_t)kCw * ((ka + 15) & ~15));
  const int64_t grid = (int64_t)ntiles * zchunks * bchunks;
  if (grid > 0x7fffffff) return hipErrorInvalidValue;
  auto k = level_pass_rows_kernel<TZ, SA, SB, WC, NCB, FULL, BF, 0, NT>;
  hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(wsz + red));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(NT), wsz + red, s, tiles, zchunks, c_base, bchunks, kbc, Z,
                     ldz, nz, A1, lda, ka, W, w_ld, w_pstride, node_shift, B1, ldb, kb, P, gs, (int)wsz, CoupleArgs<TZ>());
  return hipGetLastError();
}

// Columns c_base .. nz of Z in chunks of 64, then the rest as one narrower
// chunk, so that (up to 15 columns) no wave works on columns that do not exist.
template <typename TZ, typename SA, typename SB, int WC, bool FULL, bool BF>
static hipError_t launch_rows_chunks(hipStream_t s, int ntiles, int c_base, const Tile* tiles, TZ* Z, int64_t ldz,
                                     int nz, const SA* A1, int64_t lda, int ka, const TZ* W, int64_t w_ld,
                                     int64_t w_pstride, int node_shift, const SB* B1, int64_t ldb, int kb, TZ* P,
                                     GroupStrides gs) {
  // product-only passes have no update to repeat: their B1 columns are split
  // over workgroups too
  const int kbc = ka > 0 ? std::max(kb, 1) : 64;
  const int bchunks = kb > 0 ? (kb + kbc - 1) / kbc : 1;
  const int n64 = (nz - c_base) / 64, rest = ((nz - c_base) % 64 + 15) / 16;
  hipError_t e = hipSuccess;
#define HODLR_LPR(NCBV, CHUNKS, BASE)                                                                                \
  e = launch_rows_part<TZ, SA, SB, WC, NCBV, FULL, BF>(s, ntiles, CHUNKS, BASE, bchunks, kbc, tiles, Z, ldz, nz, A1, \
                                                       lda, ka, W, w_ld, w_pstride, node_shift, B1, ldb, kb, P, gs)
  HODLR_LPR(4 / WC, n64, c_base);
  if (e != hipSuccess || rest == 0) return e;
  const int base = c_base + 64 * n64;
  if constexpr (WC == 1) {
    if (rest == 1) HODLR_LPR(1, 1, base);
    else if (rest == 2) HODLR_LPR(2, 1, base);
    else if (rest == 3) HODLR_LPR(3, 1, base);
    else HODLR_LPR(4, 1, base);
  } else if constexpr (WC == 2) {
    if (rest <= 2) HODLR_LPR(1, 1, base);
    else HODLR_LPR(2, 1, base);
  } else {
    HODLR_LPR(1, 1, base);
  }
#undef HODLR_LPR
  return e;
}

template <typename TZ, typename SA, typename SB, bool BF>
static hipError_t launch_rows(hipStream_t s, int ntiles, int c_base, const Tile* tiles, TileShape sh, TZ* Z,
                              int64_t ldz, int nz, const SA* A1, int64_t lda, int ka, const TZ* W, int64_t w_ld,
                              int64_t w_pstride, int node_shift, const SB* B1, int64_t ldb, int kb, TZ* P,
                              GroupStrides gs) {
#define HODLR_LPS(WCV)                                                                                             \
  return sh.mult(64) ? launch_rows_chunks<TZ, SA, SB, WCV, true, BF>(s, ntiles, c_base, tiles, Z, ldz, nz, A1, lda, \
                                                                     ka, W, w_ld, w_pstride, node_shift, B1, ldb,   \
                                                                     kb, P, gs)                                     \
                     : launch_rows_chunks<TZ, SA, SB, WCV, false, BF>(s, ntiles, c_base, tiles, Z, ldz, nz, A1, lda, \
                                                                      ka, W, w_ld, w_pstride, node_shift, B1, ldb,  \
                                                                      kb, P, gs)
  // waves over columns only where every one of them has 16 columns of its own
  // (a projection of one vector on 128-row tiles: 333 us with two waves on the
  // same 16 columns, 231 us without)
  const int cols = nz - c_base;
  if constexpr (!BF) {
    if (cols <= 16 && sh.rows <= 128) {  // no more waves than rows
      const int kbc = ka > 0 ? std::max(kb, 1) : 64, bchunks = kb > 0 ? (kb + kbc - 1) / kbc : 1;
#define HODLR_LPN(FULLV, NTV)                                                                                        \
  return launch_rows_part<TZ, SA, SB, 1, 1, FULLV, BF, NTV>(s, ntiles, 1, c_base, bchunks, kbc, tiles, Z, ldz, nz, A1, \
                                                            lda, ka, W, w_ld, w_pstride, node_shift, B1, ldb, kb, P, gs)
      if (sh.rows <= 64) {
        if (sh.mult(64)) HODLR_LPN(true, 64);
        HODLR_LPN(false, 64);
      }
      if (sh.mult(64)) HODLR_LPN(true, 128);
      HODLR_LPN(false, 128);
#undef HODLR_LPN
    }
  }
  if (sh.rows <= 64 && cols > 32) HODLR_LPS(4);
  if (sh.rows <= 128 && cols > 16) HODLR_LPS(2);
  HODLR_LPS(1);
#undef HODLR_LPS
}

template <typename TZ, typename SA, typename SB, int MB, int NKS, int NCB, int RP, bool BF>
static hipError_t launch_block_part(hipStream_t s, int ntiles, int zchunks, int c_base, int nz, int bchunks,
                                    const Tile* tiles, TZ* Z, int64_t ldz, const SA* A1, int64_t lda, const TZ* W,
                                    int64_t w_ld, int64_t w_pstride, int node_shift, const SB* B1, int64_t ldb, int kb,
                                    TZ* P, GroupStrides gs) {
  if (zchunks == 0) return hipSuccess;
  constexpr int kCw = 16 * NCB;
  const size_t smem_main = sizeof(TZ) * (kCw * 4 * (size_t)NKS + 4 * (16 * kZtLd + 16 * (16 * MB + 1)));
  const size_t smem_red = MB > 0 ? sizeof(TZ) * 2 * 16 * MB * kCw : 0;
  const size_t smem = smem_main > smem_red ? smem_main : smem_red;
  const int64_t grid = (int64_t)ntiles * zchunks * bchunks;
  if (grid > 0x7fffffff) return hipErrorInvalidValue;
  auto k = level_pass_block_kernel<TZ, SA, SB, MB, NKS, NCB, RP, BF>;
  hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(kLpThreads), smem, s, tiles, zchunks, c_base, bchunks, Z, ldz, nz,
                     A1, lda, W, w_ld, w_pstride, node_shift, B1, ldb, kb, P, gs);
  return hipGetLastError();
}

// The first nblk 16-column blocks of Z: chunks of zw blocks (4; 2 or 1 where the
// leading dimension is too large for the offsets inside one), then the blocks
// that are left as one narrower chunk.
template <typename TZ, typename SA, typename SB, int MB, int NKS, int RP, bool BF = false>
static hipError_t launch_block_chunks(hipStream_t s, int ntiles, int nblk, int zw, int nz, int bchunks,
                                      const Tile* tiles, TZ* Z, int64_t ldz, const SA* A1, int64_t lda, const TZ* W,
                                      int64_t w_ld, int64_t w_pstride, int node_shift, const SB* B1, int64_t ldb, int kb,
                                      TZ* P, GroupStrides gs) {
  const int n = nblk / zw, nb = nblk % zw;
  hipError_t e = hipSuccess;
#define HODLR_LPB(NCBV, CHUNKS, BASE)                                                                              \
  e = launch_block_part<TZ, SA, SB, MB, NKS, NCBV, RP, BF>(s, ntiles, CHUNKS, BASE, nz, bchunks, tiles, Z, ldz, A1, lda, \
                                                           W, w_ld, w_pstride, node_shift, B1, ldb, kb, P, gs)
  if (zw == 4) HODLR_LPB(4, n, 0);
  else if (zw == 2) HODLR_LPB(2, n, 0);
  else HODLR_LPB(1, n, 0);
  if (e != hipSuccess) return e;
  const int base = 16 * zw * n;
  if (nb == 1) HODLR_LPB(1, 1, base);
  if (nb == 2) HODLR_LPB(2, 1, base);
  if (nb == 3) HODLR_LPB(3, 1, base);
#undef HODLR_LPB
  return e;
}

template <typename TZ, typename SA, typename SB, int MB, int RP>
static hipError_t launch_block_nks(int nks, hipStream_t s, int ntiles, int nblk, int zw, int nz, int bchunks,
                                   const Tile* tiles, TZ* Z, int64_t ldz, const SA* A1, int64_t lda, const TZ* W,
                                   int64_t w_ld, int64_t w_pstride, int node_shift, const SB* B1, int64_t ldb, int kb,
                                   TZ* P, GroupStrides gs) {
#define HODLR_LPF(NKSV)                                                                                            \
  return launch_block_chunks<TZ, SA, SB, MB, NKSV, RP>(s, ntiles, nblk, zw, nz, bchunks, tiles, Z, ldz, A1, lda, W,  \
                                                       w_ld, w_pstride, node_shift, B1, ldb, kb, P, gs)
  switch (nks) {
    case 0: HODLR_LPF(0);
    case 4: HODLR_LPF(4);
    case 8: HODLR_LPF(8);
    case 12: HODLR_LPF(12);
    default: HODLR_LPF(16);
  }
#undef HODLR_LPF
}

template <typename TZ, typename SA, typename SB, int RP>
static hipError_t launch_block(hipStream_t s, int ntiles, const Tile* tiles, TZ* Z, int64_t ldz, int nblk, int zw, int nz,
                                const SA* A1, int64_t lda, int ka, const TZ* W, int64_t w_ld, int64_t w_pstride,
                               int node_shift, const SB* B1, int64_t ldb, int kb, TZ* P, GroupStrides gs) {
  const int bchunks = kb > 0 ? (kb + 63) / 64 : 1;
#define HODLR_LPM(MBV)                                                                                              \
  return launch_block_nks<TZ, SA, SB, MBV, RP>(ka / 4, s, ntiles, nblk, zw, nz, bchunks, tiles, Z, ldz, A1, lda, W,   \
                                               w_ld, w_pstride, node_shift, B1, ldb, kb, P, gs)
  switch (kb > 0 ? std::min(kb, 64) / 16 : 0) {
    case 0: HODLR_LPM(0);
    case 1: HODLR_LPM(1);
    case 2: HODLR_LPM(2);
    case 3: HODLR_LPM(3);
    default: HODLR_LPM(4);
  }
#undef HODLR_LPM
}

// bfloat16 operands, ka and kb of 0, 16 or 32
template <typename TZ, typename SA, typename SB>
static hipError_t launch_block_bf(hipStream_t s, int ntiles, const Tile* tiles, TZ* Z, int64_t ldz, int nblk, int nz,
                                  const SA* A1, int64_t lda, int ka, const TZ* W, int64_t w_ld, int64_t w_pstride,
                                  int node_shift, const SB* B1, int64_t ldb, int kb, TZ* P, GroupStrides gs) {
#define HODLR_LPX(MBV, NKSV)                                                                                       \
  return launch_block_chunks<TZ, SA, SB, MBV, NKSV, 2, true>(s, ntiles, nblk, 4, nz, 1, tiles, Z, ldz, A1, lda, W, w_ld, \
                                                             w_pstride, node_shift, B1, ldb, kb, P, gs)
#define HODLR_LPY(MBV)               \
  if (ka == 0) HODLR_LPX(MBV, 0);    \
  if (ka == 16) HODLR_LPX(MBV, 4);   \
  HODLR_LPX(MBV, 8)
  if (kb == 0) { HODLR_LPY(0); }
  if (kb == 16) { HODLR_LPY(1); }
  HODLR_LPY(2);
#undef HODLR_LPY
#undef HODLR_LPX
}

template <typename TZ, typename SA, typename SB>
hipError_t launch_level_pass(hipStream_t s, int ntiles, const Tile* tiles, TileShape sh, TZ* Z, int64_t ldz, int nz,
                             const SA* A1, int64_t lda, int ka, const TZ* W, int64_t w_ld, int64_t w_pstride,
                             int node_shift, const SB* B1, int64_t ldb, int kb, TZ* P, GroupStrides gs, int bf) {
  if (ntiles == 0 || nz == 0 || (ka == 0 && kb == 0)) return hipSuccess;
  if (ka > 64 || sh.rows < 1 || sh.rows > kTileRows) return hipErrorInvalidValue;
  // whole 16 x 16 x 16 blocks, and byte offsets inside a 64-column chunk below
  // 2^31 (the buffer addressing of the blocked kernel).  Products alone, of whole
  // blocks of Z, may take narrower chunks of it (N = 2^22, rank 64 in FP32: 32 FP64 columns
  // 7.0 ms, 64 12.4; the row kernel 8.3 and 15.7; FP64, rank 32, 64 columns: 7.9 and
  // 8.7); with columns left over, which read all of B1 again, the row kernel is
  // faster (17 columns: 4.0 ms, 6.7 with the blocked kernel)
  auto bytes64 = [](int64_t ld, size_t size) { return 64 * ld * (int64_t)size; };
  constexpr int64_t kReach = 1ll << 31;
  const int64_t bz = bytes64(ldz, sizeof(TZ)), bb = bytes64(ldb, sizeof(SB));
  const bool small_ld = bz < kReach && bb < kReach && bytes64(lda, sizeof(SA)) < kReach;
  const int zw = bz <= kReach ? 4 : bz <= 2 * kReach ? 2 : 1;  // 16-column blocks of a chunk
  const bool blocks = sh.mult(16) && ka % 16 == 0 && kb % 16 == 0 &&
                      (small_ld || (ka == 0 && nz % 16 == 0 && bz <= 4 * kReach && bb <= kReach));
  int c_base = 0;
  if (blocks) {
    // 4-byte elements, tile heights multiples of 32, even leading dimensions
    // and 16-byte aligned operands (every paired access is naturally
    // aligned): two rows per lane
    auto al16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
    const bool pair = sizeof(TZ) == 4 && sh.mult(32) && ldz % 2 == 0 && (ka == 0 || lda % 2 == 0) &&
                      (kb == 0 || ldb % 2 == 0) && al16(Z) && (ka == 0 || al16(A1)) && (kb == 0 || al16(B1));
    // bfloat16 products only where the factorization uses them (Z and A1 both
    // Y); other shapes of a BF16 factorization, and all its passes at leading
    // dimensions beyond the buffer addressing, are computed in FP32.  The row
    // kernel moves 16 bytes a lane and nothing but W and P through LDS (N = 2^19,
    // rank 64: 5.69 ms a factorization, 6.67 ms with the turn-arounds of the
    // blocked kernel; rank 48 the same; N = 2^17, leaf 64, rank 32: 0.74 against
    // 0.79); up to rank 32 on tiles above 64 rows the blocked kernel streams
    // faster (N = 2^20, rank 32: 5.32 against 6.06 ms; N = 2^18, leaf 128: 1.23, 1.26)
    if constexpr (sizeof(TZ) == 4 && std::is_same<SA, TZ>::value) {
      if (bf && small_ld) {
        if (pair && ka <= 32 && kb <= 32 && sh.rows > 64 && nz > 16) {
          c_base = nz / 16 * 16;
          const hipError_t e = launch_block_bf<TZ, SA, SB>(s, ntiles, tiles, Z, ldz, nz / 16, nz, A1, lda, ka, W, w_ld,
                                                           w_pstride, node_shift, B1, ldb, kb, P, gs);
          if (e != hipSuccess || c_base == nz) return e;
        }
        return launch_rows<TZ, SA, SB, true>(s, ntiles, c_base, tiles, sh, Z, ldz, nz, A1, lda, ka, W, w_ld, w_pstride,
                                             node_shift, B1, ldb, kb, P, gs);
      }
    }
    // the blocked kernel from 17 columns on: it streams Z in 16-row blocks and
    // is bound by HBM (N = 2^20, rank 32, 2 r r_l columns: FP64 10.56 ms a
    // factorization against 12.06 ms with the row kernel, FP32 6.49 against
    // 6.96); one 16-column block leaves it waiting on loads, which the row
    // kernel keeps in flight (solve passes 1.29 against 1.40 ms, one vector)
    if (nz > 16) {
      c_base = nz / 16 * 16;
      hipError_t e;
      bool done = false;
      if constexpr (sizeof(TZ) == 4) {
        if (pair) {
          e = launch_block<TZ, SA, SB, 2>(s, ntiles, tiles, Z, ldz, nz / 16, zw, nz, A1, lda, ka, W, w_ld, w_pstride,
                                          node_shift, B1, ldb, kb, P, gs);
          done = true;
        }
      }
      if (!done)
        e = launch_block<TZ, SA, SB, 1>(s, ntiles, tiles, Z, ldz, nz / 16, zw, nz, A1, lda, ka, W, w_ld, w_pstride,
                                        node_shift, B1, ldb, kb, P, gs);
      if (e != hipSuccess || c_base == nz) return e;
    }
  }
  return launch_rows<TZ, SA, SB, false>(s, ntiles, c_base, tiles, sh, Z, ldz, nz, A1, lda, ka, W, w_ld, w_pstride,
                                        node_shift, B1, ldb, kb, P, gs);
}

// A narrow pass that forms W itself (see CPL of the row kernel).
template <typename TZ, typename SA, typename SB>
hipError_t launch_coupled_pass(hipStream_t s, int trans, int ntiles, const Tile* tiles, TileShape sh, TZ* Z,
                               int64_t ldz, int nz, const SA* A1, int64_t lda, int r, const TZ* Kinv, int kp,
                               const TZ* items, const int32_t* d_start, int node_shift, const SB* B1, int64_t ldb,
                               int kb, TZ* P, GroupStrides gs) {
  if (ntiles == 0 || nz == 0) return hipSuccess;
  if (r < 1 || r > 64 || r % 8 || kp < 2 * r || nz > 16 || sh.rows < 1 || sh.rows > kTileRows) return hipErrorInvalidValue;
  constexpr int kCw = 16;
  const int nt = (r + 15) / 16;
  const size_t part = std::max(sizeof(TZ) * 4 * 16 * kCw, sizeof(TZ) * kCw * 16 * nt);  // W, or a reduction buffer
  const size_t smem = 2 * part + sizeof(TZ) * 2 * nt * 256;
  const CoupleArgs<TZ> cpl{Kinv, kp, items, d_start};
#define HODLR_LC(FULL, TR)                                                                                           \
  {                                                                                                                  \
    auto k = level_pass_rows_kernel<TZ, SA, SB, 1, 1, FULL, false, TR>;                                              \
    hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);        \
    if (e != hipSuccess) return e;                                                                                   \
    hipLaunchKernelGGL(k, dim3(ntiles), dim3(kLpThreads), smem, s, tiles, 1, 0, 1, std::max(kb, 1), Z, ldz, nz, A1,   \
                       lda, r, (const TZ*)nullptr, 0, 0, node_shift, B1, ldb, kb, P, gs, (int)part, cpl);            \
  }
  if (sh.mult(64)) {
    if (trans) HODLR_LC(true, 2) else HODLR_LC(true, 1)
  } else {
    if (trans) HODLR_LC(false, 2) else HODLR_LC(false, 1)
  }
#undef HODLR_LC
  return hipGetLastError();
}

#define HODLR_LP_INST(TZ, SA, SB)                                                                                  \
  template hipError_t launch_level_pass<TZ, SA, SB>(hipStream_t, int, const Tile*, TileShape, TZ*, int64_t, int,     \
                                                    const SA*, int64_t, int, const TZ*, int64_t, int64_t, int,      \
                                                    const SB*, int64_t, int, TZ*, GroupStrides, int);
HODLR_LP_INST(double, double, double)
HODLR_LP_INST(float, float, double)
HODLR_LP_INST(float, double, float)
HODLR_LP_INST(float, float, float)
HODLR_LP_INST(double, double, float)
#undef HODLR_LP_INST
#define HODLR_LC_INST(TZ, SA, SB)                                                                                    \
  template hipError_t launch_coupled_pass<TZ, SA, SB>(hipStream_t, int, int, const Tile*, TileShape, TZ*, int64_t, int, \
                                                      const SA*, int64_t, int, const TZ*, int, const TZ*,             \
                                                      const int32_t*, int, const SB*, int64_t, int, TZ*, GroupStrides);
HODLR_LC_INST(double, double, double)
HODLR_LC_INST(float, float, double)
HODLR_LC_INST(float, double, float)
HODLR_LC_INST(float, float, float)
#undef HODLR_LC_INST

}  // namespace hodlr
