// Internal declarations of the HODLR library (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/hodlr.h"

namespace hodlr {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// Rows of one tile of a level pass: a run of <= kTileRows consecutive rows
// that lies inside one node of the pass's level.
constexpr int kTileRows = 256;
struct Tile {
  int64_t row0;
  int32_t nrows;
  int32_t node;  // node index (0-based, left to right) at the pass's level
};

// Heights of the tiles of one level: the largest, and every bit that is set
// in one of them.
struct TileShape {
  int rows = 0;
  int bits = 0;
  bool mult(int p) const { return bits % p == 0; }  // every height a multiple of the power of two p
};

// Segment of tiles summed by the reduction kernel.
constexpr int kSegTiles = 16;

// ---------------------------------------------------------------------------
// Small device helpers
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ T ld_as(const void* p, int64_t i);
template <>
__device__ __forceinline__ double ld_as<double>(const void* p, int64_t i) {
  return static_cast<const double*>(p)[i];
}
template <>
__device__ __forceinline__ float ld_as<float>(const void* p, int64_t i) {
  return static_cast<const float*>(p)[i];
}

// XCD-aware block index remap: hardware hands consecutive workgroup ids to
// the 8 XCDs round robin; this maps them so that consecutive *logical* ids
// land on the same XCD (and share its L2).  Bijective for any grid size.
__device__ __forceinline__ int64_t xcd_remap(int64_t bid, int64_t nblocks) {
  constexpr int kX = 8;
  int64_t per = nblocks / kX;           // full rounds
  int64_t rem = nblocks % kX;
  int64_t x = bid % kX, j = bid / kX;
  if (j < per) {
    // xcd x owns logical ids [x*per + min(x, rem) ... ) of length per + (x < rem)
    return x * per + (x < rem ? x : rem) + j;
  }
  // tail round (only xcds x < rem have a block here)
  return x * per + x + per;
}

// ---------------------------------------------------------------------------
// Launchers (defined in the .hip files).  T = compute type (double/float),
// S = storage type of the caller's D/U/V.
// ---------------------------------------------------------------------------

// leaf LU with partial pivoting; LU blocks col-major ldl x ldl per leaf (ldl % 16 == 0, lul = ldl),
// or in place (inplace = 1): leaf a's factor in rows [off_a, off_a + m_a) of lu with ld lul
// (every m_a % 16 == 0; lu may be D itself);
// invl: the inverted 16 x 16 diagonal blocks of L and U (2 x ldl/16 x 256 per leaf).
// bf = 1 (T = float): the trailing updates of the left-looking sweep take
// bfloat16 operands with FP32 accumulation; pivot search and panel stay FP32.
template <typename T, typename S>
hipError_t launch_leaf_lu(hipStream_t s, int nleaf, int ldl, const int64_t* d_leaf_off, const S* D, int64_t ldd,
                          T* lu, int64_t lul, int inplace, int32_t* piv, int32_t* perm, T* udinv, T* invl,
                          unsigned long long* info, int bf = 0);

// Leaf triangular solves on column chunks.
// trans = 0: X(I_a, :) = U_a^{-1} L_a^{-1} P_a^T B(I_a, :)
// trans = 1: X(I_a, :) = P_a L_a^{-T} U_a^{-T} B(I_a, :)
// B and X may alias (same type).
// dinv: per block 2 x (ldl/16) inverted 16 x 16 diagonal blocks ([0]: L, [1]: U) from the factorization.
// lu, lul, inplace: the leaf factors in either layout of launch_leaf_lu.
// bf = 1 (T = float, trans = 0): the block products take bfloat16 operands with
// FP32 accumulation (the leaf solve of a BF16 factorization).
template <typename T, typename S>
hipError_t launch_leaf_trsm(hipStream_t s, int trans, int nleaf, int ldl, const int64_t* d_leaf_off, const T* lu,
                            int64_t lul, int inplace, const int32_t* perm, const T* dinv, const S* B, int64_t ldb,
                            T* X, int64_t ldx, int ncols, int64_t gsb = 256, int64_t gsx = 256, int bf = 0);

// Fused level pass on tiles:
//   update : Z(tile, 0:nz) -= A1(tile, 0:ka) * W_node(0:ka, 0:nz)      (if ka > 0)
//   product: P_tile(0:kb, 0:nz) = B1(tile, 0:kb)^T * Z(tile, 0:nz)      (if kb > 0)
// nd = tile.node >> node_shift; W for node nd starts at W + (nd >> 1) * w_pstride + (nd & 1) * ka, ld = w_ld.
// P_tile starts at P + tile * kb * nz, col-major ld = kb.
// Row addressing of the Z, A1 and B1 operands: row i of an operand lives at
// (i >> 8) * gs + (i & 255) (plus column * ld).  gs = 256 is the plain
// column-major layout; gs = 256 * ncols with ld = 256 is the row-group blocked
// layout (each 256-row group of all columns contiguous), valid when no tile
// crosses a 256-row boundary.
// bf = 1 (4-byte TZ): the products take bfloat16 operands with FP32
// accumulation (the coupling GEMMs of a BF16 factorization); shapes without
// whole 16 x 16 x 16 blocks are computed in FP32.
struct GroupStrides {
  int64_t z = 256, a = 256, b = 256;
};
__host__ __device__ __forceinline__ int64_t group_row(int64_t row, int64_t gs) { return (row >> 8) * gs + (row & 255); }

template <typename TZ, typename SA, typename SB>
hipError_t launch_level_pass(hipStream_t s, int ntiles, const Tile* tiles, TileShape shape, TZ* Z, int64_t ldz, int nz,
                             const SA* A1, int64_t lda, int ka, const TZ* W, int64_t w_ld,
                             int64_t w_pstride, int node_shift, const SB* B1, int64_t ldb, int kb, TZ* P,
                             GroupStrides gs = GroupStrides(), int bf = 0);

// Narrow pass (nz <= 16) whose update takes W = K^{-1} rhs (trans: K^{-T} rhs) of the level's
// coupling systems, formed in the pass: Kinv and kp as launch_couple_solve, child c's items
// (r x nz each) d_start[c] .. d_start[c + 1] - 1, summed in order.  P must not overlap items.
template <typename TZ, typename SA, typename SB>
hipError_t launch_coupled_pass(hipStream_t s, int trans, int ntiles, const Tile* tiles, TileShape sh, TZ* Z,
                               int64_t ldz, int nz, const SA* A1, int64_t lda, int r, const TZ* Kinv, int kp,
                               const TZ* items, const int32_t* d_start, int node_shift, const SB* B1, int64_t ldb,
                               int kb, TZ* P, GroupStrides gs = GroupStrides());

// Segment sums of tile partials: out[s] = sum of tiles [desc[s].x, desc[s].x + desc[s].y),
// maxy = max over s of desc[s].y (<= kSegTiles).
template <typename T>
hipError_t launch_segment_reduce(hipStream_t s, int nsegs, const int2* d_desc, int64_t elems, const T* P, T* out,
                                 int maxy);

// Coupling factor for all parents of one level (children have rank r, W has Rp columns):
// K^{-1} stored kp x kp per parent (kp = 2r rounded up to 16, zero padding), Kpiv / Kud its
// interchanges and reciprocal pivots (two halves of r rounded up to 16 per parent), W = K^{-1} rhs
// (2r x Rp per parent).
// Child c's product: item seg_start[c], r x (Rp + r) col-major.
// Ranks off the multiples of 8 correct every product with K^{-1} by its
// residual: their coupling systems have the accuracy of substitution with an
// LU (rank 33, entries of V^T Y above one: error 1e-12 of x with it, 2e-10
// without).  Kt (2 r x r per parent) keeps T_a and T_b for that.
__host__ __device__ inline bool couple_corrects(int r) { return r % 8 != 0; }
template <typename T>
hipError_t launch_couple_factor(hipStream_t s, int nparents, int r, int kp, int Rp, const T* segs,
                                const int32_t* d_seg_start, T* Kinv, int32_t* Kpiv, T* Kud, T* Kt, T* W,
                                unsigned long long* info, int level, int L);

// Coupling solve for all parents of one level: w = K^{-1} rhs (trans=0) or K^{-T} rhs.
// rhs rows of child c come from its item (r x nrhs); w is 2r x nrhs per parent.
template <typename T>
hipError_t launch_couple_solve(hipStream_t s, int trans, int nparents, int r, int kp, int nrhs, const T* segs,
                               const int32_t* d_seg_start, const T* Kinv, const T* Kt, T* w);

// Pairwise sums up the projection tree (below) from level L to level 1 (blocks of elems doubles).
hipError_t launch_tree_sums(hipStream_t s, int L, int64_t elems, double* tree);

// Projection tree: for l = 1..L, the 2^l node sums (R x nrhs each, col-major ld R) of level l
// start at node slot (2^l - 2); slot k begins at tree + k * R * nrhs.
__host__ __device__ inline int64_t tree_slot(int l, int node) { return ((int64_t)1 << l) - 2 + node; }

// y = op(D) x + U G per leaf (FP64 arithmetic) from the projection tree.
template <typename S>
hipError_t launch_matvec_apply(hipStream_t s, int trans, int nleaf, int L, const int64_t* d_leaf_off,
                               const int32_t* d_rpre, int R, const S* D, int64_t ldd, const S* Ua, int64_t lda,
                               const double* X, int64_t ldx, const double* tree, double* Y, int64_t ldy, int nrhs,
                               TileShape sh);  // sh: of the leaves

// Gradient pieces.  grad_leaf: dD_a = add_a - Lam_a X_a^T on the leaf blocks (add may be null).
// grad_gen: out(I_a, c) = add(I_a, c) - Left(I_a, :) S(c, :)^T with S the projection-tree entry of
// the sibling of a's ancestor at c's level; tri = 1 restricts the sum to the columns of the
// levels above c's level.
template <typename S>
hipError_t launch_grad_leaf(hipStream_t s, int nleaf, int m_max, const int64_t* d_leaf_off, int nrhs,
                            const double* X, int64_t ldx, const double* Lam, int64_t ldl, S* dD, int64_t ldd,
                            const double* add = nullptr, int64_t ldadd = 0);
template <typename S>
hipError_t launch_grad_gen(hipStream_t s, int nleaf, int m_max, int L, const int64_t* d_leaf_off,
                           const int32_t* d_rpre, int R, int nrhs, const double* Left, int64_t ldl, const double* tree, S* out, int64_t ldo,
                           const double* add = nullptr, int64_t ldadd = 0, int tri = 0);

// Refinement helpers (FP64).
hipError_t launch_colnorms(hipStream_t s, int64_t n, int nrhs, const double* X, int64_t ldx, double* part,
                           double* out2, double* outinf);
template <typename T>
hipError_t launch_scale_down(hipStream_t s, int64_t n, int nrhs, const double* Rr, int64_t ldr, const double* sc,
                             T* out, int64_t ldo);
template <typename T>
hipError_t launch_axpy_up(hipStream_t s, int64_t n, int nrhs, const T* d, int64_t ldd, const double* sc, double* X,
                          int64_t ldx);
hipError_t launch_residual(hipStream_t s, int64_t n, int nrhs, const double* B, int64_t ldb, double* AX, int64_t ldax);
template <typename T, typename S>
hipError_t launch_convert(hipStream_t s, int64_t rows, int cols, const S* in, int64_t ldi, T* out, int64_t ldo,
                          int64_t gsi = 256);

}  // namespace hodlr

namespace hodlr {
// Fixed device scratch of the allocation-free solve (noalloc.hip): capacity in
// bytes, and this device's address of it (the current device; looked up once
// per device).
size_t scratch_capacity();
hipError_t scratch_device_ptr(void** out);
}  // namespace hodlr

namespace hodlr {
// Coupling factors of the levels that have them, for the log-determinant:
// per entry p < n, `count` parents with kp entries each (two halves of the rank
// rounded up to 16) from element kvoff of the K vectors (interchanges, 1 / pivots).
struct LogdetLevels {
  int n = 0;
  int count[HODLR_MAX_LEVELS];
  int kp[HODLR_MAX_LEVELS];
  int64_t kvoff[HODLR_MAX_LEVELS];
};
// log|det A| (out[0]) and its sign (out[1]) from the leaf factors (1 / U_jj,
// interchanges) and the coupling factors; item_log / item_par: nleaf + sum of
// counts scratch entries.
template <typename T>
hipError_t launch_logdet(hipStream_t s, int nleaf, int ldl, const int64_t* d_leaf_off, const T* udinv,
                         const int32_t* piv, const T* Kud, const int32_t* Kpiv, const LogdetLevels& lv,
                         double* item_log, int* item_par, double* out);
}  // namespace hodlr

namespace hodlr {
// Pieces of the gradient of log|det A| (logdet.hip).
template <typename S>
hipError_t launch_transpose_leaves(hipStream_t s, int nleaf, int m_max, const int64_t* d_leaf_off, const S* D,
                                   int64_t ldd, S* Dt, int64_t ldt);
template <typename T>
hipError_t launch_identity_leaves(hipStream_t s, int nleaf, int ncols, const int64_t* d_leaf_off, T* E, int64_t lde);
template <typename T>
hipError_t launch_pblocks(hipStream_t s, int nparents, int r, const T* Kinv, int64_t ldk, int64_t pstride, double* Pd);
// out(i, c) = sum_k in(i, R_{l-1} + k) M_a(k, c - R_{l-1}) for every column c (level l) and row i
// (node a of level l), M_a = P_a (trans: P_a^T) from Pd at element pdoff[l] + a r_l^2; FP64, N x R, ld N
hipError_t launch_node_mix(hipStream_t s, int64_t n, int nleaf, int m_max, int L, int R, const int64_t* d_leaf_off,
                           const int32_t* d_rpre, const int64_t* d_pdoff, const double* Pd, int trans,
                           const double* in, double* out);
}  // namespace hodlr

namespace hodlr {
// Construction by cross approximation (construct.hip).
struct ConstructKernel {
  int kind;
  int dim;
  const double* pts;
  int64_t ldp;
  const double* nrm;
  const double* w;
  const double* kap;
  double ell;
  double shift;
};
// One sibling block A(I_a, I_b): rows r0 .. r0 + m, columns c0 .. c0 + n, its
// generators in columns col .. col + rank of U_big / V_big, its tiles
// tile0 .. tile0 + ntile (each covers aca_tile_elems() rows and columns).
struct AcaBlock {
  int64_t r0, c0;
  int32_t m, n, col, rank, tile0, ntile;
};
struct AcaTile {
  int32_t blk, t, gtile;
};
// per-tile partial argmax of the residual rows (modulus, signed value, column)
// and columns (score, row); pivot rows [block][kmax]
struct AcaPartials {
  double* rp_abs;
  double* rp_val;
  int* rp_idx;
  double* cp_abs;
  int* cp_idx;
  int* piv;
};
int aca_tile_elems();
template <typename TS>
hipError_t launch_construct_leaves(hipStream_t s, const ConstructKernel& k, int nleaf, const int64_t* d_off, int m_max,
                                   TS* D, int64_t ldd);
// Blocks that one workgroup can take through all steps: the class of a block's
// kernel (0 .. 2), or 3 for the tiled steps; the classes that get a launch of
// their own (bit c; the others are tiled too) from the number of blocks, their
// tiles and the sum of rows times rank of each class; the launch for nblocks of
// a class (their tile0 and ntile are not used).
int aca_block_class(int m, int n, int rank);
int aca_own_launches(const int64_t (&blocks)[4], const int64_t (&tiles)[4], const int64_t (&work)[4]);
hipError_t launch_aca_blocks(hipStream_t s, const ConstructKernel& k, int cls, int nblocks, const AcaBlock* blocks,
                             double* U, int64_t ldu, double* V, int64_t ldv);
// step `step` of every tiled block (rank > step): the residual-row launch and the residual-column launch
hipError_t launch_aca_step(hipStream_t s, const ConstructKernel& k, int ntiles, const AcaBlock* blocks,
                           const AcaTile* tiles, int step, int kmax, double* U, int64_t ldu, double* V, int64_t ldv,
                           AcaPartials p);
template <typename TS>
hipError_t launch_store_cols(hipStream_t s, int64_t n, int ncols, const double* src, int64_t lds, TS* dst, int64_t ldd);
}  // namespace hodlr

namespace hodlr {
// Real embedding of complex matrices (embed.hip): E (2n x 2c, ld lde) =
// emb(M) for complex M (n x c, interleaved, ld ldm in complex elements), and
// back (M from the first column of each 2 x 2 block).
hipError_t launch_embed_cols(hipStream_t s, int64_t n, int ncols, const double* M, int64_t ldm, double* E, int64_t lde);
hipError_t launch_deembed_cols(hipStream_t s, int64_t n, int ncols, const double* E, int64_t lde, double* M,
                               int64_t ldm);
}  // namespace hodlr
