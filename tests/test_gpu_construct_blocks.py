"""Cross approximation of single blocks at the edges of the one-workgroup
kernels (128, 256 and 512 rows or columns, more rows than columns and the other
way round, ranks 1 to 33, which take the tiled steps), against the construction
oracle: the same pivots exactly (residuals far above rounding), approximants to
1e-12 of the block."""
import numpy as np
import pytest

import oracle as O
from test_gpu_construct import _gpu_build, _spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,dim,rank", [("gauss", 2, 8), ("matern32", 3, 32), ("matern32", 3, 33), ("laplace_dl", 2, 6),
                                           ("gauss", 1, 1)])
@pytest.mark.parametrize("m,n", [(40, 64), (128, 127), (129, 60), (200, 256), (256, 257), (512, 300), (511, 512), (513, 100)])
def test_blocks(kind, dim, rank, m, n):
    off = np.array([0, m, m + n], dtype=np.int64)
    if max(m, n) > 256:  # leaves hold up to 256 rows: halve them
        off = np.array([0, m // 2, m, m + n // 2, m + n], dtype=np.int64)
        if max(np.diff(off)) > 256:
            off = np.array(sorted({0, m // 4, m // 2, 3 * m // 4, m, m + n // 4, m + n // 2, m + 3 * n // 4, m + n}))
    L = int(np.log2(len(off) - 1))
    ranks = [rank] + [0] * (L - 1)
    spec = _spec(kind, m + n, dim, 3, 0.1)
    A = _gpu_build(spec, ranks, off)
    U, V = A.U.cpu().numpy().T, A.V.cpu().numpy().T
    for (s0, e0), (t0, f0) in (((0, m), (m, m + n)), ((m, m + n), (0, m))):
        M = O.kernel_entries(spec, np.arange(s0, e0), np.arange(t0, f0))
        Uo, Vo, I, J = O.aca(lambda ri, cj: M[np.ix_(ri, cj)], e0 - s0, f0 - t0, rank)
        for k, j in enumerate(J):
            assert j >= 0 and V[t0 + j, k] == 1.0, k
        assert np.linalg.norm(U[s0:e0] @ V[t0:f0].T - Uo @ Vo.T) <= 1e-12 * np.linalg.norm(M)


@pytest.mark.parametrize("kind,dim", [("laplace_dl", 2), ("gauss", 2), ("matern32", 3)])
@pytest.mark.parametrize("leaf,levels", [(64, 1), (128, 1), (200, 1), (256, 1), (150, 2), (256, 2)])
def test_one_workgroup_equals_the_tiled_steps_to_the_bit(kind, dim, leaf, levels):
    """The first columns of rank 33, which takes the tiled steps, are the columns
    of every smaller rank: the pivots of a block that has used up its numerical
    rank follow from the last bit of the entries."""
    n = leaf << levels
    spec = _spec(kind, n, dim, 3, 0.1)
    off = np.arange((1 << levels) + 1, dtype=np.int64) * leaf
    ranks = [0] * (levels - 1)
    tiled = _gpu_build(spec, [33] + ranks, off)
    for rank in (6, 24, 32):
        A = _gpu_build(spec, [rank] + ranks, off)
        assert (A.U == tiled.U[:rank]).all() and (A.V == tiled.V[:rank]).all(), rank


@pytest.mark.parametrize("kind,dim", [("gauss", 2), ("laplace_dl", 2)])
@pytest.mark.parametrize("row", [0, 70])
def test_rows_of_nan_are_skipped_by_both_routes(kind, dim, row):
    """A point that is not a number makes its residual row one without a pivot:
    the step is exhausted (zero columns) and the next row is taken."""
    m, rank = 100, 8
    spec = _spec(kind, 2 * m, dim, 3, 0.1)
    spec.points[row] = np.nan
    off = np.array([0, m, 2 * m], dtype=np.int64)
    A, tiled = _gpu_build(spec, [rank], off), _gpu_build(spec, [33], off)
    for got, want in ((A.U, tiled.U[:rank]), (A.V, tiled.V[:rank])):
        assert ((got == want) | (got.isnan() & want.isnan())).all()
    if row == 0:  # the first row searched by the block on top
        assert not A.U[0, :m].any() and not A.V[0, m:].any()


@pytest.mark.parametrize("n,leaf,ranks,own,tiled", [
    (4096, 64, [16] * 6, 0, 16),            # a few small blocks join the tiled steps: no launch in front of them
    (1024, 128, [16] * 3, 3, 0),            # nothing but small blocks: one launch a class
    (1 << 17, 128, [32] * 10, 3, 32),       # the tiles fill the chip with and without the small blocks
    (1 << 17, 128, [16] * 10, 2, 16),       # without the classes of 128 and 256 rows they do no more
    (1 << 17, 256, [16] * 9, 1, 16),
    (1 << 16, 128, [32] * 9, 0, 32),
    (4096, 64, [20, 20, 20, 0, 0, 4], 0, 20),
])
def test_routes_by_size(n, leaf, ranks, own, tiled):
    from paper_2208_06290_amd import hodlr
    spec = _spec("gauss", n, 2, 3, 0.1)
    hodlr.timing(True)
    _gpu_build(spec, ranks, None)
    kt = hodlr.kernel_times()
    hodlr.timing(False)
    assert kt.get("aca_block", (0, 0))[1] == own and kt.get("aca_step", (0, 0))[1] == tiled
