"""The coupling updates of a BF16 factorization, on matrices whose updates are
as large as Y_big itself (V^T Y of order one on and between the levels): the
error of Y_big relative to the updates alone, within four times what rounding
the operands of every product to bfloat16 gives in a plain emulation.  A level
pass that leaves the update out, or takes another operand, is off by all of it.
Shapes: both kernels of the bfloat16 passes and those computed in FP32."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from test_gpu_level_pass import SHAPES

DEV = "cuda"


def _matrix(name):
    leaves, ranks = SHAPES[name]
    sizes = np.array(leaves if isinstance(leaves, list) else [leaves] * 8)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    inp = W.synthetic(int(off[-1]), 0, ranks, seed=len(name), leaf_offsets=off)
    L, Rp = len(ranks), np.concatenate([[0], np.cumsum(ranks)])
    V = [inp.V[Rp[l]:Rp[l + 1]] for l in range(L)]
    for l in range(L):  # orthonormal on every node of the level
        for a in range(2 << l):
            rows = slice(int(off[a << (L - l - 1)]), int(off[(a + 1) << (L - l - 1)]))
            V[l][:, rows] = torch.linalg.qr(V[l][:, rows].T)[0].T
    rng = np.random.default_rng(7)
    scale = 4.0 * torch.as_tensor(np.repeat(sizes, sizes), dtype=torch.float64)
    U = []
    for l in range(L):
        u = 0.5 * V[l]
        for k in range(l + 1, L):  # what the finer levels' updates act on
            mix = rng.standard_normal((ranks[l], ranks[k])) / np.sqrt(ranks[k])
            u = u + torch.as_tensor(mix) @ V[k] / 2 ** ((k - l) / 2)
        U.append(u)
    inp.V, inp.U = torch.cat(V), torch.cat(U) * scale
    return inp, off


def _y_big(inp, off, rnd, updates=True):
    """Y_big with the operands of every product through rnd."""
    D, U, V, ranks = inp.D.numpy(), rnd(inp.U.numpy()), inp.V.numpy(), inp.ranks
    L, Rp = len(ranks), np.concatenate([[0], np.cumsum(ranks)])
    Y = np.empty_like(U.T)
    for a in range(1 << L):
        s = slice(off[a], off[a + 1])
        Y[s] = rnd(np.linalg.solve(D[:off[a + 1] - off[a], s].T, U[:, s].T))
    for l in range(L, 0, -1) if updates else ():
        c, r = slice(Rp[l - 1], Rp[l]), ranks[l - 1]
        for g in range(1 << (l - 1)):
            rows = [slice(off[(2 * g + h) << (L - l)], off[(2 * g + h + 1) << (L - l)]) for h in (0, 1)]
            P = [rnd(V[c, s]) @ rnd(Y[s, :Rp[l]]) for s in rows]
            K = np.block([[P[0][:, c], np.eye(r)], [np.eye(r), P[1][:, c]]])
            Wg = np.linalg.solve(K, np.vstack([P[0][:, :Rp[l - 1]], P[1][:, :Rp[l - 1]]]))
            for h, s in enumerate(rows):
                Y[s, :Rp[l - 1]] -= rnd(Y[s, c]) @ rnd(Wg[h * r:(h + 1) * r])
    return Y


def _bf16(x):
    return torch.as_tensor(x).to(torch.bfloat16).to(torch.float64).numpy()


def _bar(name):
    """(matrix, offsets, Y_big, norm of its updates, bar) over the columns that have updates."""
    inp, off = _matrix(name)
    n = sum(inp.ranks[:-1])
    Y = _y_big(inp, off, lambda x: x)[:, :n]
    size = np.linalg.norm(Y - _y_big(inp, off, lambda x: x, updates=False)[:, :n])
    bar = 4 * np.linalg.norm(_y_big(inp, off, _bf16)[:, :n] - Y) / size
    return inp, off, Y, size, bar


@pytest.mark.parametrize("name", list(SHAPES))
def test_the_bar_tells_a_missing_update(name):
    inp, off, Y, size, bar = _bar(name)
    ref = O.y_big(O.factor(O.from_inputs(inp)))[:, :Y.shape[1]]
    assert np.linalg.norm(ref - Y) < 1e-10 * size  # the emulation without rounding is the factorization
    assert size > 0.3 * np.linalg.norm(Y) and bar < 0.2


@pytest.mark.gpu
@pytest.mark.parametrize("store", [torch.float64, torch.float32])
@pytest.mark.parametrize("name", list(SHAPES))
def test_updates(name, store):
    from paper_2208_06290_amd import hodlr
    inp, off, Y, size, bar = _bar(name)
    A = hodlr.HODLRMatrix(inp.D.to(DEV, store), inp.U.to(DEV, store), inp.V.to(DEV, store), inp.ranks, off)
    got = hodlr.factor(A, "bf16").y_big().cpu().numpy().T[:, :Y.shape[1]]
    assert np.linalg.norm(got - Y) < bar * size


@pytest.mark.gpu
def test_long_leading_dimension_in_fp32(monkeypatch):
    """Where 64 columns of V reach 2^31 bytes, the products of a BF16 factorization
    are FP32 ones like its updates; with leaves of 32 rows nothing else of it
    takes bfloat16 operands.  A hundredth of what rounding them would give."""
    from paper_2208_06290_amd import hodlr
    monkeypatch.setitem(SHAPES, "rows_32", (32, [16, 16, 16]))
    inp, off, Y, size, bar = _bar("rows_32")
    wide = torch.empty(inp.V.shape[0], 1 << 22, dtype=torch.float64, device=DEV)[:, :inp.n]
    A = hodlr.HODLRMatrix(inp.D.to(DEV), inp.U.to(DEV), wide.copy_(inp.V), inp.ranks, off)
    got = hodlr.factor(A, "bf16").y_big().cpu().numpy().T[:, :Y.shape[1]]
    assert np.linalg.norm(got - Y) < bar / 400 * size
