"""Pivot ties of the leaf LU: orthogonal leaf blocks whose columns hold many
entries of equal modulus (the discrete Hartley matrix: its first column is all
ones, others tie by symmetry), equal up to the low word of a double, and all
equal (Hadamard), at leaf sizes around the 32-column panels and the 64 rows of
a wave, against the CPU oracle (1e-12, the suite's FP64 bar; the factors'
growth times unit roundoff stays below 1e-13)."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _rel(a, b):
    return float(np.max(np.linalg.norm(a - b, axis=0) / np.linalg.norm(b, axis=0)))


def _block(n, kind):
    if kind == "hadamard":
        h = np.ones((1, 1))
        while h.shape[0] < n:
            h = np.block([[h, h], [h, -h]])
        return h
    t = 2 * np.pi * np.outer(np.arange(n), np.arange(n)) / n
    q = np.cos(t) + np.sin(t)
    if kind == "low_words":  # first column: equal high words, the largest modulus in the middle
        q[:, 0] = 1.0 + 2.0 ** -40 * ((np.arange(n) * 7) % n)
    return q


@pytest.mark.parametrize("leaf,kind", [(n, k) for n in (17, 32, 33, 64, 65, 96, 128, 200, 255, 256)
                                       for k in ("hartley", "low_words")] + [(64, "hadamard"), (128, "hadamard")])
def test_pivot_ties(leaf, kind):
    from paper_2208_06290_amd import hodlr
    inp = W.synthetic(4 * leaf, leaf, [8, 8], seed=leaf)
    for a in range(4):  # column-major storage: D[q, s0 + p]; leaf 2 the other way round
        q = _block(leaf, kind)
        inp.D[:leaf, a * leaf:(a + 1) * leaf] = torch.as_tensor(np.ascontiguousarray((q[::-1] if a == 2 else q).T))
    H = O.from_inputs(inp)
    B = np.random.default_rng(leaf).standard_normal((H.N, 2))
    b = torch.as_tensor(np.ascontiguousarray(B.T), device=DEV)
    F = hodlr.factor(hodlr.HODLRMatrix.from_inputs(inp.to(DEV)), "fp64")
    assert _rel(F.solve(b).cpu().numpy().T, O.solve(O.factor(H), B)) < 1e-12
    F32 = hodlr.factor(hodlr.HODLRMatrix.from_inputs(inp.to(DEV)), "fp32")
    assert _rel(F32.solve(b).cpu().numpy().T, O.solve(O.factor(H), B)) < 1e-3
