"""Leaf solves with row interchanges: the rows of every leaf block are shuffled
or swapped in pairs, so partial pivoting moves rows singly, in runs and not at
all, at leaf sizes around the blocks of 16, 64 and 128 rows and at column counts
around the chunks, forward and adjoint, against the CPU oracle (1e-12, the
suite's FP64 bar; the matrices stay well conditioned)."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _rel(a, b):
    return float(np.max(np.linalg.norm(a - b, axis=0) / np.linalg.norm(b, axis=0)))


@pytest.mark.parametrize("leaf", [17, 48, 64, 65, 100, 112, 127, 128, 144, 256])
@pytest.mark.parametrize("cols", [65, 130])
def test_shuffled_leaves(leaf, cols):
    from paper_2208_06290_amd import hodlr
    inp = W.synthetic(4 * leaf, leaf, [min(64, leaf)] * 2, seed=leaf)
    rng = np.random.default_rng(leaf)
    for a in range(4):
        p = np.arange(leaf)
        if a == 1:
            p = rng.permutation(leaf)
        elif a == 2:
            p[[3, 9]] = p[[9, 3]]
        elif a == 3:
            p = np.roll(p, 5)
        blk = inp.D[:leaf, a * leaf:(a + 1) * leaf]
        blk[:] = blk[:, torch.as_tensor(p)].clone()
    H = O.from_inputs(inp)
    B = rng.standard_normal((H.N, cols))
    b = torch.as_tensor(np.ascontiguousarray(B.T), device=DEV)
    F = hodlr.factor(hodlr.HODLRMatrix.from_inputs(inp.to(DEV)), "fp64")
    Ho = O.factor(H)
    assert _rel(F.y_big().cpu().numpy().T, O.y_big(Ho)) < 1e-12
    assert _rel(F.solve(b).cpu().numpy().T, O.solve(Ho, B)) < 1e-12
    assert _rel(F.solve_adjoint(b).cpu().numpy().T, O.solve_adjoint(H, B)) < 1e-12
    for prec in ("fp32", "bf16"):
        x = hodlr.factor(hodlr.HODLRMatrix.from_inputs(inp.to(DEV)), prec).solve(b, refine=True, tol=1e-13)
        assert _rel(x.cpu().numpy().T, O.solve(Ho, B)) < 1e-12
