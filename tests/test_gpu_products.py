"""Matrix products and gradients around the 64-row blocks and 16-column groups
of their kernels: leaf heights of 16 to 256 rows (one kernel each up to 64, up to
128 and above), uneven ones, odd and zero ranks, 1 to 65 columns, both storage
types, against the CPU oracle: FP64 storage to 1e-13 of the largest entry (sums
of at most 2048 terms), FP32 storage's gradients to one rounding (1e-7)."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from test_gpu_level_pass import SHAPES

pytestmark = pytest.mark.gpu

DEV = "cuda"
MORE = {"64_short": ([64, 33, 17, 50, 64, 1, 16, 63], [16, 7, 1]), "zero": (96, [0, 33, 16]), "48": (48, [3, 0, 40])}


def _case(name, dtype):
    leaves, ranks = {**SHAPES, **MORE}[name]
    off = None
    if isinstance(leaves, list):
        off = np.concatenate([[0], np.cumsum(leaves)]).astype(np.int64)
        n, leaf = int(off[-1]), 0
    else:
        n, leaf = 8 * leaves, leaves
    inp = W.synthetic(n, leaf, ranks, seed=len(name), leaf_offsets=off, dtype=dtype)
    from paper_2208_06290_amd import hodlr
    return hodlr, O.from_inputs(inp), hodlr.HODLRMatrix.from_inputs(inp.to(DEV))


def _dev(B):
    return torch.as_tensor(np.ascontiguousarray(B.T), device=DEV)


def _close(a, b, tol):
    a = a.double().cpu().numpy().T
    assert a.shape == b.shape and np.max(np.abs(a - b)) <= tol * np.max(np.abs(b))


@pytest.mark.parametrize("name", list(SHAPES) + list(MORE))
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nrhs", [1, 17, 33, 65])
def test_matvec_and_gradients(name, dtype, nrhs):
    hodlr, H, A = _case(name, dtype)
    rng = np.random.default_rng(nrhs)
    X, Lam = rng.standard_normal((H.N, nrhs)), rng.standard_normal((H.N, nrhs))
    _close(A.matvec(_dev(X)), O.matvec(H, X), 1e-13)
    _close(A.matvec(_dev(X), trans=True), O.matvec(O.transpose(H), X), 1e-13)
    F = hodlr.factor(A, "fp64" if dtype == torch.float64 else "fp32")
    dD, dU, dV = F.grad(_dev(X), _dev(Lam))
    rD, rU, rV = O.grad_structured(H, X, Lam)
    tol = 1e-13 if dtype == torch.float64 else 1e-7
    _close(dU, rU, tol)
    _close(dV, rV, tol)
    for a in range(len(H.offsets) - 1):
        s, e = int(H.offsets[a]), int(H.offsets[a + 1])
        _close(dD[:e - s, s:e], rD[s:e, :e - s], tol)
