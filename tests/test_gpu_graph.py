"""Solves recorded into a HIP graph: every replay equals the eager solve of the
same right-hand side, with eager work between replays; calls that need device
memory are refused while recording, and the recording stays whole."""
import ctypes

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_recorded_solve(precision):
    from paper_2208_06290_amd import hodlr
    A = hodlr.HODLRMatrix.from_inputs(W.synthetic(2048, 64, [16, 8, 16, 24, 16], seed=3).to(DEV))
    F = hodlr.factor(A, precision)
    b = torch.zeros(2, A.n, dtype=torch.float64, device=DEV)
    x, y = torch.empty_like(b), torch.empty_like(b)
    other = hodlr.factor(A, "fp64")
    A.matvec(b)
    del other  # the library keeps blocks of the sizes the calls below need
    lib, m, h = hodlr.load_library(), A.c_struct(), ctypes.c_void_p()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        x.copy_(b)
        F.solve_noalloc_(x)
        refused = [lib.hodlr_matvec(ctypes.byref(m), 0, 2, b.data_ptr(), A.n, y.data_ptr(), A.n, s),
                   lib.hodlr_factor(ctypes.byref(m), 0, 0, s, ctypes.byref(h), None),
                   lib.hodlr_logdet_grad(F._h, y.data_ptr(), y.data_ptr(), y.data_ptr(), s)]
        F.solve_noalloc_(x, adjoint=True)
    assert refused == [-2, -2, -2]
    for seed in range(4):
        b.copy_(torch.randn(2, A.n, generator=torch.Generator().manual_seed(seed), dtype=torch.float64))
        g.replay()
        want = F.solve_adjoint(F.solve(b))
        assert torch.equal(x, want)
        F.refactor()
        assert torch.equal(A.matvec(b), A.matvec(b))
