"""Factorizations made and released in a row reuse one another's device
memory: each result equals the oracle's whatever the blocks held before, from
one thread and from several threads on streams of their own, and work still
queued when a factorization is released is not overwritten."""
import threading

import numpy as np
import pytest
import torch

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

DEV = "cuda"
SIZES = [(1024, 64, [8, 16, 8, 16]), (1000, 125, [7, 3, 12]), (4096, 128, [32] * 5), (200, 200, [])]


def _problem(k):
    n, leaf, ranks = SIZES[k % len(SIZES)]
    inp = W.synthetic(n, leaf, ranks, seed=k)
    H = O.from_inputs(inp)
    b = np.random.default_rng(k).standard_normal((n, 1 + k % 3))
    return inp, b, O.solve(O.factor(H), b)


def _solve(inp, b, prec):
    from paper_2208_06290_amd import hodlr
    A = hodlr.HODLRMatrix.from_inputs(inp.to(DEV))
    F = hodlr.factor(A, prec)
    x = F.solve(torch.as_tensor(np.ascontiguousarray(b.T), device=DEV), refine=prec != "fp64", tol=1e-13)
    Y = F.y_big() if sum(A.ranks) else None
    del F  # its memory goes back while Y may still be on its way
    return x.cpu().numpy().T, Y


def _err(x, ref):
    return float(np.max(np.linalg.norm(x - ref, axis=0) / np.linalg.norm(ref, axis=0)))


@pytest.mark.parametrize("threads", [1, 4])
def test_factor_release_repeat(threads):
    problems = [_problem(k) for k in range(8)]
    errs, fails = [], []

    def work(t):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for rep in range(3):
                    for k in range(len(problems)):
                        inp, b, ref = problems[(k + t) % len(problems)]
                        x, _ = _solve(inp, b, "fp64" if (k + rep) % 2 else "fp32")
                        errs.append(_err(x, ref))
        except Exception as e:  # a thread's failure is the test's
            fails.append(e)

    ts = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not fails, fails
    assert len(errs) == threads * 24 and max(errs) < 1e-12


def test_release_waits_for_y_big():
    inp, b, _ = _problem(2)
    ref = O.y_big(O.factor(O.from_inputs(inp)))
    for k in range(5):
        with torch.cuda.stream(torch.cuda.Stream()):
            _, Y = _solve(inp, b, "fp64")
        other, bo, want = _problem(k)  # takes the released blocks at once
        x, _ = _solve(other, bo, "fp64")
        assert _err(x, want) < 1e-12
        torch.cuda.synchronize()
        assert _err(Y.cpu().numpy().T, ref) < 1e-12


def test_y_big_queued_at_release_is_not_overwritten():
    """The factorization is released while work in front of Y_big is still
    running; a problem of the same size takes its blocks on another stream."""
    from paper_2208_06290_amd import hodlr
    inp, _, _ = _problem(2)
    ref = O.y_big(O.factor(O.from_inputs(inp)))
    A = hodlr.HODLRMatrix.from_inputs(inp.to(DEV))
    B = hodlr.HODLRMatrix(A.D.clone(), 3.0 * A.U, A.V.clone(), A.ranks)
    ahead = torch.randn(4096, 4096, device=DEV)
    torch.cuda.synchronize()
    s, t = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(4):
        with torch.cuda.stream(s):
            F = hodlr.factor(A, "fp64")
            for _ in range(40):  # some milliseconds
                ahead = (ahead @ ahead).clamp_(-1.0, 1.0)
            Y = F.y_big()
            del F
        with torch.cuda.stream(t):
            G = hodlr.factor(B, "fp64")
        torch.cuda.synchronize()
        assert _err(Y.cpu().numpy().T, ref) < 1e-12
        del G
