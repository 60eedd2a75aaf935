"""The preconditioner's work buffer on grids whose products are folded: no more
device memory than 64 vectors in FP64 and FP32, and applies of more vectors than
the buffer holds folded (about half of that), single, grouped and in the batched
eigensolver.

Bars: preconditioner normwise 1e-10 / 2e-5 as in the other preconditioner tests;
a grouped apply equals the single one bit for bit; eigenvalues 1e-10."""
import numpy as np
import pytest

from gpu_util import need_gpu, say, to_dev
from oracle import physics, problem
from workloads import normal_block

pytestmark = pytest.mark.gpu


def _make(t3, nx, ny):
    cx, cy, mu = physics.coeffs_unit_heavy(7.0)
    P = problem.make_problem(ndim=1, n=(nx, ny), L=(9.0, 6.0), alpha=7.0, v0=1.5, width=0.8)
    return t3.Operator(1, [nx, ny], [9.0, 6.0], cx, cy, v0=1.5, width=0.8, mu_hl=mu, sigma=-0.4), P


def test_work_memory():
    import torch
    t3 = need_gpu()
    _make(t3, 182, 182)[0].close()  # the library's and the runtime's own first allocations
    n = 512
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    op, _ = _make(t3, n, n)
    taken = free0 - torch.cuda.mem_get_info()[0]
    work = 64 * op.N * (8 + 4)
    # besides: the potential and about forty n x n matrices and fragment arrays
    rest = op.N * 12 + 40 * n * n * 12
    say("device memory of an operator", n, taken / 2**20, "MiB, of which work", work / 2**20)
    assert taken <= work + rest
    op.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,nvec", [(182, 182, 33), (257, 129, 31), (257, 129, 64), (257, 129, 100)])
def test_more_vectors_than_the_buffer_folds(nx, ny, nvec, prec):
    import torch
    t3 = need_gpu()
    op, P = _make(t3, nx, ny)
    dt, pbar = (torch.float64, 1e-10) if prec == "fp64" else (torch.float32, 2e-5)
    X = to_dev(normal_block(P.N, nvec, nx + nvec), dt)
    Y = torch.empty_like(X)
    say("folded in groups", nx, ny, nvec, prec)
    op.apply_prec(X, Y)
    torch.cuda.synchronize()
    want = P.preconditioner(sigma=op.sigma).apply(X.double().cpu().numpy().T).T
    err = np.max(np.linalg.norm(Y.double().cpu().numpy() - want, axis=1) / np.linalg.norm(want, axis=1))
    say("  rel err, worst vector", err)
    assert err <= pbar
    if nvec <= 64:
        small, _ = _make(t3, 40, 33)
        Xs = [X, to_dev(normal_block(small.N, nvec, 3), dt)]
        Ys = [torch.empty_like(x) for x in Xs]
        t3.apply_prec_batched([op, small], Xs, Ys)
        torch.cuda.synchronize()
        assert torch.equal(Ys[0], Y)
        small.close()
    op.close()
