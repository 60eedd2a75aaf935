"""Preconditioner of operators with second-derivative matrices given by the caller:
whether it exists is decided by the spectrum of the whole matrix, also where the
matrix has the grid's reflection symmetry and its even and odd halves could be
factorised by themselves; with that symmetry (folded products) and without it
(plain ones) the result is the oracle's (normwise 1e-10 / 2e-5)."""
import numpy as np
import pytest

from gpu_util import need_gpu, say, to_dev
from oracle import physics, problem
from workloads import normal_block

pytestmark = pytest.mark.gpu


def _symmetric_with_shared_eigenvalues(n, seed):
    """K[i][j] = K[n-1-i][n-1-j] with the eigenvalues 2, 4, ... n in both halves."""
    r, m = np.random.default_rng(seed), n // 2
    even, odd = (Q @ np.diag(2.0 * np.arange(1, m + 1)) @ np.linalg.inv(Q)
                 for Q in (r.standard_normal((m, m)), r.standard_normal((m, m))))
    A, B = (even + odd) / 2, (even - odd) / 2
    return np.block([[A, B[:, ::-1]], [B[::-1, :], A[::-1, ::-1]]])


def test_complex_pair_of_the_whole_matrix_is_refused():
    t3 = need_gpu()
    n = 20
    K = _symmetric_with_shared_eigenvalues(n, 5)
    half = K[:n // 2, :n // 2], K[:n // 2, n // 2:][:, ::-1]
    # the rounding of the two coinciding eigenvalues: a complex pair in the whole, none in the halves
    assert np.any(t3.host_schur(K)[2].imag != 0)
    assert all(np.all(t3.host_schur(h)[2].imag == 0) for h in (half[0] + half[1], half[0] - half[1]))
    op = t3.Operator(1, [n, 24], [5.0, 5.0], 1.0, 2.0, v0=1.0, width=1.0, sigma=-0.4, D2=[-K, None])
    X = to_dev(normal_block(op.N, 2, 1))
    say("given matrix with a complex pair")
    with pytest.raises(t3.Tp3bError) as e:
        op.apply_prec(X, X.clone())
    assert e.value.code == -5  # TP3B_ENOTSUP
    op.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("symmetric", [(True, True), (True, False), (False, False)])
@pytest.mark.parametrize("nx,ny", [(200, 182), (191, 173), (30, 41)])
def test_given_matrices(nx, ny, symmetric, prec):
    import torch
    t3 = need_gpu()
    cx, cy, mu = physics.coeffs_unit_heavy(7.0)
    P = problem.make_problem(ndim=1, n=(nx, ny), L=(9.0, 6.0), alpha=7.0, v0=1.5, width=0.8)
    D2 = []
    for k, s in enumerate(symmetric):
        D = 0.5 * (P.D2[k] + P.D2[k][::-1, ::-1])
        if not s:
            D[0, 0] *= 1 + 1e-14
        D2.append(D)
    op = t3.Operator(1, [nx, ny], [9.0, 6.0], cx, cy, v0=1.5, width=0.8, mu_hl=mu, sigma=-0.4, D2=D2)
    dt, pbar = (torch.float64, 1e-10) if prec == "fp64" else (torch.float32, 2e-5)
    X = to_dev(normal_block(P.N, 3, nx), dt)
    Y = torch.empty_like(X)
    say("given matrices", nx, ny, symmetric, prec)
    op.apply_prec(X, Y)
    torch.cuda.synchronize()
    want = P.preconditioner(sigma=op.sigma).apply(X.double().cpu().numpy().T).T
    err = np.linalg.norm(Y.double().cpu().numpy() - want) / np.linalg.norm(want)
    say("  rel err", err)
    assert err <= pbar
    op.close()
