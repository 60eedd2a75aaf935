"""GPU parity of the 1D mode products where their tiles can go wrong: sizes below,
at and one past the MFMA blocks, the tiles and the K chunks, odd sizes (the
middle entry of a folded mode is its own mirror; rows that are no whole number
of 16-byte pieces), leading dimensions that misalign every second vector, and
single vectors.  Every size runs the Hamiltonian apply (plain products) and the
preconditioner (one launch on the smallest, folded products above 32,768 points,
plain products between and on a parity half grid), in FP64 and FP32.

Bars: H within n-term rounding of NumPy's FP64 products with the same matrices,
componentwise 4 (n_x + n_y + 1) units of |H||W| on N(0,1) blocks; the preconditioner within the
1e-10 (FP64) and 1e-4 (FP32) of the other preconditioner tests."""
import numpy as np
import pytest

from gpu_util import need_gpu, say, to_dev
from oracle import physics, problem
from workloads import normal_block

pytestmark = pytest.mark.gpu

SIZES = [(2, 3, 1), (3, 2, 2), (5, 7, 3), (15, 16, 2), (17, 31, 3), (32, 33, 2), (63, 65, 2), (64, 128, 1),
         (127, 129, 2), (130, 257, 3), (256, 256, 2), (301, 94, 2)]


def _check(op, P, nvec, pad, dt, eps, pbar):
    import torch
    Xn = normal_block(P.N, nvec, 7 * P.N + nvec).astype(np.float32).astype(np.float64)
    buf = torch.zeros((nvec, P.N + pad), dtype=dt, device="cuda")
    buf[:, :P.N] = to_dev(Xn, dt)
    out = torch.full((nvec, P.N + pad), 7.0, dtype=dt, device="cuda")
    op.apply_H(buf[:, :P.N], out[:, :P.N])
    Y = out.double().cpu().numpy()
    nx, ny = P.n
    # the products alone: the reference takes the library's matrices and potential
    Kx, Ky, V = -P.cx * op.D2(0), -P.cy * op.D2(1), op.V().reshape(nx, ny)
    W = Xn.reshape(nvec, nx, ny)
    ref = np.matmul(Kx, W) + np.matmul(W, Ky.T) + V * W
    scale = np.matmul(abs(Kx), abs(W)) + np.matmul(abs(W), abs(Ky).T) + abs(V) * abs(W)
    herr = np.max(np.abs(Y[:, :P.N].reshape(W.shape) - ref) / scale)
    op.apply_prec(buf[:, :P.N], out[:, :P.N])
    Z = out.double().cpu().numpy()
    Zr = P.preconditioner(sigma=op.sigma).apply(Xn.T).T
    perr = np.linalg.norm(Z[:, :P.N] - Zr) / np.linalg.norm(Zr)
    say("  H componentwise", herr, "prec", perr)
    assert np.all(Y[:, P.N:] == 7.0) and np.all(Z[:, P.N:] == 7.0)
    assert herr <= 4 * (nx + ny + 1) * eps
    assert perr <= pbar


@pytest.mark.parametrize("nx,ny,nvec", SIZES)
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_mode_products_at_edges(nx, ny, nvec, prec):
    import torch
    t3 = need_gpu()
    cx, cy, mu = physics.coeffs_unit_heavy(7.0)
    P = problem.make_problem(ndim=1, n=(nx, ny), L=(9.0, 6.0), alpha=7.0, v0=1.5, width=0.8)
    op = t3.Operator(1, [nx, ny], [9.0, 6.0], cx, cy, v0=1.5, width=0.8, mu_hl=mu, sigma=-0.4)
    dt, eps, pbar = (torch.float64, 2.2e-16, 1e-10) if prec == "fp64" else (torch.float32, 6e-8, 1e-4)
    for pad in (0, 1):
        say("mode products", nx, ny, nvec, prec, "pad", pad)
        _check(op, P, nvec, pad, dt, eps, pbar)


@pytest.mark.parametrize("nx,ny,nvec", [(17, 31, 3), (64, 32, 2), (130, 70, 2)])
@pytest.mark.parametrize("parity", [(1, 1), (-1, 1), (0, 1)])
def test_mode_products_on_half_grids(nx, ny, nvec, parity):
    """Operators without the reflection symmetry in at least one mode: nothing is
    folded."""
    import torch
    t3 = need_gpu()
    P = problem.make_problem(ndim=1, n=(nx, ny), L=(6.0, 3.0), alpha=20.0, v0=0.35, shape="gauss_paper",
                             units="paper", grid="mapped", parity=parity)
    op = t3.Operator(1, [nx, ny], [6.0, 3.0], P.cx, P.cy, pot="gauss_paper", v0=0.35, mu_hl=P.mu_hl,
                     grid="mapped", parity=parity, sigma=-0.1)
    X = to_dev(normal_block(P.N, nvec, 91))
    Y, Z = torch.empty_like(X), torch.empty_like(X)
    say("half grid", nx, ny, parity)
    op.apply_H(X, Y)
    op.apply_prec(X, Z)
    Xn = X.cpu().numpy()
    Yr = P.apply(Xn.T).T
    Zr = P.preconditioner(sigma=op.sigma).apply(Xn.T).T
    assert np.linalg.norm(Y.cpu().numpy() - Yr) <= 1e-12 * np.linalg.norm(Yr)
    assert np.linalg.norm(Z.cpu().numpy() - Zr) <= 1e-10 * np.linalg.norm(Zr)
