"""GPU parity of the folded preconditioner products (grids of more than 32,768 points)
where they can go wrong: odd sizes in either mode and in both (the middle row or
column is its own mirror), rows of 1, 2 and 3 entries past a multiple of four, a very
unequal pair, single vectors, leading dimensions that misalign every second vector,
and every tile shape.  Grouped applies with instances of all forms equal the single
ones bit for bit.

Bars: normwise per vector 1e-10 (FP64) and 2e-5 (FP32) against the oracle, as for the
other preconditioner kernels."""
import functools

import numpy as np
import pytest

from gpu_util import need_gpu, say, to_dev
from oracle import physics, problem
from workloads import normal_block

pytestmark = pytest.mark.gpu

SIZES = [(200, 165, 1), (181, 182, 2), (182, 183, 3), (301, 190, 3), (190, 301, 1), (257, 129, 2), (192, 192, 3),
         (33, 1002, 2), (1001, 34, 2)]


def _make(t3, nx, ny):
    cx, cy, mu = physics.coeffs_unit_heavy(7.0)
    return t3.Operator(1, [nx, ny], [9.0, 6.0], cx, cy, v0=1.5, width=0.8, mu_hl=mu, sigma=-0.4)


@functools.lru_cache(maxsize=2)
def _reference(nx, ny, nvec):
    P = problem.make_problem(ndim=1, n=(nx, ny), L=(9.0, 6.0), alpha=7.0, v0=1.5, width=0.8)
    X = normal_block(P.N, nvec, 3 * nx + ny).astype(np.float32).astype(np.float64)
    return X, P.preconditioner(sigma=-0.4).apply(X.T).T


@pytest.mark.parametrize("nx,ny,nvec", SIZES)
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_folded_at_edges(nx, ny, nvec, prec):
    import torch
    t3 = need_gpu()
    assert nx * ny > 32768
    Xn, want = _reference(nx, ny, nvec)
    op = _make(t3, nx, ny)
    dt, bar = (torch.float64, 1e-10) if prec == "fp64" else (torch.float32, 2e-5)
    for pad in (0, 1):
        buf = torch.full((2, nvec, op.N + pad), 7.0, dtype=dt, device="cuda")
        X, Y = buf[0, :, :op.N], buf[1, :, :op.N]
        X.copy_(to_dev(Xn, dt))
        for tile in (-1, 0, 1, 2, 3, 4):
            op.set_tile(tile)
            Y.fill_(7.0)
            say("folded", nx, ny, nvec, prec, "pad", pad, "tile", tile)
            op.apply_prec(X, Y)
            torch.cuda.synchronize()
            err = np.max(np.linalg.norm(Y.double().cpu().numpy() - want, axis=1) / np.linalg.norm(want, axis=1))
            say("  rel err", err)
            assert err <= bar
            assert (buf[:, :, op.N:] == 7.0).all()
    op.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("tile", [-1, 2, 4])
def test_grouped_equals_single(prec, tile):
    import torch
    t3 = need_gpu()
    dt = torch.float64 if prec == "fp64" else torch.float32
    ops = [_make(t3, *n) for n in [(257, 129), (40, 33), (130, 70), (182, 183), (16, 16), (192, 192), (64, 100)]]
    Xs = [to_dev(normal_block(op.N, 3, i), dt) for i, op in enumerate(ops)]
    Ys = [torch.empty_like(X) for X in Xs]
    for op in ops[::2]:
        op.set_tile(tile)
    say("grouped forms", prec, "tile", tile)
    t3.apply_prec_batched(ops, Xs, Ys)
    torch.cuda.synchronize()
    for i, (op, X, Y) in enumerate(zip(ops, Xs, Ys)):
        Z = torch.empty_like(X)
        op.apply_prec(X, Z)
        torch.cuda.synchronize()
        assert torch.equal(Y, Z), (i, op.n)
    for op in ops:
        op.close()
