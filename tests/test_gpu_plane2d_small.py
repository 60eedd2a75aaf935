"""The four-mode applies with modes up to 48, which run one matrix per wave: at
the edges of the 16 x 16 MFMA blocks and of the K steps of four, mixed with
modes of the other side of the line at 48, group counts that do not divide by the
matrices of a workgroup, unequal boxes, shifts, a tabulated potential and
strided blocks.

Bars (relative, normwise): FP64 1e-12 and FP32 1e-5 for the Hamiltonian against
the oracle's tensor apply; 1e-10 and 2e-5 for the preconditioner, which is
applied in the eigenbases of the mode operators, against the oracle's
Bartels-Stewart solve."""
import numpy as np
import pytest

from gpu_util import need_gpu, say, to_dev
from oracle import physics, problem
from workloads import normal_block

pytestmark = pytest.mark.gpu

# (nx, ny), boxes of the four modes
SHAPES = [
    ((2, 5), (5.0, 4.0, 5.0, 6.0)),
    ((4, 3), (5.0, 5.0, 5.0, 5.0)),
    ((8, 9), (6.0, 5.5, 5.0, 5.0)),
    ((12, 13), (6.0, 6.0, 5.0, 6.0)),
    ((15, 17), (8.0, 8.0, 7.0, 7.0)),
    ((16, 16), (8.0, 7.0, 7.0, 8.0)),
    ((20, 21), (8.0, 8.0, 8.0, 8.0)),
    ((25, 7), (9.0, 8.0, 5.0, 5.0)),
    ((32, 11), (9.0, 9.0, 5.0, 5.0)),
    ((33, 6), (9.0, 9.5, 5.0, 5.0)),
    ((6, 41), (5.0, 5.0, 9.0, 9.5)),
    ((48, 5), (12.0, 12.0, 5.0, 5.0)),
    ((5, 48), (5.0, 5.0, 12.0, 11.0)),
    ((49, 4), (12.0, 11.0, 5.0, 5.0)),
    ((6, 63), (5.0, 5.0, 12.0, 12.0)),
]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("k", range(len(SHAPES)))
def test_small_modes(k, prec):
    import torch
    t3 = need_gpu()
    (nx, ny), L = SHAPES[k]
    n = (nx, nx, ny, ny)
    cx, cy, mu = physics.coeffs_unit_heavy(20.0)
    P = problem.make_problem(ndim=2, n=n, L=L, alpha=20.0, v0=2.5, width=0.9, shape="gauss")
    kw = dict(pot="table", V_table=P.V.ravel()) if k % 2 else dict(pot="gauss", v0=2.5, width=0.9)
    op = t3.Operator(2, list(n), list(L), cx, cy, sigma=P.two_body_shift(), mu_hl=mu, **kw)
    pk, dt, bars = ((t3.FP64, torch.float64, (1e-12, 1e-10)) if prec == "fp64"
                    else (t3.FP32, torch.float32, (1e-5, 2e-5)))
    nvec, pad = 3, k % 3
    Xn = normal_block(P.N, nvec, 40 + k)
    buf = torch.full((2, nvec, P.N + pad), 7.0, dtype=dt, device="cuda")
    X, Y = buf[0, :, :P.N], buf[1, :, :P.N]
    X.copy_(to_dev(Xn, dt))
    ref = X.double().cpu().numpy()
    shifts = np.array([0.3, -1.2, 0.0]) if k % 2 else None
    say("small modes", n, prec)
    op.apply_H(X, Y, prec=pk, shifts=None if shifts is None else to_dev(shifts))
    torch.cuda.synchronize()
    want = P.apply(ref.T).T
    if shifts is not None:
        want = want - shifts[:, None] * ref
    err = np.linalg.norm(Y.double().cpu().numpy() - want) / np.linalg.norm(want)
    op.apply_prec(X, Y, prec=pk)
    torch.cuda.synchronize()
    want = P.preconditioner(sigma=op.sigma).apply(ref.T).T
    perr = np.linalg.norm(Y.double().cpu().numpy() - want) / np.linalg.norm(want)
    say("  H", err, "P", perr)
    assert err <= bars[0] and perr <= bars[1]
    assert (buf[:, :, P.N:] == 7.0).all()
    op.close()


@pytest.mark.parametrize("nx,pad", [(3, 0), (5, 2), (28, 0)])
def test_full_equal_planes_prec(nx, pad):
    """Full 64 x 64 y planes with equal modes (FP64: the factor in registers), fewer
    and more planes than workgroups, and a strided block; bar as above."""
    import torch
    t3 = need_gpu()
    n, L = (nx, nx, 64, 64), (5.0, 5.0, 9.0, 9.0)
    cx, cy, mu = physics.coeffs_unit_heavy(20.0)
    P = problem.make_problem(ndim=2, n=n, L=L, alpha=20.0, v0=2.5, width=0.9, shape="gauss")
    op = t3.Operator(2, list(n), list(L), cx, cy, v0=2.5, width=0.9, sigma=P.two_body_shift(), mu_hl=mu)
    buf = torch.full((2, 2, P.N + pad), 7.0, dtype=torch.float64, device="cuda")
    X, Y = buf[0, :, :P.N], buf[1, :, :P.N]
    X.copy_(to_dev(normal_block(P.N, 2, 50 + nx)))
    say("full equal planes", n)
    op.apply_prec(X, Y)
    torch.cuda.synchronize()
    want = P.preconditioner(sigma=op.sigma).apply(X.cpu().numpy().T).T
    err = np.linalg.norm(Y.cpu().numpy() - want) / np.linalg.norm(want)
    say("  P", err)
    assert err <= 1e-10
    assert (buf[:, :, P.N:] == 7.0).all()
    op.close()
