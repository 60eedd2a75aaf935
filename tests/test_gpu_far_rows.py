"""2D operators whose first x pass has rows so long that a chunk of them passes
the reach of 32-bit byte offsets (n_x n_y^2 >= 33,552,384 entries): both applies
run, in FP64 and FP32.  The y modes have diagonal second-derivative matrices, so
the reference needs products along the two x modes only, formed on the device in
FP64.

Bars: H componentwise 4 (n_x + 2) units of |K||W| (the sums have 2 n_x + 2 terms),
the preconditioner normwise 1e-10 / 2e-5 as in the other preconditioner tests."""
import numpy as np
import pytest

from gpu_util import need_gpu, say

pytestmark = pytest.mark.gpu

NX, NY = 8, 2049


def _x_modes(A, W):
    """A applied along each of the two leading modes of W, one after the other."""
    import torch
    out = []
    for m in (0, 1):
        r = torch.zeros_like(W)
        for i in range(NX):
            for k in range(NX):
                r.select(m, i).add_(W.select(m, k), alpha=float(A[i, k]))
        out.append(r)
    return out


@pytest.fixture(scope="module")
def far_op():
    t3 = need_gpu()
    say("far rows: create", NX, NY)
    cy, dy = 2.0, [np.linspace(0.5, 3.0, NY), np.linspace(1.0, 2.0, NY)]
    op = t3.Operator(2, [NX, NX, NY, NY], [3.0, 3.0, 5.0, 5.0], 1.5, cy, sigma=-0.4,
                     V_table=np.zeros(NX * NX * NY * NY), D2=[None, None, np.diag(-dy[0]), np.diag(-dy[1])])
    say("  created")
    yield op, -1.5 * op.D2(0), cy * dy[0][:, None] + cy * dy[1][None, :]
    op.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_far_rows(far_op, prec):
    import torch
    op, Kx, ky = far_op
    dt, eps, pbar = (torch.float64, 2.2e-16, 1e-10) if prec == "fp64" else (torch.float32, 6e-8, 2e-5)
    g = torch.Generator(device="cuda").manual_seed(11)
    X = torch.randn((1, op.N), dtype=dt, device="cuda", generator=g)
    Y = torch.empty_like(X)
    say("far rows: H", prec)
    op.apply_H(X, Y)
    torch.cuda.synchronize()
    W = X[0].double().view(NX, NX, NY, NY)
    ky = torch.from_numpy(ky).cuda()
    ref = sum(_x_modes(Kx, W)) + ky * W
    scale = sum(_x_modes(abs(Kx), W.abs())) + ky * W.abs()
    herr = ((Y[0].double().view_as(W) - ref).abs_() / scale).max().item()
    say("  componentwise", herr)
    assert herr <= 4 * (NX + 2) * eps
    del ref, scale
    say("far rows: preconditioner", prec)
    op.apply_prec(X, Y)
    torch.cuda.synchronize()
    lam, S = np.linalg.eig(Kx)
    lam, S = lam.real, S.real
    Z = W
    for m in (0, 1):
        Z = _x_modes(np.linalg.inv(S), Z)[m]
    lx = torch.from_numpy(lam[:, None] + lam[None, :]).cuda()
    Z = Z / (lx[:, :, None, None] + ky - op.sigma)
    for m in (0, 1):
        Z = _x_modes(S, Z)[m]
    perr = ((Y[0].double().view_as(W) - Z).norm() / Z.norm()).item()
    say("  normwise", perr)
    assert perr <= pbar
