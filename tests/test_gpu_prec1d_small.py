"""The two-mode preconditioner on grids of up to 48 x 48 (FP32: 64 x 64) points, which
runs as one launch: at the edges of the 16 x 16 MFMA blocks, with unequal modes, strided
blocks and sizes past the rule.  Bars as for the other
preconditioner kernels against the oracle's Bartels-Stewart solve: FP64 1e-10,
FP32 2e-5 (normwise)."""
import numpy as np
import pytest

from gpu_util import need_gpu, say, to_dev
from oracle import physics, problem
from workloads import normal_block

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nvec,pad", [
    ((2, 2), 1, 0), ((3, 16), 2, 1), ((16, 16), 5, 0), ((17, 5), 3, 2), ((31, 33), 4, 1),
    ((32, 32), 4, 0), ((48, 48), 3, 1), ((49, 47), 16, 0), ((64, 9), 1, 3), ((63, 64), 7, 1),
    ((64, 64), 2, 0), ((65, 64), 2, 0),
])
def test_prec_small_grid(n, nvec, pad, prec):
    import torch
    t3 = need_gpu()
    L = (7.0, 6.0)
    cx, cy, mu = physics.coeffs_unit_heavy(20.0)
    P = problem.make_problem(ndim=1, n=n, L=L, alpha=20.0, v0=2.5, width=0.9, shape="gauss")
    op = t3.Operator(1, list(n), list(L), cx, cy, v0=2.5, width=0.9, mu_hl=mu, sigma=P.two_body_shift())
    dt, pk, bar = (torch.float64, t3.FP64, 1e-10) if prec == "fp64" else (torch.float32, t3.FP32, 2e-5)
    buf = torch.full((2, nvec, P.N + pad), 7.0, dtype=dt, device="cuda")
    X, Y = buf[0, :, :P.N], buf[1, :, :P.N]
    X.copy_(to_dev(normal_block(P.N, nvec, 11 + n[0]), dt))
    say("prec small grid", n, prec)
    op.apply_prec(X, Y, prec=pk)
    torch.cuda.synchronize()
    want = P.preconditioner(sigma=op.sigma).apply(X.double().cpu().numpy().T).T
    err = np.linalg.norm(Y.double().cpu().numpy() - want) / np.linalg.norm(want)
    say("  rel err", err)
    assert err <= bar
    assert (buf[:, :, P.N:] == 7.0).all()
    op.close()
