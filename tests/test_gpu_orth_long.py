"""Block orthogonalisation of long blocks (N >= 2^20) at the edges of its fused
passes: rows that do not divide by a step, one and two 8-column solves, bases of
0 to 80 columns (the norms come with the first dot up to 80 columns in all),
leading dimensions that rule the aligned passes out, and a dependent column.

Bars from the method: twice-run Gram-Schmidt and Cholesky-QR leave
|X^T X - 1| and |Q^T X| at rounding, taken as 1e-13 here (2^20 products of size
2^-20 with errors of 1e-16 each); the span stays that of the projected block, to
1e-11 for a block whose condition number is below 1e3."""
import numpy as np
import pytest

from gpu_util import need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,nq,nx,pad", [
    (1 << 20, 40, 8, 0), ((1 << 20) + 37, 40, 8, 1), ((1 << 20) + 37, 16, 9, 0), ((1 << 20) + 1, 3, 16, 1),
    ((1 << 20) + 255, 64, 16, 1), ((1 << 20) + 2, 65, 16, 0), ((1 << 20) + 64, 80, 1, 0), ((1 << 20) + 65, 0, 16, 0),
    ((1 << 20) + 63, 0, 1, 0), ((1 << 20) + 3, 24, 8, 0),
])
def test_orth_long(N, nq, nx, pad):
    import torch
    t3 = need_gpu()
    g = torch.Generator(device="cuda").manual_seed(7 + nq + nx)
    buf = torch.randn(nq + nx, N + pad, dtype=torch.float64, device="cuda", generator=g)
    Q, X = buf[:nq, :N], buf[nq:, :N]
    if nq:
        for _ in range(2):
            Q.copy_(torch.linalg.inv(torch.linalg.cholesky(Q @ Q.T)) @ Q)
    X0 = X.clone()
    say("orth long", N, nq, nx, pad)
    _, _, rank = t3.block_orth(Q if nq else None, X, want_factors=False)
    torch.cuda.synchronize()
    assert rank == nx
    eye = torch.eye(nx, dtype=torch.float64, device="cuda")
    assert float((X @ X.T - eye).abs().max()) <= 1e-13
    if nq:
        assert float((Q @ X.T).abs().max()) <= 1e-13
        X0 = X0 - (X0 @ Q.T) @ Q
    # the projected block lies in the span of the result
    assert float((X0 - (X0 @ X.T) @ X).norm() / X0.norm()) <= 1e-11


def test_orth_long_dependent_column():
    import torch
    t3 = need_gpu()
    N, nq, nx = (1 << 20) + 5, 30, 10
    buf = torch.randn(nq + nx, N + 1, dtype=torch.float64, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(3))
    Q, X = buf[:nq, :N], buf[nq:, :N]
    for _ in range(2):
        Q.copy_(torch.linalg.inv(torch.linalg.cholesky(Q @ Q.T)) @ Q)
    X[4] = 2.0 * X[1] - X[2]
    say("orth long, dependent column")
    _, _, rank = t3.block_orth(Q, X, want_factors=False)
    torch.cuda.synchronize()
    assert rank == nx - 1
    assert float((X @ X.T - torch.eye(nx, dtype=torch.float64, device="cuda")).abs().max()) <= 1e-13
    assert float((Q @ X.T).abs().max()) <= 1e-13
