"""The BF16x3 preconditioner makes the splitting errors of eigen-factors with columns
of length 1: its error against the oracle is compared with that of the same four
products emulated in NumPy with such factors.

Which bits a split cuts depends on the scale of the value, so factors of another
scale (columns longer by sqrt 2, say) give errors of about the same size that have
nothing to do with these: emulated on the three grids, correlations of -0.11, -0.03
and 0.17, against 0.96, 0.97 and 0.95 when only the sums are rounded in another way
(FP32 after each 32 products instead of at the end).  Bar: 0.8."""
import numpy as np
import pytest

from gpu_util import need_gpu, say, to_dev
from oracle import physics, problem
from workloads import normal_block

pytestmark = pytest.mark.gpu


def _fp32(a):
    return a.astype(np.float32).astype(np.float64)


def _split(a):
    """bf16 (round to nearest even) hi and lo of FP32 values."""
    def bf16(x):
        u = x.astype(np.float32).view(np.uint32).astype(np.uint64)
        return ((u + 0x7fff + ((u >> 16) & 1)) >> 16 << 16).astype(np.uint32).view(np.float32).astype(np.float64)
    a = np.ascontiguousarray(_fp32(a))
    hi = bf16(a)
    return hi, bf16(a - hi)


def _mul(A, B):
    (ah, al), (bh, bl) = _split(A), _split(B)
    return np.matmul(ah, bh) + np.matmul(ah, bl) + np.matmul(al, bh)


def _factors(K):
    lam, S = np.linalg.eig(K)
    lam, S = lam.real, S.real / np.linalg.norm(S.real, axis=0)
    return lam, S, np.linalg.inv(S)


@pytest.mark.parametrize("nx,ny,nvec", [(128, 96, 4), (65, 128, 3), (256, 256, 8)])
def test_prec_error_is_that_of_unit_factors(nx, ny, nvec):
    import torch
    t3 = need_gpu()
    cx, cy, mu = physics.coeffs_unit_heavy(7.0)
    P = problem.make_problem(ndim=1, n=(nx, ny), L=(9.0, 6.0), alpha=7.0, v0=1.5, width=0.8)
    op = t3.Operator(1, [nx, ny], [9.0, 6.0], cx, cy, v0=1.5, width=0.8, mu_hl=mu, sigma=-0.4)
    Xn = _fp32(normal_block(P.N, nvec, 5))
    X = to_dev(Xn, torch.float32)
    Y = torch.empty_like(X)
    say("bf16x3 preconditioner", nx, ny, nvec)
    op.apply_prec(X, Y, prec=t3.BF16X3)
    torch.cuda.synchronize()
    want = P.preconditioner(sigma=op.sigma).apply(Xn.T).T
    lx, Sx, Six = _factors(-P.cx * P.D2[0])
    ly, Sy, Siy = _factors(-P.cy * P.D2[1])
    Z = _fp32(_mul(Six, Xn.reshape(nvec, nx, ny)))
    Z = _fp32(_mul(Z, Siy.T.copy()) / (lx[:, None] + ly[None, :] - op.sigma))
    Z = _fp32(_mul(_fp32(_mul(Sx, Z)), Sy.T.copy()))
    err = Y.double().cpu().numpy() - want
    emu = Z.reshape(nvec, -1) - want
    corr = np.sum(err * emu) / np.linalg.norm(err) / np.linalg.norm(emu)
    say("  errors", np.linalg.norm(err) / np.linalg.norm(want), np.linalg.norm(emu) / np.linalg.norm(want),
        "correlation", corr)
    assert corr >= 0.8
    op.close()
