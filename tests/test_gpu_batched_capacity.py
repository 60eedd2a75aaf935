"""A grouped preconditioner apply over 12,000 instances of all three forms (one
launch, plain products, folded products) has room in the library's job tables, and
every instance gets the result of its own apply bit for bit.

The instances of a form share one operator and one input block, so their
intermediates, which share the operator's work buffer, are the same values."""
import pytest

from gpu_util import need_gpu, say, to_dev
from oracle import physics
from workloads import normal_block

pytestmark = pytest.mark.gpu


def test_many_mixed_instances():
    import torch
    t3 = need_gpu()
    cx, cy, mu = physics.coeffs_unit_heavy(7.0)
    each, ops, Xs, Ys, one = 4000, [], [], [], []
    for n in [(20, 24), (96, 96), (182, 182)]:
        op = t3.Operator(1, list(n), [9.0, 6.0], cx, cy, v0=1.5, width=0.8, mu_hl=mu, sigma=-0.4)
        X = to_dev(normal_block(op.N, 1, n[0]))
        Y = torch.zeros((each, op.N), dtype=X.dtype, device="cuda")
        ops += [op] * each
        Xs += [X] * each
        Ys += [Y[i:i + 1] for i in range(each)]
        one.append((op, X, Y))
    say("grouped preconditioner", len(ops), "instances")
    t3.apply_prec_batched(ops, Xs, Ys)
    torch.cuda.synchronize()
    for op, X, Y in one:
        Z = torch.empty_like(X)
        op.apply_prec(X, Z)
        torch.cuda.synchronize()
        assert (Y == Z).all()
