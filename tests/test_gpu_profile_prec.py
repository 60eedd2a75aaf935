"""With profiling on and no graph, the eigensolver times the preconditioner applies of every 1D
operator, also where they are one launch (the 32 x 32 workload): one timed group per
apply of up to `block` vectors, and the operator works as before afterwards."""
import pytest

from gpu_util import need_gpu, say
from workloads import config, normal_block

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inner", ["fp64", "fp32"])
def test_profile_times_the_preconditioner(inner):
    import torch
    t3 = need_gpu()
    cfg = config("c1")
    op = t3.Operator.from_config(cfg)
    X = torch.from_numpy(normal_block(op.N, 2, 1)).cuda()
    Y, Z = torch.empty_like(X), torch.empty_like(X)
    op.apply_prec(X, Y)
    r = op.jdqr(cfg["nev"], cfg["block"], seed=cfg["seed_start"], profile=True, graph=False,
                inner_prec=t3.FP64 if inner == "fp64" else t3.FP32)
    k = 2 if inner == "fp64" else 3
    n, v, t = r.stats["n_kernel"][k], r.stats["v_kernel"][k], r.stats["t_kernel"][k]
    say("profiled preconditioner", inner, n, v, t)
    assert 0 < n <= v <= n * cfg["block"]
    assert 0 < t < r.stats["t_total"]
    op.apply_prec(X, Z)
    torch.cuda.synchronize()
    assert torch.equal(Y, Z)
    op.close()
