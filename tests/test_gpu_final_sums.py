"""The final sums of the large-M engines with many nodes, against the FP64 oracle (1e-6 relative per output block):
the first node count with strips of 64 columns and its neighbours, sizes off the strips, several event ranges, one
chunk and several (the first stores its partials, the others add), the gradient and its restriction to the support,
decays per target, and no events at all."""
import numpy as np
import pytest
import torch

import oracle
from tests.helpers import rand_problem
from tests.test_gpu_parity import H, check, dev, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n,chunk,per_target", [(1023, 2_000, 0, False), (1024, 2_000, 0, False),
                                                  (1025, 9_000, 12, False), (1500, 3_000, 0, False),
                                                  (2111, 2_000, 0, False), (1025, 9_000, 12, True),
                                                  (1500, 30_000, 0, True), (300, 30_000, 12, True)])
def test_final_sums(H, M, n, chunk, per_target):  # noqa: F811
    p = rand_problem(M, n, M, per_target=per_target, ties=True, density=10.0 / M, rate=0.1 * M)
    ref = oracle.adjoint(*p) if per_target else oracle.forward(*p)
    check(run_gpu(H, *p, chunk), ref, label=f"M={M} n={n} per_target={per_target}")
    if not per_target:
        x = (dev(p[0], torch.float64), dev(p[1], torch.int32), *(dev(a, torch.float32) for a in p[2:5]), p[5], chunk)
        got = [a.cpu().numpy() for a in H.loglik_grad(*x, support=True)]
        check(got, (ref[0], ref[1], np.where(p[3] != 0, ref[2], 0.0), ref[3]), label=f"support M={M} n={n}")


@pytest.mark.parametrize("per_target", [False, True])
def test_no_events(H, per_target):  # noqa: F811
    M, T = 1100, 2.0
    mu, alpha = torch.full((M,), 0.1).cuda(), torch.full((M, M), 1e-4).cuda()
    beta = torch.ones(M if per_target else 1).cuda()
    t, m = torch.zeros(0, dtype=torch.float64).cuda(), torch.zeros(0, dtype=torch.int32).cuda()
    L, gmu, ga, gb = H.loglik_grad(t, m, mu, alpha, beta, T)
    assert abs(float(L) + T * float(mu.double().sum())) < 1e-6
    assert bool((gmu == -T).all()) and not bool(ga.any()) and not bool(gb.any())
