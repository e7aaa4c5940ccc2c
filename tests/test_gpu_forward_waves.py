"""The forward pass's four-wave form (two-wave above 6400 nodes) at its edges,
against the FP64 oracle (1e-6 relative per output block): rows of alpha of 0 to
40 entries that start at even and odd places (pairs split over the waves, rows
past the entries loaded ahead), sequences that end around a batch and a
segment, spans too long for anchored records; gradient, log-likelihood and
intensities."""
import numpy as np
import pytest

import oracle
from tests.helpers import rand_problem, scalar_rel
from tests.test_gpu_parity import H, check, dev, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n,rate", [(70, 1, 5.0), (70, 64, 5.0), (70, 65, 5.0), (81, 1023, 20.0), (81, 1025, 20.0),
                                      (300, 5000, 50.0), (70, 3000, 0.2), (6401, 400, 50.0)])
def test_forward_rows(H, M, n, rate):  # noqa: F811
    import torch
    rng = np.random.default_rng(M + n)
    t, m, mu, _, beta, T = rand_problem(600 + M + n, n, min(M, 400), ties=True, density=0.1, rate=rate)
    mu = rng.uniform(0.05, 0.5, M).astype(np.float32)
    alpha = np.zeros((M, M), np.float32)
    for p in range(M):
        k = p % 41
        alpha[p, rng.choice(min(M, 400), k, replace=False)] = rng.uniform(0.0, 0.02, k)
    ref = oracle.forward(t, m, mu, alpha, beta, T)
    check(run_gpu(H, t, m, mu, alpha, beta, T, 0), ref, label=f"forward M={M} n={n}")
    args = (dev(t, torch.float64), dev(m, torch.int32), dev(mu, torch.float32), dev(alpha, torch.float32),
            dev(beta, torch.float32), T)
    assert scalar_rel(H.loglik(*args).item(), ref[0]) < 1e-6
    lam = H.intensity(*args).cpu().numpy()
    idx = np.unique(np.linspace(0, n - 1, 70).astype(np.int64))
    lref = oracle.intensity_at(t, m, mu, alpha, beta, idx)
    assert np.max(np.abs(lam[idx] - lref) / lref) < 1e-6
