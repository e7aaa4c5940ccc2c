"""The one-kernel engine for 9 to 64 nodes and one shared decay at its edges,
against the FP64 oracle (1e-6 relative per output block): node counts around
the lane groups of 16, 32 and 64; sequences that end inside a group's batch, at
a group, a segment and a pair of segments, and over several chunks; rates at
which no batch, some batches and every batch are walked with per-event decays
(beta times the batch's span above 600).  The gradient, the log-likelihood and
the intensity forms."""
import numpy as np
import pytest

import oracle
from tests.helpers import rand_problem, scalar_rel
from tests.test_gpu_parity import H, check, dev, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n,chunk,rate", [(9, 1, 0, 5.0), (10, 17, 0, 5.0), (15, 63, 0, 5.0), (16, 64, 0, 5.0),
                                            (17, 65, 0, 5.0), (31, 127, 0, 20.0), (32, 129, 0, 20.0),
                                            (33, 255, 0, 20.0), (63, 1023, 0, 20.0), (64, 1024, 0, 20.0),
                                            (16, 1025, 0, 20.0), (32, 2047, 0, 20.0), (64, 2049, 0, 20.0),
                                            (12, 9000, 12, 0.02), (30, 9000, 12, 0.05), (50, 9000, 12, 0.1),
                                            (16, 4100, 12, 0.5), (64, 12289, 12, 0.1)])
def test_narrow_engine(H, M, n, chunk, rate):  # noqa: F811
    import torch
    t, m, mu, alpha, beta, T = rand_problem(700 + M + n, n, M, ties=True, density=0.5, rate=rate)
    ref = oracle.forward(t, m, mu, alpha, beta, T)
    check(run_gpu(H, t, m, mu, alpha, beta, T, chunk), ref, label=f"narrow M={M} n={n} rate={rate}")
    args = (dev(t, torch.float64), dev(m, torch.int32), dev(mu, torch.float32), dev(alpha, torch.float32),
            dev(beta, torch.float32), T, chunk)
    assert scalar_rel(H.loglik(*args).item(), ref[0]) < 1e-6
    lam = H.intensity(*args).cpu().numpy()
    idx = np.unique(np.linspace(0, n - 1, 70).astype(np.int64))
    lref = oracle.intensity_at(t, m, mu, alpha, beta, idx)
    assert np.max(np.abs(lam[idx] - lref) / lref) < 1e-6
