"""A batch whose larger sequence has one node less than max_m, in exactly the
workspace that the query names, against the FP64 oracle (1e-6 relative per
output block)."""
import types

import numpy as np
import pytest

import oracle
from tests.helpers import rand_problem
from tests.test_gpu_parity import H, check  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ms,lens", [((80, 81), (100_000, 10)), ((128, 129), (1_000, 10)), ((5, 64, 65), (50, 9_000, 7))])
def test_batch_in_the_queried_workspace(H, ms, lens):  # noqa: F811
    ps = [rand_problem(500 + m, n, m, density=0.2, rate=20.0) for m, n in zip(ms, lens)]
    cat = lambda k, dt: np.concatenate([np.asarray(p[k], dt).reshape(-1) for p in ps])  # noqa: E731
    bw = types.SimpleNamespace(ev_off=np.concatenate([[0], np.cumsum(lens)]), m_s=np.array(ms),
                               T_s=np.array([p[5] for p in ps]), t=cat(0, np.float64), m=cat(1, np.int32),
                               mu=cat(2, np.float32), alpha=cat(3, np.float32), beta=cat(4, np.float32))
    ll, gmu, ga, gb = [x.cpu().numpy() for x in H.loglik_grad_batched(H.Batch.from_numpy(bw))]
    mo = ao = 0
    for s, (p, M) in enumerate(zip(ps, ms)):
        check((ll[s], gmu[mo:mo + M], ga[ao:ao + M * M].reshape(M, M), gb[s:s + 1]), oracle.forward(*p),
              label=f"sequence {s} of {M} nodes")
        mo, ao = mo + M, ao + M * M
