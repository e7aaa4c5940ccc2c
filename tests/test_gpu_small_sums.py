"""The last sums of batches with up to 8 nodes where one sequence holds most of the items, against the FP64 oracle
(1e-6 relative per output block): one level of sums with up to and above 512 sequences, two levels with chunks of
few items (256 threads) and with full ones among them, and empty sequences in each."""
import types

import numpy as np
import pytest

import oracle
from tests.helpers import rand_problem, scalar_rel
from tests.test_gpu_parity import H, check  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,M,at,long", [(64, 8, 63, 30_000), (100, 1, 0, 29_000), (512, 5, 100, 20_000),
                                         (513, 8, 512, 20_000), (1400, 3, 700, 9_000), (1500, 8, 1499, 60_000),
                                         (2500, 1, 3, 40)])
def test_one_long_sequence(H, S, M, at, long):  # noqa: F811
    lens = np.full(S, 16)
    lens[at] = long
    lens[1] = 0
    ps = [rand_problem(40 + s, max(int(n), 1), M, ties=True, density=0.8, rate=20.0) for s, n in enumerate(lens)]
    cat = lambda k, dt: np.concatenate([np.asarray(p[k], dt).reshape(-1)[:n] if k < 2 else  # noqa: E731
                                        np.asarray(p[k], dt).reshape(-1) for p, n in zip(ps, lens)])
    bw = types.SimpleNamespace(ev_off=np.concatenate([[0], np.cumsum(lens)]), m_s=np.full(S, M),
                               T_s=np.array([p[5] for p in ps]), t=cat(0, np.float64), m=cat(1, np.int32),
                               mu=cat(2, np.float32), alpha=cat(3, np.float32), beta=cat(4, np.float32))
    ll, gmu, ga, gb = [x.cpu().numpy() for x in H.loglik_grad_batched(H.Batch.from_numpy(bw))]
    for s, (p, n) in enumerate(zip(ps, lens)):
        got = (ll[s], gmu[s * M:(s + 1) * M], ga[s * M * M:(s + 1) * M * M].reshape(M, M), gb[s:s + 1])
        if n:
            check(got, oracle.forward(*p), label=f"S={S} sequence {s}")
        else:
            assert scalar_rel(got[0], -p[5] * float(np.sum(p[2], dtype=np.float64))) < 1e-6
            assert np.allclose(got[1], -p[5]) and not got[2].any() and not got[3].any()
