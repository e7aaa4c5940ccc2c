"""The engine for up to 8 nodes at its edges, against the FP64 oracle (1e-6
relative per output block).  One sequence: items in one wave, at 16 and 17
waves (the scan over waves takes 16 at a time), below and above 2048 items
(one or two levels of sums), around 16384 items (four or two lanes an item) and
at the first longer item.  Batches: fewer and
more than 64 sequences (the threads of the last sums), 1024 and 1025 (the
setup's rounds), with empty sequences among them, and more
than 32768 items (two lanes an item at 8 nodes)."""
import types

import numpy as np
import pytest

import oracle
from tests.helpers import rand_problem, scalar_rel
from tests.test_gpu_parity import H, check, dev, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n", [(1, 1), (2, 16), (8, 17), (3, 1024), (5, 1025), (1, 16384), (2, 16385), (4, 17409),
                                 (8, 32735), (8, 32752), (1, 32768), (1, 393231), (2, 393232), (3, 262111), (3, 262144)])
def test_one_sequence(H, M, n):  # noqa: F811
    import torch
    t, m, mu, alpha, beta, T = rand_problem(900 + M + n, n, M, ties=True, density=0.7, rate=20.0)
    ref = oracle.forward(t, m, mu, alpha, beta, T)
    check(run_gpu(H, t, m, mu, alpha, beta, T), ref, label=f"one M={M} n={n}")
    ll = H.loglik(dev(t, torch.float64), dev(m, torch.int32), dev(mu, torch.float32), dev(alpha, torch.float32),
                  dev(beta, torch.float32), T)
    assert scalar_rel(ll.item(), ref[0]) < 1e-6


@pytest.mark.parametrize("S,hi", [(63, 400), (64, 400), (65, 3000), (40, 5000), (1024, 30), (1025, 30), (2100, 20),
                                  (16, 120000)])
def test_batch(H, S, hi):  # noqa: F811
    rng = np.random.default_rng(S)
    lens = rng.integers(1, hi, S)
    lens[rng.integers(0, S, 3)] = 0
    lens[-1] = 0
    ps = [rand_problem(1000 + s, max(int(n), 1), 1 + s % 8, ties=True, density=0.7, rate=20.0)
          for s, n in enumerate(lens)]
    cat = lambda k, dt: np.concatenate([np.asarray(p[k], dt).reshape(-1)[:n] if k < 2 else  # noqa: E731
                                        np.asarray(p[k], dt).reshape(-1) for p, n in zip(ps, lens)])
    bw = types.SimpleNamespace(ev_off=np.concatenate([[0], np.cumsum(lens)]), m_s=np.array([1 + s % 8 for s in range(S)]),
                               T_s=np.array([p[5] for p in ps]), t=cat(0, np.float64), m=cat(1, np.int32),
                               mu=cat(2, np.float32), alpha=cat(3, np.float32),
                               beta=np.array([np.asarray(p[4]).reshape(-1)[0] for p in ps], np.float32))
    ll, gmu, ga, gb = [x.cpu().numpy() for x in H.loglik_grad_batched(H.Batch.from_numpy(bw))]
    mo = ao = 0
    for s, (p, n) in enumerate(zip(ps, lens)):
        M = 1 + s % 8
        got = (ll[s], gmu[mo:mo + M], ga[ao:ao + M * M].reshape(M, M), gb[s:s + 1])
        if n:
            check(got, oracle.forward(*p), label=f"S={S} seq {s}")
        else:
            assert scalar_rel(got[0], -p[5] * float(np.sum(p[2], dtype=np.float64))) < 1e-6
            assert np.allclose(got[1], -p[5]) and not got[2].any() and not got[3].any()
        mo, ao = mo + M, ao + M * M
