"""The per-target engine's dense dL/dalpha and short segments at their edges,
against the FP64 oracle's reverse-mode pass (1e-6 relative per output block):
node counts around the blocks of 128 targets and columns; sequences of fewer
events than waves, with shares that end inside and at a segment, over segments
of 256 and 1024 events and over several chunks; steps between events that the
decay's polynomial takes whole, halved a few times and halved many times."""
import pytest

import oracle
from tests.helpers import rand_problem
from tests.test_gpu_parity import H, check, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n,chunk,rate", [(2, 2, 0, 5.0), (127, 31, 0, 5.0), (128, 511, 0, 5.0), (129, 512, 0, 5.0),
                                            (128, 513, 0, 5000.0), (3, 1025, 0, 0.05), (255, 4097, 0, 20.0),
                                            (256, 8192, 0, 5000.0), (257, 8193, 12, 20.0), (130, 9000, 12, 1e-4),
                                            (100, 20001, 0, 100.0), (385, 12289, 12, 0.5)])
def test_per_target_dense_edges(H, M, n, chunk, rate):  # noqa: F811
    t, m, mu, alpha, beta, T = rand_problem(800 + M + n, n, M, per_target=True, ties=True, density=0.2, rate=rate)
    ref = oracle.adjoint(t, m, mu, alpha, beta, T)
    check(run_gpu(H, t, m, mu, alpha, beta, T, chunk), ref, label=f"per-target M={M} n={n} rate={rate}")
