"""The dense dL/dalpha kernels' blocks and tiles at their edges, against the
FP64 oracle (1e-6 relative per output block, as everywhere): node counts around
the tiles of 16 rows, the 64 padded columns, the change from float64 to float32
state rows (384 nodes) and from one column block to several (1024 nodes);
sequences that end at, before and after a block, a group of 64 records and a
segment; every block length; wide blocks (gaps far above 1 / beta) in each of
these; event ranges without events."""
import numpy as np
import pytest

import oracle
from tests.helpers import rand_problem
from tests.test_gpu_parity import H, check, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n,cols", [(65, 1024, 0), (79, 1025, 64), (80, 6143, 128), (81, 65, 256),
                                      (129, 12289, 0), (383, 8255, 0), (384, 8256, 0), (385, 8257, 64),
                                      (400, 255, 128), (513, 4097, 0), (1023, 5000, 0), (1024, 5120, 256),
                                      (1025, 5119, 0), (1100, 5121, 64), (2100, 4000, 128), (3100, 3001, 0)])
def test_blocks_and_tiles(H, M, n, cols):  # noqa: F811
    t, m, mu, alpha, beta, T = rand_problem(500 + M, n, M, ties=True, density=min(1.0, 8.0 / M), rate=40.0)
    try:
        H.set_tuning(dense_cols=cols)
        got = run_gpu(H, t, m, mu, alpha, beta, T, 12)
    finally:
        H.set_tuning()
    check(got, oracle.forward(t, m, mu, alpha, beta, T), label=f"blocks M={M} n={n} cols={cols or 'auto'}")


@pytest.mark.parametrize("M,cols", [(70, 64), (200, 128), (390, 256), (1030, 256)])
def test_wide_blocks(H, M, cols):  # noqa: F811
    rng = np.random.default_rng(M)
    n = 4000
    gaps = rng.exponential(0.05, size=n)
    gaps[rng.random(n) < 0.01] = 300.0
    t = np.cumsum(gaps)
    m = rng.integers(0, M, size=n).astype(np.int32)
    _, _, mu, alpha, beta, _ = rand_problem(31, 10, M)
    T = float(t[-1] + 0.5)
    try:
        H.set_tuning(dense_cols=cols)
        got = run_gpu(H, t, m, mu, alpha, beta, T)
    finally:
        H.set_tuning()
    check(got, oracle.forward(t, m, mu, alpha, beta, T), label=f"wide blocks M={M}")


def test_ranges_without_events(H):  # noqa: F811
    # more event ranges than blocks in the last, short chunk
    t, m, mu, alpha, beta, T = rand_problem(77, 4096 + 70, 90, density=0.1, rate=40.0)
    try:
        H.set_tuning(dense_ranges=4)
        got = run_gpu(H, t, m, mu, alpha, beta, T, 12)
    finally:
        H.set_tuning()
    check(got, oracle.forward(t, m, mu, alpha, beta, T), label="ranges without events")
