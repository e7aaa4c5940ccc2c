"""The dense dL/dalpha with several column blocks (from 1025 nodes on; its records kept in a list per block of events
and column block), against the FP64 oracle (1e-6 relative per output block): the first node counts with two and three
column blocks and with blocks of 512 and 1024 events, chunks that end inside a block and a group, several chunks;
marks that all fall into one column block (a list of 16 groups) and into one row block (more own events of a block
than one batch of 64, with such lists), blocks too long in time for anchored factors; and several columns a node
below 33 nodes (several decay kernels)."""
import numpy as np
import pytest

import oracle
from tests.helpers import rand_problem
from tests.test_gpu_parity import H, check, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n,chunk,rate,marks", [(1025, 5_000, 0, 100.0, ""), (1200, 1_023, 0, 100.0, ""),
                                                  (1201, 3_001, 0, 100.0, ""), (2048, 5_000, 12, 200.0, ""),
                                                  (2049, 9_000, 12, 200.0, ""), (2304, 1_025, 0, 200.0, ""),
                                                  (2305, 3_000, 0, 200.0, ""), (3073, 2_049, 0, 300.0, ""),
                                                  (2400, 6_000, 0, 200.0, "columns"), (1300, 6_000, 0, 100.0, "columns"),
                                                  (2400, 6_000, 12, 200.0, "rows"), (1100, 6_000, 0, 100.0, "rows"),
                                                  (1300, 3_000, 0, 0.5, ""), (2400, 3_000, 0, 2.0, "columns")])
def test_column_lists(H, M, n, chunk, rate, marks):  # noqa: F811
    t, m, mu, alpha, beta, T = rand_problem(M + n, n, M, ties=True, density=10.0 / M, rate=rate)
    if marks == "columns":
        m = (m % 300 + 100).astype(np.int32)
    elif marks == "rows":
        m = np.where(m % 4 > 0, m % 16 + 32, m).astype(np.int32)
    p = (t, m, mu, alpha, beta, T)
    check(run_gpu(H, *p, chunk), oracle.forward(*p), label=f"lists M={M} n={n} {marks}")


@pytest.mark.parametrize("M,K,n", [(1, 2, 3_000), (2, 3, 3_000), (3, 2, 1_025), (16, 2, 3_000), (31, 2, 3_000),
                                   (32, 2, 3_000), (33, 2, 3_000)])
def test_columns_of_few_nodes(H, M, K, n):  # noqa: F811
    t, m, mu, alpha, _, T = rand_problem(M + K, n, M, ties=True, rate=5.0)
    a = np.stack([alpha * np.float32(0.5 / (k + 1)) for k in range(K)])
    p = (t, m, mu, a, np.array([1.0, 0.2, 5.0][:K], np.float32), T)
    check(run_gpu(H, *p), oracle.forward(*p), label=f"columns M={M} K={K}")
