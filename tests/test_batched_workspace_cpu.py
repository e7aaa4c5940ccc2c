"""The workspace query of batches with more than 8 nodes is enough for every
sequence such a batch can hold (host arithmetic only): the large-M engine's
layout is not monotone in the node count, so the query for max_m nodes has to
cover every smaller node count too."""
import ctypes
import random

import pytest


@pytest.fixture(scope="module")
def H():
    import paper_2604_01342_amd as H
    return H


def large_part(H, n, max_m, grad):
    """What the batched query leaves beside the small-M engine's workspace."""
    L = H.lib()
    small = L.hawkes_batched_workspace_bytes(1, n, 8, grad)
    return L.hawkes_batched_workspace_bytes(1, n, max_m, grad) - (small + 255 & ~255)


def alone(H, n, m, grad):
    return H.lib().hawkes_workspace_bytes(ctypes.byref(H._Problem(n, m, 1, 0, 0, 1.0)), grad)


@pytest.mark.parametrize("n,m,max_m", [(100_000, 80, 81), (1_000_000, 512, 513), (20_000, 1024, 1025),
                                       (1_000, 128, 129), (600_000, 383, 384), (1_000_000, 64, 65)])
def test_next_smaller_node_count_fits(H, n, m, max_m):
    assert large_part(H, n + 10, max_m, 1) >= alone(H, n, m, 1)


@pytest.mark.parametrize("n", [0, 1, 700, 5_000, 20_000, 300_000, 1_000_000, 40_000_000])
@pytest.mark.parametrize("tuning", [{}, {"dense_ranges": 8}, {"dense_ranges": 64, "dense_cols": 64},
                                    {"dense_cols": 256, "dense_rows": 16}])
def test_every_smaller_sequence_fits(H, n, tuning):
    rng = random.Random(n)
    try:
        H.set_tuning(**tuning)
        for max_m in [9, 64, 65, 130, 400, 1100, rng.randint(9, 2200)]:
            for grad in (0, 1):
                have = large_part(H, n, max_m, grad)
                for m in range(9, max_m + 1):
                    assert have >= alone(H, n, m, grad), (max_m, m, grad)
                    k = rng.randint(0, n)
                    assert have >= alone(H, k, m, grad), (max_m, m, k, grad)
    finally:
        H.set_tuning()
