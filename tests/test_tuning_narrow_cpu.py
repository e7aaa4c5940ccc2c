"""The dense kernels' knobs leave the engine for 9 to 64 nodes and one shared decay alone (host arithmetic only): its
workspace, and with it its workgroups, do not follow them, and the autotuner keeps its shapes apart and times
nothing there."""
import pytest

import paper_2604_01342_amd as H
from paper_2604_01342_amd import autotune as AT


@pytest.mark.parametrize("M", [9, 16, 50, 64])
@pytest.mark.parametrize("grad", [False, True])
def test_dense_knobs_do_not_reach_the_narrow_engine(M, grad):
    base = H.workspace_bytes(1_000_000, M, grad=grad)
    try:
        for tuning in ({"dense_ranges": 4}, {"dense_ranges": 4096}, {"dense_cols": 64}, {"dense_rows": 16}):
            H.set_tuning(**tuning)
            assert H.workspace_bytes(1_000_000, M, grad=grad) == base
    finally:
        H.set_tuning()


def test_shape_classes():
    key = AT.shape_class_single
    assert key(10**6, 64, False, 0) != key(10**6, 65, False, 0)          # one power of two, two engines
    assert key(10**6, 64, False, 0) != key(10**6, 64, False, 0, K=2)
    assert key(10**6, 64, False, 0, K=2) == key(10**6, 65, False, 0)
    # the small engine's settings stay where they were stored
    assert key(10**6, 5, False, 0) == "single|M2|n19|pt0|ch20"
    assert key(10**6, 500, True, 0) == "single|M8|n19|pt1|ch20"
    for M, per_target, K, some in ((9, False, 1, False), (64, False, 1, False), (65, False, 1, True),
                                   (64, False, 2, True), (500, True, 1, False), (5, False, 1, True)):
        assert (AT.candidates_single(10**6, M, per_target, 0, K) != [{}]) == some
