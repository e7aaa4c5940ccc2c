"""The dense dL/dalpha with the state between blocks in float64 from 384 nodes on (dense_rows = 16), against the FP64
oracle (1e-6 relative per output block): one column block and several (384 columns each at most), a last block that
is nearly empty, several event ranges and chunks, and columns of 64 and 128 events a block."""
import pytest

import oracle
from tests.helpers import rand_problem
from tests.test_gpu_parity import H, check, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n,chunk,tuning", [(384, 5_000, 0, {"dense_rows": 16}), (385, 5_000, 0, {"dense_rows": 16}),
                                              (513, 9_000, 12, {"dense_rows": 16, "dense_ranges": 2}),
                                              (768, 5_000, 0, {"dense_rows": 16}), (769, 20_000, 0, {"dense_rows": 16}),
                                              (1153, 3_000, 0, {"dense_rows": 16}), (400, 20_000, 0, {"dense_cols": 64}),
                                              (700, 20_000, 14, {"dense_cols": 128})])
def test_float64_rows(H, M, n, chunk, tuning):  # noqa: F811
    p = rand_problem(60 + M, n, M, ties=True, density=0.02, rate=0.1 * M)
    try:
        H.set_tuning(**tuning)
        got = run_gpu(H, *p, chunk)
    finally:
        H.set_tuning()
    check(got, oracle.forward(*p), label=f"float64 rows M={M} n={n} {tuning}")
