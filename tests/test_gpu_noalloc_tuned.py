"""hawkes_loglik_grad_noalloc with the dense kernels' knobs set, whose layout is above the fixed scratch: longer
blocks, fewer ranges and chunks half as long, against the FP64 oracle (1e-6 relative per output block)."""
import pytest
import torch

import oracle
from tests.helpers import rand_problem
from tests.test_gpu_parity import H, check, dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,M,tuning", [(530_000, 100, {"dense_ranges": 4}), (10_978, 886, {"dense_ranges": 64}),
                                        (270_000, 974, {"dense_ranges": 1, "dense_rows": 16})])
def test_fitted_layouts(H, n, M, tuning):  # noqa: F811
    p = rand_problem(n % 97, n, M, density=min(1.0, 10.0 / M), rate=0.2 * M)
    try:
        H.set_tuning(**tuning)
        assert H.workspace_bytes(n, M) > H.NOALLOC_SCRATCH_BYTES
        out = H.loglik_grad_noalloc(dev(p[0], torch.float64), dev(p[1], torch.int32),
                                    *(dev(x, torch.float32) for x in p[2:5]), p[5])
    finally:
        H.set_tuning()
    check([x.cpu().numpy() for x in out], oracle.forward(*p), label=f"noalloc M={M} {tuning}")
