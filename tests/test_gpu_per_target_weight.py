"""The weight with which an own event joins the adjoint state of the per-target dense kernel: it carries its lane in
its 6 lowest mantissa bits, so dL/dalpha of one event pair without any decay is within 2^-46 relative of the exact
value 1 (all events at one time, alpha = 0, mu = beta = 1: w = 1, and the seed and the event count cancel)."""
import pytest
import torch

from tests.test_gpu_parity import H  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [2, 63, 64, 100, 127, 128, 255])
def test_weight_of_one_own_event(H, p):  # noqa: F811
    M, n = 256, 128
    m = torch.full((n,), 1, dtype=torch.int32)
    m[-2], m[-1] = 0, p                      # both in the last wave's share of the events
    one = torch.ones(M, device="cuda")
    _, _, ga, _ = H.loglik_grad(torch.ones(n, dtype=torch.float64).cuda(), m.cuda(), one,
                                torch.zeros(M, M, device="cuda"), one, 1.0)
    # the lane's bits (2^-46) and two roundings of sums near 2 (2^-52 each)
    assert abs(float(ga[p, 0]) - 1.0) <= 2.0 ** -46 + 2.0 ** -51
